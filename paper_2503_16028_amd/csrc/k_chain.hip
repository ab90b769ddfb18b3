// A whole pCN-GM move stage (Alg. 2) in one launch for the problems whose potential a few lanes can
// compute: the closed-form L^2 mixture (Example 1, at most 128 modes) and the 1D Darcy problem (at most
// 256 intervals).  The particles of a stage do not interact, so each particle's lanes run all its moves
// with the state in registers; only the final state goes to memory.
//
// As one launch per step (proposal, potential, decision; four with a synthesis) such a move is a chain
// of small kernels: at N = 20000 and 64 modes 41 us of launches that read and write the state, where
// the arithmetic (dominated by the Box-Muller normals in FP64) takes about 10; at N = 256 in 1D 55 us,
// nearly all of it latency.  Measured per 200-move stage of 20000 particles, M = 8: 7.98 -> 2.60 ms;
// per 10-move stage of 256 particles on 64 intervals: 547 -> 73 us.
//
// The random numbers, the proposal and the decision are those of the step kernels (the proposal and
// its ratio differ from theirs in the order of sums).
#include <algorithm>

#include "common.hpp"

namespace smc {

namespace {

// The partner whose lane index differs by the mask 15, 7, 3 or 1 inside a 16-lane row (row_mirror,
// row_half_mirror and quad permutations): four masks that together reach every lane of the row.
template <int MASK>
__device__ __forceinline__ double row_partner(double v) {
    constexpr int CTRL = MASK == 15 ? 0x140 : MASK == 7 ? 0x141 : MASK == 3 ? 0x1B : 0xB1;
    static_assert(MASK == 15 || MASK == 7 || MASK == 3 || MASK == 1, "row masks");
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, false);
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// Sums of Q = 1, 2, 4, 8 or 16 quantities over a particle's LANES (16 or 64) lanes, one per lane: lane
// `sub` of a row gets the sum of quantity sub / (16 / Q).  Halving the quantities with each step costs
// Q - 1 exchanges and log2(16 / Q) more, where a butterfly per quantity costs 4 Q.
template <int Q, int LANES>
__device__ __forceinline__ double scatter_sum(double (&v)[Q], int sub) {
    auto halve = [&](auto width, auto mask) __attribute__((always_inline)) {
        constexpr int W = decltype(width)::value, MK = decltype(mask)::value;   // W quantities -> W / 2
        const bool up = sub & ((MK + 1) / 2);
#pragma unroll
        for (int i = 0; i < W / 2; ++i) {
            const double keep = up ? v[i + W / 2] : v[i], send = up ? v[i] : v[i + W / 2];
            v[i] = keep + row_partner<MK>(send);
        }
    };
    if constexpr (Q >= 2) halve(std::integral_constant<int, Q>{}, std::integral_constant<int, 15>{});
    else v[0] += row_partner<15>(v[0]);
    if constexpr (Q >= 4) halve(std::integral_constant<int, Q / 2>{}, std::integral_constant<int, 7>{});
    else v[0] += row_partner<7>(v[0]);
    if constexpr (Q >= 8) halve(std::integral_constant<int, Q / 4>{}, std::integral_constant<int, 3>{});
    else v[0] += row_partner<3>(v[0]);
    if constexpr (Q >= 16) halve(std::integral_constant<int, Q / 8>{}, std::integral_constant<int, 1>{});
    else v[0] += row_partner<1>(v[0]);
    double r = v[0];
    if constexpr (LANES == 64) {   // the rows of the wave
        double a, b;
        b = xor_partner<32>(r, a);
        r = a + b;
        b = xor_partner<16>(r, a);
        r = a + b;
    }
    return r;
}

// Log-sum-exp over the lanes of a row reached by the masks below 2 W (W = 8: the row's half), every lane
// holding one value (-inf for none).
template <int W>
__device__ __noinline__ double row_lse(double x) {
    double mx = x;
    if constexpr (W >= 16) mx = fmax(mx, row_partner<15>(mx));
    mx = fmax(mx, row_partner<7>(mx));
    mx = fmax(mx, row_partner<3>(mx));
    mx = fmax(mx, row_partner<1>(mx));
    double e = (x > -INFINITY) ? exp(x - mx) : 0.0;
    if constexpr (W >= 16) e += row_partner<15>(e);
    e += row_partner<7>(e);
    e += row_partner<3>(e);
    e += row_partner<1>(e);
    return mx + log(e);
}

// The mixture of a stage as its moves use it, in LDS: per component and mode (1 - gamma) mean, 1 / scale
// and beta sqrt(scale) (0, 1 and beta on the modes the mixture leaves alone, where the forward and
// reverse terms of the ratio cancel exactly; 0, 1 and 0 past K, where everything stays zero), the log
// weights less half the log determinants, and the running weight sums that pick a component.  Rows of
// KP modes and MB components, so that a lane reads its modes at immediate offsets.
template <int MB, int KP>
struct ChainMix {
    static constexpr int DOUBLES = 3 * MB * KP + 2 * MAX_M;
    double2* mi;      // [MB][KP]: (1 - gamma) mean, 1 / scale
    double* bs;       // [MB][KP]: beta sqrt(scale)
    double* lw;       // [MAX_M]
    double* cumw;     // [MAX_M]
    __device__ __forceinline__ explicit ChainMix(double* at)
        : mi(reinterpret_cast<double2*>(at)), bs(at + 2 * MB * KP), lw(bs + MB * KP), cumw(lw + MAX_M) {}

    // Fill the tables (every thread of the workgroup; barriers inside).
    __device__ __forceinline__ void fill(const MoveParams& q, const int32_t* __restrict__ slot, int K, double beta,
                                         double gamma) const {
        const int M = q.M, kr = q.kr, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
        for (int i = threadIdx.x; i < MB * KP; i += blockDim.x) {
            const int m = i / KP, k = i % KP, sl = k < K && m < M ? slot[k] : -1;
            const double mean = sl >= 0 ? q.mean[m * kr + sl] : 0.0, s = sl >= 0 ? q.scale[m * kr + sl] : 1.0;
            mi[i] = make_double2((1.0 - gamma) * mean, 1.0 / s);
            bs[i] = k < K ? beta * sqrt(s) : 0.0;
        }
        for (int m = wave; m < M; m += nw) {
            const double h = wave_sum(lane < kr ? 0.5 * log(q.scale[m * kr + lane]) : 0.0);
            if (lane == 0) lw[m] = q.logw[m] - h;
        }
        if (threadIdx.x < MAX_M) cumw[threadIdx.x] = (int)threadIdx.x < M ? exp(q.logw[threadIdx.x]) : 0.0;
        __syncthreads();
        if (threadIdx.x == 0)   // the running sum of choose_component, so the same component is picked
            for (int m = 1; m < M; ++m) cumw[m] += cumw[m - 1];
        __syncthreads();
    }
};

// Functions of their own: inlined into the loop over the moves, the constants of their polynomials are
// hoisted out of it and take more registers than everything else (235 instead of under 128).
__device__ __noinline__ double2 chain_normals(uint64_t seed, uint64_t ctr, uint32_t block, uint32_t particle) {
    double2 z;
    box_muller(draw(seed, ctr, block, particle), z.x, z.y);
    return z;
}

// The draws a move shares between a particle's lanes, made for 16 moves at a time (lane sub of a row: move
// base + sub): the component and the log of the acceptance uniform.
struct MoveDraw {
    int comp;
    double log_ua;
};
template <typename MIX>
__device__ __forceinline__ MoveDraw move_draw(const MoveParams& q, uint64_t ctr, int64_t n, const MIX& t) {
    const uint4 w = draw(q.seed, ctr, UNIFORM_BLOCK, (uint32_t)n);
    const double uc = res53(w.x, w.y);
    int j = q.M - 1;
    for (int m = 0; m < q.M; ++m)
        if (t.cumw[m] > uc) {
            j = m;
            break;
        }
    return MoveDraw{j, log(res53(w.z, w.w))};
}
__device__ __forceinline__ MoveDraw move_draw_of(const MoveDraw& d, int which) {   // which: lane of the row
    const long long b = __double_as_longlong(d.log_ua);
    const int lo = __shfl((int)b, which, 16), hi = __shfl((int)(b >> 32), which, 16);
    return MoveDraw{__shfl(d.comp, which, 16),
                    __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo))};
}

// Both exponents' terms of one mode for every component: the reverse displacement d1 = xi - gamma v and
// the forward one d2 = v - gamma xi, alpha_j summing d^2 - (d - (1 - gamma) m)^2 / s.  mi: the mode's column.
template <int MB, int KP>
__device__ __forceinline__ void ratio_terms(double x, double v, double gamma, const double2* __restrict__ mi,
                                            double (&pf)[MB], double (&pb)[MB]) {
#pragma clang fp contract(off)
    const double d1 = x - gamma * v, d2 = v - gamma * x;
    const double s1 = d1 * d1, s2 = d2 * d2;
#pragma unroll
    for (int m = 0; m < MB; ++m) {
        const double2 ms = mi[m * KP];
        const double e1 = d1 - ms.x, e2 = d2 - ms.x;
        pf[m] += s1 - e1 * e1 * ms.y;
        pb[m] += s2 - e2 * e2 * ms.y;
    }
}

// log R from the per-lane sums: the difference of the log-sum-exps over the components.
template <int MB, int LANES, typename MIX>
__device__ __forceinline__ double log_ratio(double (&pf)[MB], double (&pb)[MB], double inv2b2, const MIX& t, int M,
                                            int sub) {
    if constexpr (MB == 16) {
        const double f = scatter_sum<16, LANES>(pf, sub), b = scatter_sum<16, LANES>(pb, sub);
        const double lw = sub < M ? t.lw[sub] : -INFINITY;
        return row_lse<16>(lw + f * inv2b2) - row_lse<16>(lw + b * inv2b2);
    } else {   // lanes 0 - 7 of a row take the forward sums, 8 - 15 the backward ones
        double v[2 * MB];
#pragma unroll
        for (int m = 0; m < MB; ++m) {
            v[m] = pf[m];
            v[MB + m] = pb[m];
        }
        const double s = scatter_sum<2 * MB, LANES>(v, sub);
        constexpr int PER = 8 / MB;   // lanes that hold the same component
        const int m = (sub & 7) / PER;
        // one lane of each component enters the sum
        const double x = (m < M && (sub & 7) % PER == 0) ? t.lw[m] + s * inv2b2 : -INFINITY;
        const double l = row_lse<8>(x), o = row_partner<15>(l);
        return (sub & 8) ? o - l : l - o;
    }
}

__device__ __forceinline__ bool accepted(double tau, double phi, double pn, double lr, double log_ua) {
    if (!isfinite(pn) || !(lr > -INFINITY)) return false;
    return log_ua < fmin(0.0, tau * (phi - pn) + lr);
}

}  // namespace

// L^2 mixture: sixteen lanes per particle; a lane owns normal blocks sub, sub + 16, ... (NBL of them, two
// modes each).  TB >= T likelihood terms.
template <int MB, int NBL, int TB>
__global__ __launch_bounds__(256) void chain_l2mix_kernel(int64_t N, int K, int n_moves, MoveParams q,
                                                          const int32_t* __restrict__ slot,
                                                          const double* __restrict__ sqrt_lam,
                                                          const double* __restrict__ c, int T, double inv2s2,
                                                          double* __restrict__ xi, double* __restrict__ phi,
                                                          int32_t* __restrict__ n_acc, int32_t* flags) {
    extern __shared__ double smem[];
    const double beta = mp_beta(q, 0), tau = mp_tau(q, 0);
    const int sub = threadIdx.x & 15;
    const int64_t n = (int64_t)blockIdx.x * (blockDim.x >> 4) + (threadIdx.x >> 4);
    const bool live = n < N;
    if (!mp_valid(beta, tau)) {   // every proposal would be rejected
        if (live && sub == 0) n_acc[n] = 0;
        if (blockIdx.x == 0 && threadIdx.x == 0 && flags) atomicOr(flags, SMC_FLAG_BADPARAM);
        return;
    }
    const double gamma = sqrt(1.0 - beta * beta), inv2b2 = 0.5 / (beta * beta);
    const int M = q.M;
    constexpr int KP = 32 * NBL;
    const ChainMix<MB, KP> t(smem);
    double* ct = smem + t.DOUBLES;   // [TB][KP] likelihood centres
    for (int i = threadIdx.x; i < TB * KP; i += blockDim.x)
        ct[i] = (i / KP < T && i % KP < K) ? c[(i / KP) * K + i % KP] : 0.0;
    t.fill(q, slot, K, beta, gamma);   // its barriers publish ct too
    if (!live) return;
    const uint64_t ctr = mp_ctr(q);
    double x[2 * NBL], sl[2 * NBL];   // the lane's modes 2 (sub + 16 b) + h, zero past K
#pragma unroll
    for (int i = 0; i < 2 * NBL; ++i) {
        const int k = 2 * (sub + 16 * (i >> 1)) + (i & 1);
        x[i] = k < K ? xi[n * K + k] : 0.0;
        sl[i] = k < K ? sqrt_lam[k] : 0.0;
    }
    double ph = phi[n];
    int acc = 0;
    MoveDraw dr{};
    for (int m = 0; m < n_moves; ++m) {
        if ((m & 15) == 0) dr = move_draw(q, ctr + m + sub, n, t);
        const MoveDraw d = move_draw_of(dr, m & 15);
        double v[2 * NBL], pf[MB], pb[MB], dist[TB];
#pragma unroll
        for (int j = 0; j < MB; ++j) pf[j] = pb[j] = 0.0;
#pragma unroll
        for (int i = 0; i < TB; ++i) dist[i] = 0.0;
#pragma unroll
        for (int b = 0; b < NBL; ++b) {
            const double2 z = chain_normals(q.seed, ctr + m, (uint32_t)(sub + 16 * b), (uint32_t)n);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int i = 2 * b + h, k = 2 * (sub + 16 * b) + h;
                asm volatile("" ::: "memory");   // each mode's tables are read anew: hoisted, they spill
                v[i] = gamma * x[i] + t.mi[d.comp * KP + k].x + t.bs[d.comp * KP + k] * (h ? z.y : z.x);
                ratio_terms<MB, KP>(x[i], v[i], gamma, t.mi + k, pf, pb);
                const double u = sl[i] * v[i];
#pragma unroll
                for (int e = 0; e < TB; ++e) {
                    const double w = u - ct[e * KP + k];
                    dist[e] += w * w;
                }
            }
        }
        const double lr = log_ratio<MB, 16>(pf, pb, inv2b2, t, M, sub);
        // Phi = -log sum_i exp(-dist_i / (2 sigma^2)), one term per lane (copies of a term masked)
        const double ds = scatter_sum<TB, 16>(dist, sub);
        constexpr int PER = 16 / TB;
        const double pn = -row_lse<16>((sub / PER < T && sub % PER == 0) ? -ds * inv2s2 : -INFINITY);
        if (accepted(tau, ph, pn, lr, d.log_ua)) {   // the same in every lane of the particle
#pragma unroll
            for (int i = 0; i < 2 * NBL; ++i) x[i] = v[i];
            ph = pn;
            ++acc;
        }
    }
#pragma unroll
    for (int i = 0; i < 2 * NBL; ++i) {
        const int k = 2 * (sub + 16 * (i >> 1)) + (i & 1);
        if (k < K) xi[n * K + k] = x[i];
    }
    if (sub == 0) {
        phi[n] = ph;
        n_acc[n] = acc;
    }
}

// Every workgroup fills the mixture's tables for its sixteen particles, which for a large cloud costs up to a
// move or two, most with sixteen components and where the lanes' 64 or 128 modes are not filled.  So the
// step kernels, which have one table for all, keep the calls of one or two moves where they are the faster:
// at 262144 particles and one move, with 16 modes and M = 16 326 us by steps and 472 in one launch; with 64
// modes and M = 8 it is 451 and 273.  From four moves the one launch was faster in every combination measured.
bool chain_l2mix_wanted(int64_t N, int K, int T, int M, int n_moves) {
    if (K > 128) return false;
    if (N <= 32768 || n_moves > 2) return true;
    if (n_moves == 2) return M <= 8 || (K > 48 && K <= 64);
    return M <= 8 && ((K > 48 && K <= 64) || (K > 96 && T <= 4));
}

template <int MB, int NBL>
static void chain_l2mix_terms(int64_t N, int K, int n_moves, const MoveParams& q, const int32_t* slot,
                              const double* sqrt_lam, const double* c, int T, double inv2s2, double* xi, double* phi,
                              int32_t* n_acc, int32_t* flags, int n_cu, hipStream_t s) {
    // Four particles per wave.  While there are fewer waves than SIMDs each takes a workgroup of its own
    // (a compute unit's other SIMDs and LDS stay free for it); beyond, four waves share one's tables.
    const unsigned threads = N <= (int64_t)16 * n_cu ? 64u : 256u;
    const dim3 grid((unsigned)((N * 16 + threads - 1) / threads));
    const size_t lds = sizeof(double) * (size_t)(ChainMix<MB, 32 * NBL>::DOUBLES + (T <= 4 ? 4 : 16) * 32 * NBL);
    if (T <= 4)
        chain_l2mix_kernel<MB, NBL, 4><<<grid, dim3(threads), lds, s>>>(N, K, n_moves, q, slot, sqrt_lam, c, T, inv2s2, xi,
                                                                     phi, n_acc, flags);
    else
        chain_l2mix_kernel<MB, NBL, 16><<<grid, dim3(threads), lds, s>>>(N, K, n_moves, q, slot, sqrt_lam, c, T, inv2s2,
                                                                      xi, phi, n_acc, flags);
}

template <int NBL>
static void chain_l2mix_mix(int64_t N, int K, int n_moves, const MoveParams& q, const int32_t* slot,
                            const double* sqrt_lam, const double* c, int T, double inv2s2, double* xi, double* phi,
                            int32_t* n_acc, int32_t* flags, int n_cu, hipStream_t s) {
    auto run = [&](auto mb) {
        chain_l2mix_terms<decltype(mb)::value, NBL>(N, K, n_moves, q, slot, sqrt_lam, c, T, inv2s2, xi, phi, n_acc, flags,
                                                  n_cu, s);
    };
    if (q.M == 1) run(std::integral_constant<int, 1>{});
    else if (q.M <= 4) run(std::integral_constant<int, 4>{});
    else if (q.M <= 8) run(std::integral_constant<int, 8>{});
    else run(std::integral_constant<int, 16>{});
}

hipError_t launch_chain_l2mix(int64_t N, int K, int n_moves, const MoveParams& q, const int32_t* slot,
                              const double* sqrt_lam, const double* c, int T, double inv2s2, double* xi, double* phi,
                              int32_t* n_acc, int32_t* flags, int n_cu, hipStream_t s) {
    if (N <= 0) return hipSuccess;
    if (K <= 64)
        chain_l2mix_mix<2>(N, K, n_moves, q, slot, sqrt_lam, c, T, inv2s2, xi, phi, n_acc, flags, n_cu, s);
    else
        chain_l2mix_mix<4>(N, K, n_moves, q, slot, sqrt_lam, c, T, inv2s2, xi, phi, n_acc, flags, n_cu, s);
    return hipGetLastError();
}

// 1D Darcy: one wave per particle, lane l owning mode l (K <= 64) and, of every 64 nodes, node l.  The
// basis, mode-major, sits in LDS beside the mixture.  The solve is solve1d_kernel's closed form with the
// sums over the faces as wave sums and the states at the faces as a scan.
__device__ __forceinline__ double wave_scan(double v, int lane) {   // inclusive
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const double o = __shfl_up(v, off, 64);
        if (lane >= off) v += o;
    }
    return v;
}

template <int MB, int NC>   // NC chunks of 64 nodes (n <= 64 NC)
__global__ __launch_bounds__(1024) void chain1d_kernel(int64_t N, int K, int n, int n_moves, MoveParams q,
                                                       const int32_t* __restrict__ slot,
                                                       const double* __restrict__ sqrt_lam,
                                                       const double* __restrict__ basis, SolveArgs a,
                                                       double* __restrict__ xi, double* __restrict__ phi,
                                                       int32_t* __restrict__ n_acc, int32_t* flags) {
    extern __shared__ double smem[];
    const double beta = mp_beta(q, 0), tau = mp_tau(q, 0);
    const int lane = threadIdx.x & 63, sub = lane & 15, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const int64_t p = (int64_t)blockIdx.x * waves + wave;
    const bool live = p < N;
    if (!mp_valid(beta, tau)) {   // every proposal would be rejected
        if (live && lane == 0) n_acc[p] = 0;
        if (blockIdx.x == 0 && threadIdx.x == 0 && flags) atomicOr(flags, SMC_FLAG_BADPARAM);
        return;
    }
    const double gamma = sqrt(1.0 - beta * beta), inv2b2 = 0.5 / (beta * beta);
    const int M = q.M;
    const ChainMix<MB, 64> t(smem);
    double* B = smem + t.DOUBLES;                        // [K][n + 1]
    double* cs = B + (size_t)K * (n + 1) + wave * 64;    // the wave's coefficients
    for (int i = threadIdx.x; i < K * (n + 1); i += blockDim.x) {
        const int node = i / K, k = i - node * K;
        B[k * (n + 1) + node] = basis[i];
    }
    t.fill(q, slot, K, beta, gamma);            // its barriers publish B too
    if (!live) return;                          // whole waves; no barrier below
    const uint64_t ctr = mp_ctr(q);
    const bool in = lane < K;
    const double sl = in ? sqrt_lam[lane] : 0.0, h = 1.0 / n;
    double x = in ? xi[p * K + lane] : 0.0, ph = phi[p];
    const int ob = lane < a.n_obs ? a.obs[lane] : 0;
    const double y = lane < a.n_obs ? a.y[lane] : 0.0;
    int acc = 0;
    MoveDraw dr{};
    for (int m = 0; m < n_moves; ++m) {
        if ((m & 15) == 0) dr = move_draw(q, ctr + m + sub, p, t);
        const MoveDraw d = move_draw_of(dr, m & 15);
        asm volatile("" ::: "memory");   // the tables are read anew: hoisted into registers they spill
        double pf[MB], pb[MB];
        const double2 zz = chain_normals(q.seed, ctr + m, (uint32_t)(lane >> 1), (uint32_t)p);
        const double z = (lane & 1) ? zz.y : zz.x;
#pragma unroll
        for (int j = 0; j < MB; ++j) pf[j] = pb[j] = 0.0;
        const double v = gamma * x + t.mi[d.comp * 64 + lane].x + t.bs[d.comp * 64 + lane] * z;   // 0 past K
        ratio_terms<MB, 64>(x, v, gamma, t.mi + lane, pf, pb);
        const double lr = log_ratio<MB, 64>(pf, pb, inv2b2, t, M, sub);
        // exp(u / 2) at the lane's nodes (and, for the last chunk's last face, at node n)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the wave's own LDS, in order
        if (in) cs[lane] = sl * v;
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        double u[NC], un[NC];   // node 64 ch + lane, and the node after it
#pragma unroll
        for (int ch = 0; ch < NC; ++ch) u[ch] = 0.0;
        double last = 0.0;
#pragma unroll 4
        for (int k = 0; k < K; ++k) {
            const double ck = cs[k];
#pragma unroll
            for (int ch = 0; ch < NC; ++ch) {
                const int node = 64 * ch + lane;
                u[ch] = fma(B[k * (n + 1) + (node < n ? node : n)], ck, u[ch]);
            }
            last = fma(B[k * (n + 1) + n], ck, last);
        }
        const double en = exp(0.5 * last);
#pragma unroll
        for (int ch = 0; ch < NC; ++ch) u[ch] = exp(0.5 * u[ch]);
#pragma unroll
        for (int ch = 0; ch < NC; ++ch) {   // the next chunk's first node for lane 63; node n past the end
            const double first = ch + 1 < NC ? __shfl(u[ch + 1 < NC ? ch + 1 : ch], 0, 64) : en;
            const double o = __shfl_down(u[ch], 1, 64);
            un[ch] = lane == 63 ? first : o;
            if (64 * ch + lane == n - 1) un[ch] = en;
        }
        double ia[NC], s1 = 0.0, s0 = 0.0;
#pragma unroll
        for (int ch = 0; ch < NC; ++ch) {
            const int k = 64 * ch + lane;
            ia[ch] = k < n ? 1.0 / (u[ch] * un[ch]) : 0.0;   // 1 / face coefficient a_{k+1/2}
            s1 += k * h * a.f * ia[ch];
            s0 += ia[ch];
        }
        const double F0 = wave_sum(s1) / wave_sum(s0);
        double carry = 0.0, val = 0.0;
#pragma unroll
        for (int ch = 0; ch < NC; ++ch) {   // w at node k + 1 in lane k of the chunk
            const int k = 64 * ch + lane;
            const double w = carry + wave_scan(k < n ? h * (F0 - k * h * a.f) * ia[ch] : 0.0, lane);
            carry = __shfl(w, 63, 64);
            const double at = __shfl(w, (ob - 1) & 63, 64);   // observed nodes are interior: 1 .. n - 1
            if ((ob - 1) >> 6 == ch) val = at;
        }
        const double dl = lane < a.n_obs ? val - y : 0.0;
        const double pn = wave_sum(dl * dl) * a.inv2s2;
        if (accepted(tau, ph, pn, lr, d.log_ua)) {   // the same in every lane
            x = v;
            ph = pn;
            ++acc;
        }
    }
    if (in) xi[p * K + lane] = x;
    if (lane == 0) {
        phi[p] = ph;
        n_acc[p] = acc;
    }
}

// Largest LDS a workgroup may take, and what one of `waves` waves needs.
constexpr size_t CHAIN_LDS = 160 * 1024;
static size_t chain1d_lds(int n, int K, int M, int waves) {
    const int MB = M == 1 ? 1 : M <= 4 ? 4 : M <= 8 ? 8 : 16;
    return sizeof(double) * (size_t)(3 * MB * 64 + 2 * MAX_M + K * (n + 1) + 64 * waves);
}
static int chain1d_waves(int64_t N, int n, int n_cu) { return N <= n_cu ? 1 : n <= 64 ? 4 : n <= 128 ? 8 : 16; }

// Grids whose basis fits LDS beside the mixture and the waves' coefficients.  For a large cloud each workgroup
// of four particles pays for its tables (about 1 ns a particle and 0.1 per component, at the device's rate), and
// a move gains by the nodes, a wave being idle beyond them: nothing on 8 intervals, 0.4 ns a particle on
// 16, 0.8 on 32.  The step kernels keep the calls whose moves do not pay for the tables: 262144
// particles on 8 intervals, 8 modes, M = 16, one move 445 us by steps and 1105 in one launch (16 moves 6.7 and
// 8.7 ms); on 32 intervals, 64 modes, M = 8 one move is 1.30 and 1.06 ms.  The lines are drawn through 1440 such
// pairs so that one launch is nowhere the slower by more than 3 %.
bool chain1d_wanted(int64_t N, int n, int K, int M, int n_moves) {
    if (n > 256 || K > 64 || chain1d_lds(n, K, M, 16) > CHAIN_LDS) return false;
    const int64_t m = n_moves;
    if (N <= 8192) return true;
    if (N <= 32768) return 2 * m * (n - 4) > std::max(8, 3 * M);
    return m * (n - 8) * (16 + K) >= (M <= 4 ? 1100 : M <= 8 ? 1600 : 4600);
}

hipError_t launch_chain1d(int64_t N, int K, int n, int n_moves, const MoveParams& q, const int32_t* slot,
                          const double* sqrt_lam, const double* basis, const SolveArgs& a, double* xi, double* phi,
                          int32_t* n_acc, int32_t* flags, int n_cu, hipStream_t s) {
    if (N <= 0) return hipSuccess;
    // one particle per compute unit while there are enough units (its reads of the basis then have the
    // unit's LDS to themselves); beyond, as many waves as share one copy of the basis
    const int waves = chain1d_waves(N, n, n_cu);
    const dim3 grid((unsigned)((N + waves - 1) / waves)), block(64 * waves);
    const size_t lds = chain1d_lds(n, K, q.M, waves);
    auto chunks = [&](auto mb, auto nc) {
        chain1d_kernel<decltype(mb)::value, decltype(nc)::value><<<grid, block, lds, s>>>(
            N, K, n, n_moves, q, slot, sqrt_lam, basis, a, xi, phi, n_acc, flags);
    };
    auto run = [&](auto mb) {
        if (n <= 64) chunks(mb, std::integral_constant<int, 1>{});
        else if (n <= 128) chunks(mb, std::integral_constant<int, 2>{});
        else chunks(mb, std::integral_constant<int, 4>{});
    };
    if (q.M == 1) run(std::integral_constant<int, 1>{});
    else if (q.M <= 4) run(std::integral_constant<int, 4>{});
    else if (q.M <= 8) run(std::integral_constant<int, 8>{});
    else run(std::integral_constant<int, 16>{});
    return hipGetLastError();
}

// LDS limits above the default, set once (launches may be captured).
hipError_t prepare_chain_kernels() {
    hipError_t e = hipSuccess;
    auto ck = [&](const void* f) {
        if (e == hipSuccess) e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)CHAIN_LDS);
    };
    auto mb = [&](auto m) {
        constexpr int MB = decltype(m)::value;
        ck((const void*)chain_l2mix_kernel<MB, 2, 4>);
        ck((const void*)chain_l2mix_kernel<MB, 2, 16>);
        ck((const void*)chain_l2mix_kernel<MB, 4, 4>);
        ck((const void*)chain_l2mix_kernel<MB, 4, 16>);
        ck((const void*)chain1d_kernel<MB, 1>);
        ck((const void*)chain1d_kernel<MB, 2>);
        ck((const void*)chain1d_kernel<MB, 4>);
    };
    mb(std::integral_constant<int, 1>{});
    mb(std::integral_constant<int, 4>{});
    mb(std::integral_constant<int, 8>{});
    mb(std::integral_constant<int, 16>{});
    return e;
}

}  // namespace smc
