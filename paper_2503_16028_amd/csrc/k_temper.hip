// Re-weighting, next temperature and systematic resampling (Alg. 1; App. C): a few reductions over N
// values.  A small cloud takes one workgroup (the cost is the latency of a pass); a larger one a chain
// of launches over the whole device, one per reduction: each workgroup first folds the partial sums of the
// launch before, in one fixed order, so all of them take the same decision without a grid-wide wait.
#include <algorithm>

#include "common.hpp"
#include "stage_graph.hpp"

namespace smc {

namespace {

// ------------------------------------------------------------------ next temperature
// ESS(h) = (sum W)^2 / sum W^2 with W_n = exp(-h d_n), d_n = Phi_n - Phi_min; non-finite Phi weigh 0.
// One pass gives S1 = sum W, S2 = sum W^2, D1 = sum d W and D2 = sum d W^2, so that
//   f(h) = log(ESS(h) / (rho N)) = log(S1^2 / (S2 rho N)),   f'(h) = -2 D1 / S1 + 2 D2 / S2.
// The first pass takes S1 and S2 at the whole remaining step and, of h = 0, the number of finite
// potentials, sum d and sum d^2, whose ESS and variance give the first point.
struct Sums {
    double v[5];
};
constexpr int S1 = 0, S2 = 1, D1 = 2, D2 = 3;        // of a point
constexpr int CNT = 2, SUM_D = 3, SUM_DD = 4;        // of the first pass, beside S1 and S2

// A search for h between passes.  The next increment in (0, 1 - tau]: the whole remaining step if its ESS
// passes, else the root of the decreasing f, kept in a bracket [lo, hi] with f(lo) >= 0 > f(hi).  The
// first point is the root of the expansion f(h) ~ f(0) - h^2 Var(d); then Newton steps in log h (ESS
// falls off like a power of h for spread-out potentials), replaced by the bracket's geometric (or
// arithmetic) mean whenever a step would leave the bracket.  It ends when the bracket is 2^-52 relative or
// the bisection resolution (1 - tau) 2^-64 wide; a point that Newton's step would move by no more than a few such
// widths is therefore left for its other side, 1, 4, 16 ... widths away, until both ends are near the root.  The
// returned h always has f(h) >= 0, ESS >= rho N, as the lower end of a bisection would; about 11 passes replace 66.
enum TemperMode { MODE_FIRST = 0, MODE_NEWTON = 1, MODE_DONE = 2, MODE_NONE = 3 };   // NONE: no finite potential
struct Temper {
    double pmin, tau, lo, hi, x, s1, reach;   // s1: sum W at lo
    int mode, it, last;

    __device__ __forceinline__ void first(const Sums& e, double goal) {   // goal: rho N
        const double rest = 1.0 - tau;
        if (e.v[S1] * e.v[S1] / (e.v[S2] * goal) >= 1.0) {
            lo = rest;
            s1 = e.v[S1];
            last = 1;
            mode = MODE_DONE;
            return;
        }
        lo = 0.0;
        hi = rest;
        s1 = e.v[CNT];
        reach = 1.0;
        it = 0;
        mode = MODE_NEWTON;
        const double f0 = log(e.v[CNT] / goal), m = e.v[SUM_D] / e.v[CNT], v = e.v[SUM_DD] / e.v[CNT] - m * m;
        x = (v > 0.0 && f0 > 0.0) ? fmin(sqrt(f0 / v), 0.5 * rest) : 0.5 * rest;
    }
    __device__ __forceinline__ void step(const Sums& e, double goal) {
        const double fx = log(e.v[S1] * e.v[S1] / (e.v[S2] * goal)), floor_w = (1.0 - tau) * 0x1p-64;
        const bool pass = fx >= 0.0;
        if (pass) {
            lo = x;
            s1 = e.v[S1];
        } else {
            hi = x;
        }
        mode = MODE_DONE;
        if (!(hi - lo > fmax(floor_w, hi * 0x1p-52)) || ++it >= 96) return;
        const double dfx = -2.0 * e.v[D1] / e.v[S1] + 2.0 * e.v[D2] / e.v[S2];
        const double st = -fx / (dfx * x), width = fmax(floor_w, x * 0x1p-52);
        double xn = (fabs(st) < 50.0) ? x * exp(st) : NAN;   // Newton in log h
        if (fabs(xn - x) <= 4.0 * width) {                    // next to the root: to its other side
            xn = reach > 4096.0 ? NAN : pass ? x + reach * width : x - reach * width;
            reach *= 4.0;
        }
        if (!(xn > lo && xn < hi)) xn = lo > 0.0 && hi > 2.0 * lo ? sqrt(lo * hi) : 0.5 * (lo + hi);
        if (!(xn > lo && xn < hi)) return;   // neighbouring doubles
        x = xn;
        mode = MODE_NEWTON;
    }
};

// One particle's share of a pass at x (first pass: of the points 1 - tau, given as x, and 0), without a
// branch, so that the exponentials of several particles overlap.
template <bool FIRST>
__device__ __forceinline__ void add_point(Sums& e, double p, double pmin, double x) {
    const bool fin = isfinite(p);
    const double d = fin ? p - pmin : 0.0;
    const double y = exp(-x * d), w = fin ? y : 0.0;
    e.v[S1] += w;
    e.v[S2] = __builtin_fma(w, w, e.v[S2]);   // the same bits in every pass
    if constexpr (FIRST) {
        e.v[CNT] += fin ? 1.0 : 0.0;
        e.v[SUM_D] += d;
        e.v[SUM_DD] += d * d;
    } else {
        e.v[D1] += d * w;
        e.v[D2] += d * (w * w);
    }
}
// Entries beg, beg + step, ... of p.
template <bool FIRST>
__device__ __forceinline__ Sums add_points(const double* __restrict__ p, int64_t beg, int64_t N, int64_t step,
                                           double pmin, double x) {
    Sums e{};
    int64_t k = beg;
    for (; k + 3 * step < N; k += 4 * step) {
        double v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = p[k + i * step];
#pragma unroll
        for (int i = 0; i < 4; ++i) add_point<FIRST>(e, v[i], pmin, x);
    }
    for (; k < N; k += step) add_point<FIRST>(e, p[k], pmin, x);
    return e;
}

// Sums over a workgroup of NT threads, the same value in every thread.
template <int NT>
__device__ __forceinline__ Sums block_sums(Sums e, double (*red)[5]) {
#pragma unroll
    for (int i = 0; i < 5; ++i) e.v[i] = wave_sum(e.v[i]);
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int i = 0; i < 5; ++i) red[threadIdx.x >> 6][i] = e.v[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) t += red[w][i];
        e.v[i] = uniform(t);
    }
    __syncthreads();   // red is reused by the next pass
    return e;
}
template <int NT>
__device__ __forceinline__ double block_min(double v, double (*red)[5]) {
    v = -wave_max(-v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][0] = v;
    __syncthreads();
    double m = INFINITY;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) m = fmin(m, red[w][0]);
    __syncthreads();
    return uniform(m);
}

__device__ __forceinline__ double finite_min(double m, double p) { return isfinite(p) ? fmin(m, p) : m; }

// The scalars of a finished search (one thread).
__device__ __forceinline__ void temper_scalars(const Temper& t, int64_t N, double* h_out, double* tau_out,
                                               double* log_z, int32_t* flags) {
    if (t.mode == MODE_NONE) {   // nothing to weigh
        *h_out = 0.0;
        *tau_out = t.tau;
        *log_z = -INFINITY;
        if (flags) atomicOr(flags, SMC_FLAG_NONFINITE);
        return;
    }
    *h_out = t.lo;
    *tau_out = t.last ? 1.0 : t.tau + t.lo;
    *log_z = -t.lo * t.pmin + log(t.s1) - log((double)N);
    if (t.lo == 0.0 && 1.0 - t.tau > 0.0 && flags) atomicOr(flags, SMC_FLAG_STALL);   // tau = 1: nothing left
}
__device__ __forceinline__ double weight(double p, const Temper& t, double ls1) {
    return (t.mode != MODE_NONE && isfinite(p)) ? exp(-t.lo * (p - t.pmin) - ls1) : 0.0;
}

}  // namespace

// One workgroup.  CACHED: the d_n sit in LDS (-1 for a non-finite potential), N <= TEMPER_ONE; else
// each pass reads the potentials.  Four waves when cached: a pass then costs the exponentials of N / 256
// particles a lane and one wave's reductions per SIMD; with sixteen, four waves' reductions and decisions share
// each SIMD and cost more than the exponentials (4096 particles: 85 us with sixteen waves and 16 passes, 33
// with four and 11).
constexpr int TEMPER_ONE = 8064;   // 63 KB
template <int NT, bool CACHED>
__global__ __launch_bounds__(NT) void temper_kernel(int64_t N, const double* __restrict__ phi,
                                                    const double* __restrict__ tau_in, double goal,
                                                    double* __restrict__ h_out, double* __restrict__ tau_out,
                                                    double* W, double* __restrict__ log_z,
                                                    int32_t* __restrict__ flags) {
    extern __shared__ double dl[];
    __shared__ double red[NT / 64][5];
    const int tid = threadIdx.x;
    Temper t{};
    t.pmin = INFINITY;
    for (int64_t k = tid; k < N; k += NT) {
        const double p = phi[k];
        if constexpr (CACHED) dl[k] = p;
        t.pmin = finite_min(t.pmin, p);
    }
    t.pmin = block_min<NT>(t.pmin, red);
    t.tau = *tau_in;
    t.mode = isfinite(t.pmin) ? MODE_FIRST : MODE_NONE;
    t.x = 1.0 - t.tau;
    while (t.mode < MODE_DONE) {
        const double* d = CACHED ? dl : phi;   // a thread's own entries of dl: no barrier
        if (t.mode == MODE_FIRST)
            t.first(block_sums<NT>(add_points<true>(d, tid, N, NT, t.pmin, t.x), red), goal);
        else
            t.step(block_sums<NT>(add_points<false>(d, tid, N, NT, t.pmin, t.x), red), goal);
    }
    const double ls1 = log(t.s1);
    for (int64_t k = tid; k < N; k += NT) W[k] = weight(CACHED ? dl[k] : phi[k], t, ls1);
    if (tid == 0) temper_scalars(t, N, h_out, tau_out, log_z, flags);
}

// Many workgroups: the chain min, first pass, Newton passes (those after the end of the search
// return at once), a finish by one workgroup in case the search is still open, the weights.  State
// and partial sums live in the first SCRATCH entries of W, in two copies that alternate between
// launches; a last one-workgroup launch writes the weights of those entries.  A single workgroup
// takes 1M particles through a pass in 0.7 ms, one compute unit's rate of FP64 exponentials; the whole
// chain takes 122 us there (8.6 ms with one workgroup), of which 85, its time at 8065 particles, are launches and
// the latency of the sums.
constexpr int TEMPER_BLOCKS = 256, STATE = 16;
constexpr int SCRATCH = 2 * (STATE + 5 * TEMPER_BLOCKS);
// Newton passes launched: 8 to 15 are taken for chi^2 potentials, up to 19 for spreads of ten decades.  One more costs
// an idle launch, 2.4 us; one too few a pass by one workgroup, 40 us at 65536 particles and 0.7 ms at 2^20.
static int temper_passes(int64_t N) { return N <= 65536 ? 16 : 20; }
static_assert(SCRATCH <= TEMPER_ONE && sizeof(Temper) <= STATE * sizeof(double), "the scratch fits W");

namespace {

__device__ __forceinline__ Temper* state_of(double* W, int par) {
    return reinterpret_cast<Temper*>(W + par * STATE);
}
__device__ __forceinline__ double* part_of(double* W, int par) {
    return W + 2 * STATE + par * 5 * TEMPER_BLOCKS;
}
template <int NT>
__device__ __forceinline__ Sums fold(const double* part, int blocks, double (*red)[5]) {
    Sums e{};
    if ((int)threadIdx.x < blocks) {
#pragma unroll
        for (int i = 0; i < 5; ++i) e.v[i] = part[i * TEMPER_BLOCKS + threadIdx.x];
    }
    return block_sums<NT>(e, red);
}

}  // namespace

__global__ __launch_bounds__(256) void temper_min_kernel(int64_t N, const double* __restrict__ phi, double* W) {
    __shared__ double red[4][5];
    double m = INFINITY;
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < N; k += (int64_t)gridDim.x * 256)
        m = finite_min(m, phi[k]);
    m = block_min<256>(m, red);
    if (threadIdx.x == 0) part_of(W, 0)[blockIdx.x] = m;
}

template <bool START>
__global__ __launch_bounds__(256) void temper_pass_kernel(int64_t N, const double* __restrict__ phi,
                                                          const double* __restrict__ tau_in, double goal,
                                                          double* W, int par) {   // reads copy par, writes the other
    static_assert(TEMPER_BLOCKS <= 256, "one partial per thread");
    __shared__ double red[4][5];
    const int blocks = gridDim.x, tid = threadIdx.x;
    Temper t{};
    if constexpr (START) {
        t.pmin = block_min<256>(tid < blocks ? part_of(W, par)[tid] : INFINITY, red);
        t.tau = *tau_in;
        t.x = 1.0 - t.tau;
        t.mode = isfinite(t.pmin) ? MODE_FIRST : MODE_NONE;
    } else {
        t = *state_of(W, par);
        if (t.mode < MODE_DONE) {
            const Sums e = fold<256>(part_of(W, par), blocks, red);
            if (t.mode == MODE_FIRST) t.first(e, goal);
            else t.step(e, goal);
        }
    }
    if (blockIdx.x == 0 && tid == 0) *state_of(W, par ^ 1) = t;
    if (t.mode >= MODE_DONE) return;
    const Sums e = block_sums<256>(
        add_points<START>(phi, (int64_t)blockIdx.x * 256 + tid, N, (int64_t)blocks * 256, t.pmin, t.x), red);
    if (tid < 5) {
        double v = e.v[0];
#pragma unroll
        for (int i = 1; i < 5; ++i) v = tid == i ? e.v[i] : v;
        part_of(W, par ^ 1)[tid * TEMPER_BLOCKS + blockIdx.x] = v;
    }
}

__global__ __launch_bounds__(1024) void temper_finish_kernel(int64_t N, const double* __restrict__ phi, double goal,
                                                             double* W, int par, int blocks,
                                                             double* __restrict__ h_out,
                                                             double* __restrict__ tau_out,
                                                             double* __restrict__ log_z,
                                                             int32_t* __restrict__ flags) {
    __shared__ double red[16][5];
    Temper t = *state_of(W, par);
    bool folded = false;
    while (t.mode < MODE_DONE) {
        const Sums e = folded ? block_sums<1024>(add_points<false>(phi, threadIdx.x, N, 1024, t.pmin, t.x), red)
                              : fold<1024>(part_of(W, par), blocks, red);   // the last pass of the chain
        folded = true;
        if (t.mode == MODE_FIRST) t.first(e, goal);
        else t.step(e, goal);
    }
    if (threadIdx.x == 0) {
        *state_of(W, par ^ 1) = t;
        temper_scalars(t, N, h_out, tau_out, log_z, flags);
    }
}

// The weights of entries beg <= k < end; the state is read before an entry of the scratch is written
// (beg = 0: one workgroup).
__global__ __launch_bounds__(256) void temper_weight_kernel(int64_t beg, int64_t end,
                                                            const double* __restrict__ phi, double* W, int par) {
    const Temper t = *state_of(W, par);
    const double ls1 = log(t.s1);
    __syncthreads();
    for (int64_t k = beg + (int64_t)blockIdx.x * 256 + threadIdx.x; k < end; k += (int64_t)gridDim.x * 256)
        W[k] = weight(phi[k], t, ls1);
}

// The chain wants W apart from what it reads, as it writes its scratch there before the last reading; a
// cloud weighed in place takes the one-workgroup kernel, where each entry's last reading is its
// writer's.  The line is the LDS a launch gets without asking for more, short of where the two meet (8064
// particles: 52 us in one workgroup, 84 in the chain).  The chain's launches cost its 70 us also where the
// first pass ends the search, once in a run, which one workgroup does in 20 to 60 us up to 50000 particles; the
// other steps of the run take it 110 to 500 us there.
hipError_t launch_temper(int64_t N, const double* phi, const double* tau_in, double ess_frac, double* h,
                         double* tau_new, double* W, double* log_z, int32_t* flags, hipStream_t s) {
    const double goal = ess_frac * (double)N;
    const uintptr_t w0 = (uintptr_t)W, w1 = (uintptr_t)(W + N);
    auto apart = [&](const double* a, int64_t n) { return (uintptr_t)(a + n) <= w0 || (uintptr_t)a >= w1; };
    if (N <= TEMPER_ONE) {
        temper_kernel<256, true><<<dim3(1), dim3(256), sizeof(double) * N, s>>>(N, phi, tau_in, goal, h, tau_new, W,
                                                                               log_z, flags);
        return hipGetLastError();
    }
    if (!apart(phi, N) || !apart(tau_in, 1)) {
        temper_kernel<1024, false><<<dim3(1), dim3(1024), 0, s>>>(N, phi, tau_in, goal, h, tau_new, W, log_z, flags);
        return hipGetLastError();
    }
    const int blocks = (int)std::min<int64_t>((N + 1023) / 1024, TEMPER_BLOCKS);
    const dim3 grid(blocks), block(256);
    int par = 0;
    temper_min_kernel<<<grid, block, 0, s>>>(N, phi, W);
    temper_pass_kernel<true><<<grid, block, 0, s>>>(N, phi, tau_in, goal, W, par);
    for (int i = 0; i < temper_passes(N); ++i)
        temper_pass_kernel<false><<<grid, block, 0, s>>>(N, phi, tau_in, goal, W, par ^= 1);
    temper_finish_kernel<<<dim3(1), dim3(1024), 0, s>>>(N, phi, goal, W, par ^= 1, blocks, h, tau_new, log_z, flags);
    par ^= 1;
    temper_weight_kernel<<<dim3((unsigned)((N - SCRATCH + 1023) / 1024)), block, 0, s>>>(SCRATCH, N, phi, W, par);
    temper_weight_kernel<<<dim3(1), block, 0, s>>>(0, SCRATCH, phi, W, par);
    return hipGetLastError();
}

// ------------------------------------------------------------------ systematic resampling
// On integers: q_n = floor(W_n 2^53), inclusive scan C, Q = C_{N-1};
// idx_i = min{n : C_n > floor(T_i Q / D)} with T_i = i 2^53 + u53 and D = N 2^53.  For an
// integer C, C > floor(x) iff C > x, so output i belongs to particle n exactly when
// C_{n-1} D <= T_i Q < C_n D: every particle owns a contiguous range of outputs, starting at
//   first(C_{n-1}) = min{i : T_i Q >= C_{n-1} D} = ceil(C_{n-1} N / Q - u53 / 2^53),
// evaluated exactly on 128-bit integers.  Tiles of particles, eight in a row per thread, are scanned by the
// workgroup and each thread writes its particles' ranges.  Integer sums make the result independent
// of summation order, and no CDF is stored, so N is limited only by the 32-bit output indices.
//
// The weights must be normalised: each W_n in [0, 1] and finite, and their sum at most
// 1 + 2N 2^-53 (the rounding of a normalisation in FP64), so that every q_n <= 2^53 and
// Q <= QMAX = 2^53 + 2N.  Sums are capped at QMAX + 1 < 2^54, so that the 512 or 1024 capped sums that a scan
// adds stay below 2^64.  Any weight outside [0, 1] (NaN included) or Q > QMAX sets
// SMC_FLAG_BADWEIGHTS and gives idx = 0..N-1, as do all-zero weights.
namespace {

__device__ __forceinline__ bool weight_ok(double w) { return w >= 0.0 && w <= 1.0; }   // false for NaN

__device__ __forceinline__ uint64_t qweight53(double w) { return (uint64_t)(w * 9007199254740992.0); }

// What the outputs of a resampling are computed from.
struct Outputs {
    uint64_t N, Q, u_hi, u_lo;   // u53 Q in two words
    double scale;                // N / Q
    __device__ __forceinline__ Outputs(int64_t n, uint64_t q, uint64_t u53)
        : N((uint64_t)n), Q(q), u_hi(__umul64hi(u53, q)), u_lo(u53 * q), scale((double)n / (double)q) {}
    // min{i >= 0 : (i 2^53 + u53) Q >= C N 2^53} = q + [r 2^53 > u53 Q], where C N = q Q + r
    // (0 <= r < Q).  The double estimate of q <= N <= 2^24 is within 2^-26 of C N / Q, so its floor is
    // off by one at most, and r, below 2 Q < 2^55 in magnitude, is exact in 64 bits.
    __device__ __forceinline__ int64_t first(uint64_t C) const {
        int64_t q = (int64_t)((double)C * scale);
        int64_t r = (int64_t)(C * N - (uint64_t)q * Q);
        const bool low = r < 0, high = r >= (int64_t)Q;
        q += (high ? 1 : 0) - (low ? 1 : 0);
        r += low ? (int64_t)Q : high ? -(int64_t)Q : 0;
        const uint64_t hi = (uint64_t)r >> 11, lo = (uint64_t)r << 53;
        return q + ((hi > u_hi || (hi == u_hi && lo > u_lo)) ? 1 : 0);
    }
};

// The uniform of a resampling: given, or with ctr drawn here as smc_philox_u53(seed, *ctr + ctr_off) draws it
// on the host: the first two words of the counter block RESAMPLE_BLOCK, 27 + 26 bits.
struct Uniform53 {
    uint64_t u53, seed, ctr_off;
    const uint64_t* ctr;
    __device__ __forceinline__ uint64_t value() const {
        if (!ctr) return u53;
        const uint4 w = draw(seed, *ctr + ctr_off, RESAMPLE_BLOCK, 0u);
        return ((uint64_t)(w.x >> 5) << 26) | (uint64_t)(w.y >> 6);
    }
};

__device__ __forceinline__ uint64_t q_cap(int64_t N) { return (1ull << 53) + 2ull * (uint64_t)N + 1; }   // QMAX + 1

// Inclusive scan over a workgroup of NT threads; `total` the sum.  The barriers also order reuse of `red`.
template <int NT>
__device__ __forceinline__ uint64_t block_scan(uint64_t v, uint64_t* red, uint64_t& total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint64_t o = __shfl_up((unsigned long long)v, off, 64);
        if (lane >= off) v += o;
    }
    if (lane == 63) red[wave] = v;
    __syncthreads();
    total = 0;
    uint64_t before = 0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) {
        if (w == wave) before = total;
        total += red[w];
    }
    __syncthreads();
    return before + v;
}

// The thread's RUN particles from row `at` (clipped to `end`) as integers, and their capped sum; false if
// a weight is out of range.
template <int RUN>
__device__ __forceinline__ bool load_run(const double* __restrict__ W, int64_t at, int64_t end, uint64_t cap,
                                         uint64_t (&q)[RUN], uint64_t& sum) {
    double w[RUN];
#pragma unroll
    for (int i = 0; i < RUN; ++i) w[i] = at + i < end ? W[at + i] : 0.0;
    bool ok = true;
    sum = 0;
#pragma unroll
    for (int i = 0; i < RUN; ++i) {
        const bool good = weight_ok(w[i]);
        ok = ok && good;
        q[i] = good ? qweight53(w[i]) : 0;
        sum += q[i];
        sum = sum < cap ? sum : cap;
    }
    return ok;
}

// Writes the outputs of RUN particles from row n, C the scan before them, that fall into [out_beg, out_end).  A
// particle with many outputs has them written by its whole wave (every lane of which calls this), 16 bytes a lane and
// eight stores in flight: with all the weight on one of 2^20, one thread took 33 ms for them, the wave 0.09.
template <int RUN>
__device__ __forceinline__ void write_run(const uint64_t (&q)[RUN], uint64_t C, int64_t n, const Outputs& out,
                                          int64_t out_beg, int64_t out_end, int32_t* __restrict__ idx) {
    int64_t at[RUN + 1];
    at[0] = out.first(C);
#pragma unroll
    for (int i = 0; i < RUN; ++i) {   // apart from the writes, so that the chains of the divisions overlap
        C += q[i];
        at[i + 1] = out.first(C);
    }
#pragma unroll
    for (int i = 0; i < RUN; ++i) {   // empty without weight, as past the last particle
        const int64_t b = at[i] > out_beg ? at[i] : out_beg, e = at[i + 1] < out_end ? at[i + 1] : out_end;
        const bool many = e - b > 64;
        for (int64_t o = b; o < e && !many; ++o) idx[o] = (int32_t)(n + i);
        for (unsigned long long left = __ballot(many); left; left &= left - 1) {
            const int of = __ffsll(left) - 1, lane = threadIdx.x & 63;   // outputs, particles: below 2^24
            const int first = __shfl((int)b, of, 64), end = __shfl((int)e, of, 64), row = __shfl((int)n, of, 64) + i;
            const int head = (int)(-((uintptr_t)(idx + first) >> 2) & 3), tail = (end - first - head) & 3;
            if (lane < head) idx[first + lane] = row;   // to 16 bytes, then four outputs a lane
            if (lane < tail) idx[end - 1 - lane] = row;
            const int4 four = make_int4(row, row, row, row);
            int o = first + head + 4 * lane;
            for (; o + 7 * 256 + 3 < end; o += 8 * 256) {
#pragma unroll
                for (int k = 0; k < 8; ++k) *reinterpret_cast<int4*>(idx + o + 256 * k) = four;
            }
            for (; o + 3 < end; o += 256) *reinterpret_cast<int4*>(idx + o) = four;
        }
    }
}

}  // namespace

// One workgroup, N <= 1024 RUN.
template <int RUN>
__global__ __launch_bounds__(1024) void resample_kernel(int64_t N, const double* __restrict__ W, Uniform53 uni,
                                                        int32_t* __restrict__ idx, int32_t* __restrict__ flags) {
    __shared__ uint64_t red[16];
    const int tid = threadIdx.x;
    const uint64_t u53 = uni.value(), cap = q_cap(N);
    uint64_t q[RUN], sum, Q;
    const bool ok = load_run<RUN>(W, (int64_t)tid * RUN, N, cap, q, sum);
    const uint64_t C = block_scan<1024>(sum, red, Q) - sum;
    if (__syncthreads_or(!ok) || Q == 0 || Q >= cap) {
        for (int64_t i = tid; i < N; i += 1024) idx[i] = (int32_t)i;
        if (tid == 0 && flags) atomicOr(flags, SMC_FLAG_BADWEIGHTS);
        return;
    }
    write_run(q, C, (int64_t)tid * RUN, Outputs(N, Q, u53), 0, N, idx);
}

// Many workgroups, each owning a chunk of particles: their integer sums (kept as two words each in the
// first entries of idx), the outputs past those entries, and in a last one-workgroup launch the outputs
// that lie in them.  One workgroup takes 1M particles in 2.4 ms; the three launches 19 us,
// 15 at 8193 where one workgroup takes 10 for 8192.
constexpr int RESAMPLE_BLOCKS = 512, RUN = 8, TILE = 256 * RUN;
constexpr uint64_t BAD_CHUNK = ~0ull;
__device__ __forceinline__ int64_t chunk_of(int64_t N) {   // particles per workgroup, whole tiles
    const int64_t tiles = (N + TILE - 1) / TILE;
    return (tiles + RESAMPLE_BLOCKS - 1) / RESAMPLE_BLOCKS * TILE;
}
static int resample_blocks(int64_t N) {   // workgroups: chunks of chunk_of(N)
    const int64_t tiles = (N + TILE - 1) / TILE, per = (tiles + RESAMPLE_BLOCKS - 1) / RESAMPLE_BLOCKS;
    return (int)((tiles + per - 1) / per);
}

__global__ __launch_bounds__(256) void resample_sums_kernel(int64_t N, const double* __restrict__ W,
                                                            int32_t* __restrict__ idx) {
    __shared__ uint64_t red[4];
    const int64_t chunk = chunk_of(N), beg = blockIdx.x * chunk, end = beg + chunk < N ? beg + chunk : N;
    const uint64_t cap = q_cap(N);
    uint64_t q[RUN], sum, run = 0;
    bool ok = true;
    for (int64_t at = beg + (int64_t)threadIdx.x * RUN; at < end; at += TILE) {
        ok = load_run(W, at, end, cap, q, sum) && ok;
        run += sum;
        run = run < cap ? run : cap;
    }
    uint64_t total;
    block_scan<256>(run, red, total);
    total = total < cap ? total : cap;
    if (__syncthreads_or(!ok)) total = BAD_CHUNK;
    if (threadIdx.x == 0) {
        idx[2 * blockIdx.x] = (int32_t)(uint32_t)total;
        idx[2 * blockIdx.x + 1] = (int32_t)(uint32_t)(total >> 32);
    }
}

// The scan of the chunk sums: start[b] the sum before chunk b (start[blocks] = Q).  False for bad weights.
__device__ __forceinline__ bool chunk_starts(const int32_t* idx, int blocks, uint64_t cap, uint64_t* start,
                                             uint64_t* red) {
    static_assert(RESAMPLE_BLOCKS == 512, "two chunk sums per thread");
    const int tid = threadIdx.x;
    uint64_t v[2], Q;
    bool bad = false;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int b = 2 * tid + i;
        v[i] = b < blocks ? (uint64_t)(uint32_t)idx[2 * b] | ((uint64_t)(uint32_t)idx[2 * b + 1] << 32) : 0;
        if (v[i] == BAD_CHUNK) {
            bad = true;
            v[i] = 0;
        }
    }
    const uint64_t c = block_scan<256>(v[0] + v[1], red, Q);
    start[2 * tid] = c - v[1] - v[0];
    start[2 * tid + 1] = c - v[1];
    if (tid == 255) start[2 * 256] = Q;
    return !(__syncthreads_or(bad) || Q == 0 || Q >= cap);   // publishes start
}

__device__ __forceinline__ void write_chunk(int64_t N, const double* __restrict__ W, int64_t beg, int64_t end, uint64_t C,
                                            const Outputs& out, int64_t out_beg, int64_t out_end,
                                            int32_t* __restrict__ idx, uint64_t* red) {
    for (int64_t at = beg; at < end; at += TILE) {   // uniform
        const int64_t n = at + (int64_t)threadIdx.x * RUN;
        uint64_t q[RUN], sum, total;
        load_run(W, n, end, q_cap(N), q, sum);
        const uint64_t c = block_scan<256>(sum, red, total);
        write_run(q, C + c - sum, n, out, out_beg, out_end, idx);
        C += total;
    }
}

__global__ __launch_bounds__(256) void resample_write_kernel(int64_t N, const double* __restrict__ W, Uniform53 uni,
                                                             int32_t* idx) {
    __shared__ uint64_t red[4], start[RESAMPLE_BLOCKS + 1];
    const int blocks = gridDim.x;
    const int64_t chunk = chunk_of(N), beg = blockIdx.x * chunk, end = beg + chunk < N ? beg + chunk : N;
    const int64_t own = 2 * blocks;   // entries that hold the chunk sums
    const uint64_t cap = q_cap(N), u53 = uni.value();
    if (!chunk_starts(idx, blocks, cap, start, red)) {
        for (int64_t i = beg + threadIdx.x; i < end; i += 256)
            if (i >= own) idx[i] = (int32_t)i;
        return;
    }
    write_chunk(N, W, beg, end, start[blockIdx.x], Outputs(N, start[RESAMPLE_BLOCKS], u53), own, N, idx, red);
}

__global__ __launch_bounds__(256) void resample_head_kernel(int64_t N, int blocks, const double* __restrict__ W,
                                                            Uniform53 uni, int32_t* idx,
                                                            int32_t* __restrict__ flags) {
    __shared__ uint64_t red[4], start[RESAMPLE_BLOCKS + 1];
    const int64_t chunk = chunk_of(N), own = 2 * blocks;
    const uint64_t cap = q_cap(N), u53 = uni.value();
    if (!chunk_starts(idx, blocks, cap, start, red)) {
        for (int64_t i = threadIdx.x; i < own; i += 256) idx[i] = (int32_t)i;
        if (threadIdx.x == 0 && flags) atomicOr(flags, SMC_FLAG_BADWEIGHTS);
        return;
    }
    const Outputs out(N, start[RESAMPLE_BLOCKS], u53);
    int64_t first = 0;   // of chunk 0: the first output is i = 0
    for (int b = 0; b < blocks && first < own; ++b) {   // uniform
        if (start[b + 1] == start[b]) continue;
        const int64_t next = out.first(start[b + 1]);
        if (next > first) {
            const int64_t beg = b * chunk, end = beg + chunk < N ? beg + chunk : N;
            write_chunk(N, W, beg, end, start[b], out, 0, own, idx, red);
        }
        first = next;
    }
}

static hipError_t resample(int64_t N, const double* W, const Uniform53& uni, int32_t* idx, int32_t* flags,
                           hipStream_t s) {
    if (N <= 4096) {
        resample_kernel<4><<<dim3(1), dim3(1024), 0, s>>>(N, W, uni, idx, flags);
        return hipGetLastError();
    }
    if (N <= 1024 * RUN) {
        resample_kernel<RUN><<<dim3(1), dim3(1024), 0, s>>>(N, W, uni, idx, flags);
        return hipGetLastError();
    }
    const int blocks = resample_blocks(N);   // 2 blocks <= N: a chunk has at least a tile of particles
    resample_sums_kernel<<<dim3(blocks), dim3(256), 0, s>>>(N, W, idx);
    resample_write_kernel<<<dim3(blocks), dim3(256), 0, s>>>(N, W, uni, idx);
    resample_head_kernel<<<dim3(1), dim3(256), 0, s>>>(N, blocks, W, uni, idx, flags);
    return hipGetLastError();
}

hipError_t launch_resample(int64_t N, const double* W, uint64_t u53, int32_t* idx, int32_t* flags, hipStream_t s) {
    return resample(N, W, Uniform53{u53, 0, 0, nullptr}, idx, flags, s);
}

hipError_t launch_resample_ctr(int64_t N, const double* W, uint64_t seed, const uint64_t* ctr, uint64_t ctr_off,
                               int32_t* idx, int32_t* flags, hipStream_t s) {
    return resample(N, W, Uniform53{0, seed, ctr_off, ctr}, idx, flags, s);
}

constexpr int TB = 1024;

// End of a tempering stage for G samplers, one workgroup: for every group still running (its first
// row not parked; always, without a level map) the acceptance rate of its moves (an integer sum),
// a record of the stage (tau, h, the beta the moves used, the rate, the log-evidence increment) at
// row ctr / stride - 1, then the step-size rule (double beta above a rate of 0.3, halve it below
// 0.15, at most 1), and a group whose temperature has reached 1 parks its rows.  Last, the counter
// moves to the next stage.
__global__ __launch_bounds__(TB) void stage_rule_kernel(StageRule r) {
    __shared__ unsigned long long part[TB];
    const int tid = threadIdx.x;
    const uint64_t c = *r.ctr;
    const int64_t row = (int64_t)(c / r.stride) - 1;
    for (int g = 0; g < r.G; ++g) {
        const int64_t off = r.off[g], n = r.count[g];
        const bool running = !r.level || r.level[off] != SMC_LEVEL_PARKED;   // uniform
        if (!running) continue;
        unsigned long long a = 0;
        for (int64_t k = tid; k < n; k += TB) a += (unsigned long long)r.n_acc[off + k];
        part[tid] = a;
        __syncthreads();
        for (int w = TB / 2; w > 0; w >>= 1) {
            if (tid < w) part[tid] += part[tid + w];
            __syncthreads();
        }
        const unsigned long long acc = part[0];
        __syncthreads();
        const double beta = r.beta[g], tau = r.tau[g];
        if (tid == 0) {
            const double rate = (double)acc / ((double)n * (double)(r.n_moves > 1 ? r.n_moves : 1));
            if (row >= 0 && row < r.max_stages) {
                double* rec = r.record + ((size_t)row * r.G + g) * 5;
                rec[0] = tau;
                rec[1] = r.h[g];
                rec[2] = beta;
                rec[3] = rate;
                rec[4] = r.log_z[g];
            }
            r.beta[g] = rate > 0.3 ? fmin(1.0, 2.0 * beta) : (rate < 0.15 ? 0.5 * beta : beta);
        }
        if (r.level && tau >= 1.0)
            for (int64_t k = tid; k < n; k += TB) r.level[off + k] = SMC_LEVEL_PARKED;
        __syncthreads();
    }
    __syncthreads();   // every thread has read the counter (the loop may have had no barrier)
    if (tid == 0) *r.ctr = c + r.stride;
}

hipError_t launch_stage_rule(const StageRule& r, hipStream_t s) {
    stage_rule_kernel<<<dim3(1), dim3(TB), 0, s>>>(r);
    return hipGetLastError();
}

}  // namespace smc
