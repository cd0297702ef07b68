// Analysis of the per-MCS history on the GPU (double precision).
//
// Paper: thermal averages of M, chi and the specific heat ("Thermal
// averages"); cumulants of the magnetisation for finite-size scaling
// ("Critical exponents"); equilibrium correlation times ("Dynamic
// behavior"); single and multiple histogram reweighting ("Histogram and
// multiple histogram methods").
//
// A series is the history of one replica at one temperature/field step,
// history[r][s][m][5] = (E, Mx, My, Mz, accepted), MCS m0 .. M-1.  Every sum
// is taken in a fixed order (strided per thread, then a fixed tree), so the
// results are reproducible run to run.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "hsim_host.h"
#include "wave.h"

namespace hsim {

namespace {

constexpr int kAT = 1024;            // threads of the per-series blocks, at most
constexpr int kMT = 256;             // threads of the multiple-histogram blocks
constexpr int kMW = kMT / 64;

// Block-wide sums of NV values (fixed order: a tree over each wave, then the
// waves in order); every thread gets the results.  lds: NT / 64 * NV doubles.
template <int NV, int NT>
__device__ __forceinline__ void block_sums(double (&v)[NV], double *lds)
{
#pragma unroll
    for (int q = 0; q < NV; ++q) v[q] = wave_all(v[q], OpAdd());
    if constexpr (NT == 64) return;
    const int w = threadIdx.x >> 6;
    __syncthreads();                 // the previous use of lds is over
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int q = 0; q < NV; ++q) lds[w * NV + q] = v[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        double t = lds[q];
#pragma unroll
        for (int k = 1; k < NT / 64; ++k) t += lds[k * NV + q];
        v[q] = t;
    }
}

template <int NT>
__device__ __forceinline__ double block_max(double v, double *lds)
{
    v = wave_all(v, OpMax());
    if constexpr (NT == 64) return v;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = lds[0];
#pragma unroll
    for (int k = 1; k < NT / 64; ++k) t = fmax(t, lds[k]);
    return t;
}

// One series: its records of 5 doubles from MCS m0 on.
struct Series {
    const double *rec;
    __device__ Series(const double *hist, int64_t series, int M, int m0)
        : rec(hist + (series * M + m0) * 5) {}
    __device__ double E(int m) const { return rec[(size_t)m * 5]; }
    __device__ double A(int m) const
    {
        const double *h = rec + (size_t)m * 5;
        return sqrt((h[1] * h[1] + h[2] * h[2]) + h[3] * h[3]);
    }
};

// Thermal summary of count samples (get(i, e, a): energy and |M|) with
// log-weights logw(i, e) (weights shifted by their maximum); out[9] =
// (e, m_abs, m2, m4, cv, chi, u4, v1, v2) for N sites at beta.  K > 0: at
// most K samples per thread, held in registers between the three passes (the
// weights' maximum, the means, the central moments); K = 0: any count, read
// again by each pass.
template <int K, int NT, typename GET, typename LW>
__device__ __forceinline__ void thermal_block(int64_t count, GET get, LW logw, double N, double beta,
                                              double *lds, double *out)
{
    double e[K > 0 ? K : 1], a[K > 0 ? K : 1];
    double mx = -INFINITY;
    if constexpr (K > 0) {
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int i = (int)threadIdx.x + j * NT;
            e[j] = 0.0;
            a[j] = 0.0;
            if (i < count) get(i, e[j], a[j]);
        }
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int i = (int)threadIdx.x + j * NT;
            mx = i < count ? fmax(mx, logw(i, e[j])) : mx;
        }
    } else {
        for (int64_t i = threadIdx.x; i < count; i += NT) {
            get(i, e[0], a[0]);
            mx = fmax(mx, logw(i, e[0]));
        }
    }
    mx = block_max<NT>(mx, lds);
    double s[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    auto first = [&](double wi, double ei, double ai) {
        const double a2 = ai * ai;
        s[0] += wi;
        s[1] += wi * ei;
        s[2] += wi * ai;
        s[3] += wi * a2;
        s[4] += wi * (a2 * a2);
    };
    if constexpr (K > 0) {
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int i = (int)threadIdx.x + j * NT;
            if (i < count) first(exp(logw(i, e[j]) - mx), e[j], a[j]);
            __builtin_amdgcn_sched_barrier(0);   // one exponential's registers at a time
        }
    } else {
        for (int64_t i = threadIdx.x; i < count; i += NT) {
            get(i, e[0], a[0]);
            first(exp(logw(i, e[0]) - mx), e[0], a[0]);
        }
    }
    block_sums<5, NT>(s, lds);
    const double W = s[0], mE = s[1] / W, mA = s[2] / W, mA2 = s[3] / W, mA4 = s[4] / W;
    double c[4] = {0.0, 0.0, 0.0, 0.0};
    auto second = [&](double wi, double ei, double ai) {
        const double dE = ei - mE, dA = ai - mA, dA2 = ai * ai - mA2;
        c[0] += wi * (dE * dE);
        c[1] += wi * (dA * dA);
        c[2] += wi * (dA * dE);
        c[3] += wi * (dA2 * dE);
    };
    if constexpr (K > 0) {
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int i = (int)threadIdx.x + j * NT;
            if (i < count) second(exp(logw(i, e[j]) - mx), e[j], a[j]);
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
        for (int64_t i = threadIdx.x; i < count; i += NT) {
            get(i, e[0], a[0]);
            second(exp(logw(i, e[0]) - mx), e[0], a[0]);
        }
    }
    block_sums<4, NT>(c, lds);
    if (threadIdx.x == 0) {
        const double vE = c[0] / W, vA = c[1] / W, c1 = c[2] / W, c2 = c[3] / W;
        const double m2 = mA2 / (N * N), m4 = mA4 / (N * N * N * N);
        out[0] = mE / N;
        out[1] = mA / N;
        out[2] = m2;
        out[3] = m4;
        out[4] = beta * beta * vE / N;
        out[5] = beta * vA / N;
        out[6] = m2 > 0 ? 1.0 - m4 / (3.0 * m2 * m2) : 0.0;
        out[7] = mA > 0 ? -c1 / mA : 0.0;
        out[8] = mA2 > 0 ? -c2 / mA2 : 0.0;
    }
}

// The inverse temperatures of a thermal call, [series][1 + n_eval]: the
// sampling value, then the evaluation values.  Up to kArgBeta of them (3 KiB
// of the 4 KiB of arguments) travel in the kernel's arguments, and a call then
// allocates and copies nothing; more go to device memory.
constexpr int kArgBeta = 384;
struct BetaTable {
    double v[kArgBeta];
};

// grid (series, n_eval): series t at its sampling beta, evaluated with weights
// exp(-(beta - beta0) E).  One block per evaluation, bounded by latency where
// series are few: one of up to 12 * 1024 samples is read once and kept by the
// threads between the three passes (4 samples per thread in registers; of 12,
// under the 128 registers of 1024 threads, a part in scratch, 196 bytes per
// lane), a longer one is read by each pass.  64 series of 9000 samples at 3
// betas: 65.6 us with 256 threads that read it three times, 26 us now.  Where
// series are many and short, threads without a sample cost as much as others,
// so a block is no larger than 4 samples per thread ask for: 12832 series of
// 50 samples at 3 betas: 939 us in blocks of 1024 threads, 150 in blocks of 64
// (370 in blocks of 256 that read three times).
template <int K, int NT, bool ARG>
__global__ __launch_bounds__(NT) void k_thermal(const double *hist, int M, int m0, int n, double N,
                                                 const double *tab, BetaTable bt, int n_eval, double *out)
{
    __shared__ double lds[NT / 64 * 5];
    const int t = blockIdx.x, j = blockIdx.y;
    const size_t row = (size_t)t * (1 + n_eval);
    const double b0 = ARG ? bt.v[row] : tab[row], b = ARG ? bt.v[row + 1 + j] : tab[row + 1 + j];
    const double db = b - b0;
    const Series sr(hist, t, M, m0);
    auto get = [&](int64_t i, double &e, double &a) {
        e = sr.E((int)i);
        a = sr.A((int)i);
    };
    auto logw = [&](int64_t, double e) { return db == 0.0 ? 0.0 : -db * e; };
    thermal_block<K, NT>(n, get, logw, N, b, lds, out + ((size_t)t * n_eval + j) * 9);
}

// Integrated autocorrelation time of series t (observable 0: E, 1: |M|) with
// the automatic window of Sokal: lags are evaluated kLags at a time, each as
// one ordered sum, and thread 0 walks them until lag >= c tau.
//
// The sums sum_m d[m] d[m + lag] are a sliding correlation: wave w of the
// block takes kLagW consecutive lags, lane l a contiguous run of m of odd
// length, and slides a window of kLagW values along it, so a step reads two
// LDS words and does kLagW multiply-adds (the odd run length spreads the
// lanes over the banks).  Series of up to kTauRes samples stay in LDS;
// longer ones pass through it in segments.  64 series of 9000 samples with
// windows of up to 240 lags: 9.4 ms with one thread per lag walking the whole
// series in global memory, 60 us now.
constexpr int kLagW = 8;             // lags per wave
constexpr int kTauRes = 18432;       // samples of a resident series (144 KiB of LDS)
constexpr int kTauSeg = 8192;        // samples of a segment otherwise

// pad: zeros held behind a resident series.
template <int NT>
__global__ __launch_bounds__(NT) void k_tau(const double *hist, int M, int m0, int n, int pad, int obs, double c,
                                             double *tau_out, int32_t *win_out)
{
    extern __shared__ double dyn[];
    constexpr int kLags = NT / 64 * kLagW;   // lags at a time
    __shared__ double lds[NT / 64];
    __shared__ double rho[kLags];
    __shared__ int done;
    const int t = blockIdx.x;
    const Series sr(hist, t, M, m0);
    auto x = [&](int m) { return obs == 0 ? sr.E(m) : sr.A(m); };
    const bool res = n <= kTauRes;
    double s[1] = {0.0};
    for (int m = threadIdx.x; m < n; m += NT) {
        const double v = x(m);
        if (res) dyn[m] = v;
        s[0] += v;
    }
    for (int m = threadIdx.x; m < pad; m += NT) dyn[n + m] = 0.0;
    block_sums<1, NT>(s, lds);
    const double mean = s[0] / n;
    double q[1] = {0.0};
    for (int m = threadIdx.x; m < n; m += NT) {
        const double d = (res ? dyn[m] : x(m)) - mean;
        if (res) dyn[m] = d;
        q[0] += d * d;
    }
    block_sums<1, NT>(q, lds);
    const double c0 = q[0] / n;
    double tau = 0.5;
    int win = n / 2;
    if (threadIdx.x == 0) done = c0 > 0.0 ? 0 : 1;
    __syncthreads();
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (int base = 1; base <= n / 2 && !done; base += kLags) {
        const int lag0 = base + wv * kLagW;
        double r[kLagW];
#pragma unroll
        for (int u = 0; u < kLagW; ++u) r[u] = 0.0;
        const int seg = res ? n : kTauSeg;
        for (int s0 = 0; s0 < n; s0 += seg) {
            // A: d[s0 ..], la values; B: d[s0 + base ..], lb values (0 past it)
            const int la = min(seg, n - s0), lb = max(0, min(seg + kLags, n - s0 - base));
            const double *A = dyn, *B = res ? dyn + base : dyn + kTauSeg;
            if (!res) {
                __syncthreads();
                for (int m = threadIdx.x; m < la; m += NT) dyn[m] = x(s0 + m) - mean;
                for (int m = threadIdx.x; m < lb; m += NT) dyn[kTauSeg + m] = x(s0 + base + m) - mean;
                __syncthreads();
            }
            const int run = ((la + 63) / 64) | 1;
            const int lo = lane * run, hi = min(lo + run, la), off = wv * kLagW;
            auto slide = [&](auto bval) {
                double wd[kLagW];
#pragma unroll
                for (int u = 0; u < kLagW - 1; ++u) wd[u] = bval(lo + off + u);
                int m = lo;
                for (; m + kLagW <= hi; m += kLagW) {
                    double a[kLagW], nx[kLagW];
#pragma unroll
                    for (int u = 0; u < kLagW; ++u) {
                        a[u] = A[m + u];
                        nx[u] = bval(m + off + kLagW - 1 + u);
                    }
#pragma unroll
                    for (int v = 0; v < kLagW; ++v) {
                        wd[kLagW - 1] = nx[v];
#pragma unroll
                        for (int u = 0; u < kLagW; ++u) r[u] = fma(a[v], wd[u], r[u]);
#pragma unroll
                        for (int u = 0; u < kLagW - 1; ++u) wd[u] = wd[u + 1];
                    }
                }
                for (; m < hi; ++m) {
                    wd[kLagW - 1] = bval(m + off + kLagW - 1);
                    const double d = A[m];
#pragma unroll
                    for (int u = 0; u < kLagW; ++u) r[u] = fma(d, wd[u], r[u]);
#pragma unroll
                    for (int u = 0; u < kLagW - 1; ++u) wd[u] = wd[u + 1];
                }
            };
            if (lag0 <= n / 2 && lo < hi) {
                // past the series' end B counts as 0: either the zeros behind
                // the resident series reach that far, or each read is checked
                if (res && base + kLags + kLagW <= pad)
                    slide([&](int k) { return B[k]; });
                else
                    slide([&](int k) {
                        const double v = B[max(min(k, lb - 1), 0)];
                        return k < lb ? v : 0.0;
                    });
            }
        }
#pragma unroll
        for (int u = 0; u < kLagW; ++u) r[u] = wave_all(r[u], OpAdd());
        if (lane == 0)
#pragma unroll
            for (int u = 0; u < kLagW; ++u) rho[wv * kLagW + u] = r[u] / (n - (lag0 + u)) / c0;
        __syncthreads();
        if (wv == 0) {
            // tau up to each lag: a scan over the lanes, 64 lags at a time
            for (int h = 0; h < kLags && base + h <= n / 2; h += 64) {
                const int lag = base + h + lane;
                const bool in = h + lane < kLags && lag <= n / 2;
                double p = in ? rho[h + lane] : 0.0;
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const double q = __shfl_up(p, o, 64);
                    p = lane >= o ? p + q : p;
                }
                const double tl = tau + p;
                const unsigned long long hit = __ballot(in && lag >= c * tl);
                const int at = hit ? __ffsll(hit) - 1 : 63;
                tau = __shfl(tl, at, 64);
                if (hit) {
                    win = base + h + at;
                    if (lane == 0) done = 1;
                    break;
                }
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        tau_out[t] = c0 > 0.0 ? tau : 0.5;
        if (win_out) win_out[t] = c0 > 0.0 ? win : 0;
    }
}

// ------------------------------------------------------- multiple histograms
// Outcome of a multiple-histogram call.
struct MhCtl {
    int32_t done, iters;
};

// The samples of the K series, series after series: energies and |M| copied
// side by side (COPY), or read in the history, where calls of many samples
// need no memory for the copies (16 bytes each, beside ln D's 8).
template <bool COPY>
struct MhSamples {
    const double *copy_E, *copy_A;
    const double *hist;
    const int32_t *rs;      // [K][2] (replica, step)
    int S, M, m0, n;
    __device__ __forceinline__ double E(int64_t i) const
    {
        if constexpr (COPY) return copy_E[i];
        const int64_t k = i / n;
        return series(k).E((int)(i - k * n));
    }
    __device__ __forceinline__ double A(int64_t i) const
    {
        if constexpr (COPY) return copy_A[i];
        const int64_t k = i / n;
        return series(k).A((int)(i - k * n));
    }
    __device__ __forceinline__ Series series(int64_t k) const
    {
        return Series(hist, (int64_t)rs[2 * k] * S + rs[2 * k + 1], M, m0);
    }
};

__global__ __launch_bounds__(kMT) void k_mh_gather(MhSamples<false> sm, int64_t tot, double *E, double *A)
{
    const int64_t i = (int64_t)blockIdx.x * kMT + threadIdx.x;
    if (i >= tot) return;
    E[i] = sm.E(i);
    A[i] = sm.A(i);
}

// Tables no thread of the launch writes, read through the constant address
// space (scalar loads).
typedef const __attribute__((address_space(4))) double *ConstD;

// ln D = ln sum_j n_j exp(f_j - beta_j E), shifted by the largest exponent.
template <typename F>
__device__ __forceinline__ double mh_logd(double e, double ln_n, int K, ConstD beta_k, F f)
{
    double mx = -INFINITY;
#pragma unroll 4
    for (int j = 0; j < K; ++j) mx = fmax(mx, ln_n + f(j) - beta_k[j] * e);
    double s = 0.0;
#pragma unroll 4
    for (int j = 0; j < K; ++j) s += exp(ln_n + f(j) - beta_k[j] * e - mx);
    return mx + log(s);
}

template <bool COPY>
__global__ __launch_bounds__(kMT) void k_mh_logd(int64_t tot, int K, MhSamples<COPY> sm, const double *beta_k,
                                                 const double *f, double *logd)
{
    const int64_t i = (int64_t)blockIdx.x * kMT + threadIdx.x;
    if (i < tot)
        logd[i] = mh_logd(sm.E(i), log((double)sm.n), K, (ConstD)beta_k, [&](int j) { return ((ConstD)f)[j]; });
}

// The self-consistent equations
//   f_k = -ln sum_i exp(-beta_k E_i - ln D_i),  f_0 = 0
// are iterated by one launch per iteration.  Launch j first completes
// iteration j: it adds the sums that the blocks of launch j - 1 left and
// tests convergence (every block by itself, in the same order, so all agree;
// block 0 keeps the result).  Then each block takes its samples (per of them,
// a multiple of kMT): ln D of each, and for every k the block's largest
// exponent m and the sum s of exponentials relative to it, for launch j + 1.
// No block waits for another and the host looks at the outcome once per
// batch of launches; once done is set, later launches return at once.  An
// iteration over 16 series of 2000 samples: 140 us with one block per k and a
// copy to the host and back each time, 14 us so (11 with four lanes per sample,
// k_mh_iter_quad; 30 us with the last block
// to finish adding the sums behind a device-wide counter).
// An exponent of -inf adds 0 (unless every one is -inf), NaN stays NaN.
constexpr int kMhG = 16;             // lanes that add the blocks' sums of one k
constexpr int kMhBlocks = 512;       // blocks at most
constexpr int kMhK = 64;             // k whose block sums are formed together
// K and K x blocks up to which every block adds the sums itself (64 KiB of
// them read per block); beyond, a launch of one block per k adds them.
constexpr int kMhFusedK = 256, kMhFusedSums = 4096;

__device__ __forceinline__ double mh_term(double v, double m)
{
    const double t = exp(v - m);         // NaN where m = v = -inf
    return m == -INFINITY ? (v == v ? 0.0 : v) : t;
}

// -ln of the sum over the nb blocks (p[b] = (m, s)), by G = 16 or 64 lanes;
// every lane gets the result.
template <int G>
__device__ __forceinline__ double mh_combine(const double2 *p, int nb, int gl)
{
    auto all = [](double v, auto op) { return G == 16 ? row_all(v, op) : wave_all(v, op); };
    double m = -INFINITY, s = 0.0;
    for (int q = gl; q < nb; q += G) m = fmax(m, p[q].x);
    m = all(m, OpMax());
    for (int q = gl; q < nb; q += G) s += p[q].x == -INFINITY ? p[q].y : p[q].y * exp(p[q].x - m);
    s = all(s, OpAdd());
    return m == -INFINITY ? NAN : -(m + log(s));
}

__global__ __launch_bounds__(64) void k_mh_combine(int nb, const double2 *part, double *raw, const MhCtl *ctl)
{
    if (ctl->done) return;
    const double r = mh_combine<kMhG>(part + (size_t)blockIdx.x * nb, nb, threadIdx.x % kMhG);
    if (threadIdx.x == 0) raw[blockIdx.x] = r;
}

// What launch j does first: completes iteration j and tests convergence; true
// when the iterations are over.  The raw values are in shf (FUSED, added here
// by G lanes per k) or raw (from k_mh_combine); f0: their shift.
template <bool FUSED, int THREADS, int G>
__device__ __forceinline__ bool mh_complete(int j, int K, int max_iter, double tol, double *fbuf,
                                            const double *raw, const double2 *part, double *shf, MhCtl *ctl,
                                            double &f0)
{
    // the outcome and f are fetched with the sums, not before them
    int over = ctl->done;
    f0 = 0.0;
    if (j == 0) return false;
    const int lane = threadIdx.x & 63, nb = gridDim.x;
    const double *prev = fbuf + (size_t)((j - 1) & 1) * K;
    const double mine = prev[min(lane, K - 1)];
    if constexpr (FUSED) {
        const double2 *p = part + (size_t)((j - 1) & 1) * K * nb;
        for (int k0 = 0; k0 < K; k0 += THREADS / G) {
            const int k = k0 + (int)threadIdx.x / G;
            const double r = mh_combine<G>(p + (size_t)min(k, K - 1) * nb, nb, threadIdx.x % G);
            if (k < K && threadIdx.x % G == 0) shf[k] = r;
        }
        __syncthreads();
    } else {
        // Thread 0, which may set the outcome below, reads it for the whole
        // block: a wave that read it by itself could find it set by a faster
        // one and leave before its share of next[] is written.  (With the
        // sums added here the barrier above comes after every wave's read.)
        __shared__ int was;
        if (threadIdx.x == 0) was = over;
        __syncthreads();
        over = was;
    }
    if (over) return true;
    const double *rw = FUSED ? shf : raw;
    double *next = fbuf + (size_t)(j & 1) * K;
    f0 = rw[0];
    double dmax = fmax(0.0, fabs(rw[min(lane, K - 1)] - f0 - mine));   // NaN counts as 0
    for (int k = lane + 64; k < K; k += 64) dmax = fmax(dmax, fabs(rw[k] - f0 - prev[k]));
    dmax = wave_all(dmax, OpMax());
    if (blockIdx.x == 0)
        for (int k = threadIdx.x; k < K; k += THREADS) next[k] = rw[k] - f0;
    if (!(dmax < tol || j == max_iter)) return false;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        ctl->iters = j;
        ctl->done = 1;
    }
    return true;
}

// fbuf [2][K]: f of iteration j in row j & 1; raw [K]: without the shift to
// f_0 = 0 (from k_mh_combine, not FUSED); part [2][K][blocks].  ONE: per ==
// kMT, one sample per thread.
template <bool FUSED, bool ONE, bool COPY>
__global__ __launch_bounds__(kMT) void k_mh_iter(int j, int64_t tot, int per, int K, int max_iter, double tol,
                                                 MhSamples<COPY> sm, const double *beta_k, double *fbuf,
                                                 const double *raw, double *logd, double2 *part, MhCtl *ctl)
{
    __shared__ double2 sh[kMhK][kMW];
    __shared__ double shf[FUSED ? kMhFusedK : 1];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nb = gridDim.x;
    double f0;
    if (mh_complete<FUSED, kMT, kMhG>(j, K, max_iter, tol, fbuf, raw, part, shf, ctl, f0)) return;
    auto f = [&](int k) { return j > 0 ? (FUSED ? shf[k] : ((ConstD)raw)[k]) - f0 : 0.0; };
    const int64_t i0 = (int64_t)blockIdx.x * per, i1 = min(tot, i0 + per);
    const double ln_n = log((double)sm.n);
    // a thread's own samples: i0 + threadIdx.x, + kMT, ...; the first stays in
    // registers
    const int64_t mine = i0 + threadIdx.x;
    double e = 0.0, ld = 0.0;
    if (mine < i1) {
        e = sm.E(mine);
        ld = mh_logd(e, ln_n, K, (ConstD)beta_k, f);
    }
    if constexpr (!ONE)
        for (int64_t i = mine + kMT; i < i1; i += kMT) logd[i] = mh_logd(sm.E(i), ln_n, K, (ConstD)beta_k, f);
    double2 *out = part + (size_t)(j & 1) * K * nb;
    for (int k0 = 0; k0 < K; k0 += kMhK) {
        const int kn = min(kMhK, K - k0);
        if constexpr (ONE) {
            // four k at a time (the last repeated), branch-free: their chains
            // of dependent steps overlap
            for (int k = 0; k < kn; k += 4) {
                double v[4], m[4], s[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    v[u] = -((ConstD)beta_k)[k0 + min(k + u, kn - 1)] * e - ld;
                    m[u] = mine < i1 ? v[u] : -INFINITY;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) m[u] = wave_all(m[u], OpMax());
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const double t = mh_term(v[u], m[u]);
                    s[u] = mine < i1 ? t : 0.0;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) s[u] = wave_all(s[u], OpAdd());
                if (lane == 0)
#pragma unroll
                    for (int u = 0; u < 4; ++u) sh[min(k + u, kn - 1)][w] = make_double2(m[u], s[u]);
            }
        } else {
            for (int k = 0; k < kn; ++k) {
                const double b = ((ConstD)beta_k)[k0 + k], v0 = -b * e - ld;
                double m = mine < i1 ? v0 : -INFINITY;
                for (int64_t i = mine + kMT; i < i1; i += kMT) m = fmax(m, -b * sm.E(i) - logd[i]);
                m = wave_all(m, OpMax());
                double s = mine < i1 ? mh_term(v0, m) : 0.0;
                for (int64_t i = mine + kMT; i < i1; i += kMT) s += mh_term(-b * sm.E(i) - logd[i], m);
                s = wave_all(s, OpAdd());
                if (lane == 0) sh[k][w] = make_double2(m, s);
            }
        }
        __syncthreads();
        if ((int)threadIdx.x < kn) {
            const int k = threadIdx.x;
            double m = sh[k][0].x, s = 0.0;
#pragma unroll
            for (int q = 1; q < kMW; ++q) m = fmax(m, sh[k][q].x);
#pragma unroll
            for (int q = 0; q < kMW; ++q)
                s += sh[k][q].x == -INFINITY ? sh[k][q].y : sh[k][q].y * exp(sh[k][q].x - m);
            out[(size_t)(k0 + k) * nb + blockIdx.x] = make_double2(m, s);
        }
        __syncthreads();
    }
}

// The same for kMhQuadMin + 1 .. kMhQuadK series and kMT samples per block,
// all sums added by every block.  The K exponentials of a sample, twice, are a
// chain that a thread per sample leaves the chip waiting for (125 blocks of 4
// waves for 16 series of 2000 samples): here four neighbouring lanes share a
// sample, each with every fourth k in registers, in blocks of 16 waves with as
// many samples as before, so the sums to add do not get more (with four times
// the blocks they did: 22 us an iteration).  A call with 16 series of 2000
// samples: 7.43 -> 5.70 ms, 20 of 450: 11.6 -> 10.1, 9 of 1224: 1.82 -> 1.75;
// with 5 of 550 the larger blocks cost more than they give, 0.53 -> 0.58 ms.
constexpr int kMhQuadMin = 8, kMhQuadK = 32, kMhQ = 4;
constexpr int kMQT = kMT * kMhQ, kMQW = kMQT / 64;

__global__ __launch_bounds__(kMQT) void k_mh_iter_quad(int j, int64_t tot, int n, int K, int max_iter, double tol,
                                                       const double *E, const double *beta_k, double *fbuf,
                                                       double2 *part, MhCtl *ctl)
{
    constexpr int KQ = kMhQuadK / kMhQ;
    __shared__ double2 sh[kMhQuadK][kMQW];
    __shared__ double shf[kMhQuadK], shb[kMhQuadK];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nb = gridDim.x, ql = lane % kMhQ;
    const int64_t i = (int64_t)blockIdx.x * kMT + threadIdx.x / kMhQ;
    const bool mine = i < tot;
    const double e = E[mine ? i : tot - 1], ln_n = log((double)n);
    if ((int)threadIdx.x < K) shb[threadIdx.x] = beta_k[threadIdx.x];
    double f0;
    if (mh_complete<true, kMQT, 64>(j, K, max_iter, tol, fbuf, nullptr, part, shf, ctl, f0)) return;
    __syncthreads();
    // ln D; this lane's k are ql, ql + 4, ...: one past the end repeats the
    // last and adds nothing
    const int kq = (K + kMhQ - 1) / kMhQ;
    double a[KQ], mx = -INFINITY, s = 0.0;
#pragma unroll
    for (int u = 0; u < KQ; ++u)
        if (u < kq) {
            const int k = min(u * kMhQ + ql, K - 1);
            a[u] = ln_n + (j > 0 ? shf[k] - f0 : 0.0) - shb[k] * e;
            mx = fmax(mx, a[u]);
        }
    mx = fmax(mx, dpp_move<0xB1>(mx));   // quad_perm [1,0,3,2]
    mx = fmax(mx, dpp_move<0x4E>(mx));   // quad_perm [2,3,0,1]
#pragma unroll
    for (int u = 0; u < KQ; ++u)
        if (u < kq) {
            const double t = exp(a[u] - mx);
            s += u * kMhQ + ql < K ? t : 0.0;
        }
    s += dpp_move<0xB1>(s);
    s += dpp_move<0x4E>(s);
    const double ld = mx + log(s);
    double m[KQ];
#pragma unroll
    for (int u = 0; u < KQ; ++u)
        if (u < kq) {
            a[u] = -shb[min(u * kMhQ + ql, K - 1)] * e - ld;
            m[u] = quarter_all(mine ? a[u] : -INFINITY, OpMax());
        }
#pragma unroll
    for (int u = 0; u < KQ; ++u)
        if (u < kq) {
            const double t = mh_term(a[u], m[u]);
            const double r = quarter_all(mine ? t : 0.0, OpAdd());
            if (lane < kMhQ && u * kMhQ + ql < K) sh[u * kMhQ + ql][w] = make_double2(m[u], r);
        }
    __syncthreads();
    // the waves' sums of a k, by a row of 16 lanes
    const int k = (int)threadIdx.x / kMQW;
    if (k < K) {
        const double2 v = sh[k][threadIdx.x % kMQW];
        const double mb = row_all(v.x, OpMax());
        const double sb = row_all(v.x == -INFINITY ? v.y : v.y * exp(v.x - mb), OpAdd());
        if (threadIdx.x % kMQW == 0)
            part[(size_t)((j & 1) * K + k) * nb + blockIdx.x] = make_double2(mb, sb);
    }
}

// Thermal summary at beta_eval[j] from all samples of the K series with
// weights exp(-beta E - ln D).
template <bool COPY>
__global__ __launch_bounds__(kAT) void k_mh_thermal(int64_t tot, double N, MhSamples<COPY> sm, const double *logd,
                                                    const double *beta_eval, double *out)
{
    __shared__ double lds[kAT / 64 * 5];
    const int j = blockIdx.x;
    const double b = beta_eval[j];
    auto get = [&](int64_t i, double &e, double &a) {
        e = sm.E(i);
        a = sm.A(i);
    };
    auto logw = [&](int64_t i, double e) { return -b * e - logd[i]; };
    thermal_block<0, kAT>(tot, get, logw, N, b, lds, out + (size_t)j * 9);
}

void check_hist(const double *h, int32_t R, int32_t S, int32_t M, int32_t m0)
{
    if (!h || R < 1 || S < 1 || M < 1 || m0 < 0 || M - m0 < 2)
        throw Error(HSIM_E_ARG, "analysis: bad history shape or first MCS");
}

}  // namespace

void analysis_thermal_impl(const double *d_hist, int32_t R, int32_t S, int32_t M, int32_t m0,
                           int64_t n_sites, const double *beta, int32_t n_eval,
                           const double *beta_eval, double *d_out, hipStream_t st)
{
    check_hist(d_hist, R, S, M, m0);
    if (n_sites < 1 || !beta || n_eval < 1 || !d_out || (n_eval > 1 && !beta_eval))
        throw Error(HSIM_E_ARG, "analysis_thermal: bad argument");
    const int T = R * S;
    std::vector<double> tab((size_t)T * (1 + n_eval));
    for (int t = 0; t < T; ++t) {
        double *row = tab.data() + (size_t)t * (1 + n_eval);
        if (!std::isfinite(beta[t]) || beta[t] < 0) throw Error(HSIM_E_PARAM, "beta must be finite and >= 0");
        row[0] = beta[t];
        for (int j = 0; j < n_eval; ++j) {
            const double b = beta_eval ? beta_eval[(size_t)t * n_eval + j] : beta[t];
            if (!std::isfinite(b) || b < 0) throw Error(HSIM_E_PARAM, "beta must be finite and >= 0");
            row[1 + j] = b;
        }
    }
    DevBuf d_tab;
    BetaTable bt{};
    const bool arg = tab.size() <= (size_t)kArgBeta;
    if (arg) std::copy(tab.begin(), tab.end(), bt.v);
    else d_tab.upload(tab);
    const int n = M - m0;
    const dim3 grid((unsigned)T, (unsigned)n_eval);
    auto launch = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, grid, dim3((unsigned)threads), 0, st, d_hist, M, m0, n, (double)n_sites,
                           (const double *)d_tab.p, bt, n_eval, d_out);
    };
    if (n <= 4 * 64) launch(arg ? k_thermal<4, 64, true> : k_thermal<4, 64, false>, 64);
    else if (n <= 4 * 256) launch(arg ? k_thermal<4, 256, true> : k_thermal<4, 256, false>, 256);
    else if (n <= 4 * kAT) launch(arg ? k_thermal<4, kAT, true> : k_thermal<4, kAT, false>, kAT);
    else if (n <= 12 * kAT) launch(arg ? k_thermal<12, kAT, true> : k_thermal<12, kAT, false>, kAT);
    else launch(arg ? k_thermal<0, kAT, true> : k_thermal<0, kAT, false>, kAT);
    hip_check(hipGetLastError(), "thermal launch");
    hip_check(hipStreamSynchronize(st), "hipStreamSynchronize");   // before the table is freed
}

void analysis_tau_impl(const double *d_hist, int32_t R, int32_t S, int32_t M, int32_t m0,
                       int32_t obs, double c, double *d_tau, int32_t *d_win, hipStream_t st)
{
    check_hist(d_hist, R, S, M, m0);
    if ((obs != 0 && obs != 1) || !(c > 0.0) || !d_tau) throw Error(HSIM_E_ARG, "analysis_tau: bad argument");
    const int n = M - m0;
    auto launch = [&](auto kernel, int threads) {
        const int lags = threads / 64 * kLagW;
        const int pad = n <= kTauRes ? std::min(n / 2 + 2 * lags, kTauRes - n) : 0;
        const size_t dyn = (n <= kTauRes ? (size_t)(n + pad) : (size_t)(2 * kTauSeg + lags)) * sizeof(double);
        if (dyn > 65536)
            hip_check(hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn),
                      "hipFuncSetAttribute");
        hipLaunchKernelGGL(kernel, dim3((unsigned)(R * S)), dim3((unsigned)threads), dyn, st, d_hist, M, m0, n, pad,
                           obs, c, d_tau, d_win);
    };
    // Blocks of 256 threads where there are more series than CUs and a block's
    // LDS leaves room for six of them (us, 256 | 1024 threads, correlation
    // time 10 samples: 12832 series of 50: 81 | 316, of 400: 166 | 377; 1024
    // of 2000: 57 | 71), and for series too short to feed more (one of 100: 23
    // | 26); a few longer series want all lags at once (64 of 1024: 33 | 30).
    const int cus = device_cus() > 0 ? device_cus() : 256;
    if (n <= 128 || (n <= 2048 && R * S > cus)) launch(k_tau<256>, 256);
    else launch(k_tau<kAT>, kAT);
    hip_check(hipGetLastError(), "tau launch");
    hip_check(hipStreamSynchronize(st), "hipStreamSynchronize");
}

void analysis_multihist_impl(const double *d_hist, int32_t R, int32_t S, int32_t M, int32_t m0,
                             int64_t n_sites, int32_t K, const int32_t *series,
                             const double *beta_k, int32_t n_eval, const double *beta_eval,
                             int32_t max_iter, double tol, double *f_out, int32_t *iters_out,
                             double *d_out, hipStream_t st)
{
    check_hist(d_hist, R, S, M, m0);
    if (n_sites < 1 || K < 1 || !series || !beta_k || n_eval < 0 || (n_eval > 0 && (!beta_eval || !d_out)) ||
        max_iter < 1 || !(tol > 0.0) || !f_out)
        throw Error(HSIM_E_ARG, "analysis_multihist: bad argument");
    std::vector<int32_t> rs(series, series + 2 * (size_t)K);
    for (int k = 0; k < K; ++k) {
        if (rs[2 * k] < 0 || rs[2 * k] >= R || rs[2 * k + 1] < 0 || rs[2 * k + 1] >= S)
            throw Error(HSIM_E_ARG, "analysis_multihist: series outside the history");
        if (!std::isfinite(beta_k[k]) || beta_k[k] < 0) throw Error(HSIM_E_PARAM, "beta must be finite and >= 0");
    }
    for (int j = 0; j < n_eval; ++j)
        if (!std::isfinite(beta_eval[j]) || beta_eval[j] < 0) throw Error(HSIM_E_PARAM, "beta must be finite and >= 0");
    const int n = M - m0;
    const int64_t tot = (int64_t)K * n;
    const int64_t chunks = (tot + kMT - 1) / kMT;            // of kMT samples
    const int per = (int)((chunks + kMhBlocks - 1) / kMhBlocks) * kMT;
    const int nb = (int)((tot + per - 1) / per);
    const bool fused = K <= kMhFusedK && (int64_t)K * nb <= kMhFusedSums;
    const bool quad = fused && per == kMT && K > kMhQuadMin && K <= kMhQuadK;
    // Energies and |M| are copied side by side (of 900,000 samples, read by
    // every k of an iteration) as long as the copies take at most a quarter
    // of the memory that is free; at one sample per thread they are 2 MB.
    bool copy = per == kMT;
    if (!copy) {
        size_t free_bytes = 0, total_bytes = 0;
        hip_check(hipMemGetInfo(&free_bytes, &total_bytes), "hipMemGetInfo");
        copy = 16 * (size_t)tot <= free_bytes / 4;
    }
    // one allocation: the copies and ln D of every sample, the blocks' sums,
    // f, then the tables written from the host in one copy: the outcome and f
    // (zeros), the inverse temperatures, the series
    static_assert(sizeof(MhCtl) == sizeof(double), "the outcome takes one word");
    std::vector<double> tab(1 + 4 * (size_t)K + (size_t)n_eval, 0.0);
    double *h = tab.data() + 1 + 2 * (size_t)K;
    std::copy(beta_k, beta_k + K, h);
    if (n_eval > 0) std::copy(beta_eval, beta_eval + n_eval, h + K);
    std::memcpy(h + K + n_eval, rs.data(), (size_t)K * 8);
    const size_t samples = (copy ? 3 : 1) * (size_t)tot + (tot & 1);   // even: the sums are 16-byte aligned
    const size_t sums = 4 * (size_t)K * nb;
    DevBuf buf;
    auto *logd = (double *)buf.alloc((samples + sums + K + tab.size()) * 8);
    double *E = copy ? logd + tot : nullptr, *A = copy ? E + tot : nullptr;
    auto *part = (double2 *)(logd + samples);
    double *raw = logd + samples + sums, *d_tab = raw + K;
    auto *ctl = (MhCtl *)d_tab;
    double *fbuf = d_tab + 1;
    const double *bk = fbuf + 2 * (size_t)K, *be = bk + K;
    const auto *d_rs = (const int32_t *)(be + n_eval);
    hip_check(hipMemcpyAsync(d_tab, tab.data(), tab.size() * 8, hipMemcpyHostToDevice, st), "hipMemcpyAsync");
    const dim3 all((unsigned)chunks);
    const MhSamples<false> sm{nullptr, nullptr, d_hist, d_rs, S, M, m0, n};
    const MhSamples<true> smc{E, A, d_hist, d_rs, S, M, m0, n};
    if (copy) hipLaunchKernelGGL(k_mh_gather, all, dim3(kMT), 0, st, sm, tot, E, A);
    // launch j of the iterations
    auto launch = [&](auto kernel, const auto &src, int j) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)nb), dim3(kMT), 0, st, j, tot, per, K, max_iter, tol, src, bk,
                           fbuf, (const double *)raw, logd, part, ctl);
    };
    auto iterate = [&](int j) {
        if (!fused && j > 0)
            hipLaunchKernelGGL(k_mh_combine, dim3((unsigned)K), dim3(64), 0, st, nb,
                               (const double2 *)(part + (size_t)((j - 1) & 1) * K * nb), raw, (const MhCtl *)ctl);
        if (quad)
            hipLaunchKernelGGL(k_mh_iter_quad, dim3((unsigned)nb), dim3(kMQT), 0, st, j, tot, n, K, max_iter, tol,
                               (const double *)E, bk, fbuf, part, ctl);
        else if (per == kMT)
            launch(fused ? k_mh_iter<true, true, true> : k_mh_iter<false, true, true>, smc, j);
        else if (copy)
            launch(fused ? k_mh_iter<true, false, true> : k_mh_iter<false, false, true>, smc, j);
        else
            launch(fused ? k_mh_iter<true, false, false> : k_mh_iter<false, false, false>, sm, j);
    };
    // iterations are enqueued in growing batches (launch j completes
    // iteration j, so max_iter iterations take max_iter + 1 launches)
    MhCtl now{};
    int64_t sent = 0;
    for (int batch = 8; !now.done; batch = std::min(2 * batch, 64)) {
        const int64_t end = std::min<int64_t>(sent + batch, (int64_t)max_iter + 1);
        for (; sent < end; ++sent) iterate((int)sent);
        hip_check(hipGetLastError(), "multihist launch");
        hip_check(hipMemcpyAsync(&now, ctl, sizeof now, hipMemcpyDeviceToHost, st), "hipMemcpyAsync");
        hip_check(hipStreamSynchronize(st), "hipStreamSynchronize");
    }
    const double *f = fbuf + (size_t)(now.iters & 1) * K;
    auto evaluate = [&](auto logd_kernel, auto thermal_kernel, const auto &src) {
        hipLaunchKernelGGL(logd_kernel, all, dim3(kMT), 0, st, tot, K, src, bk, f, logd);
        hipLaunchKernelGGL(thermal_kernel, dim3((unsigned)n_eval), dim3(kAT), 0, st, tot, (double)n_sites, src,
                           (const double *)logd, be, d_out);
    };
    if (n_eval > 0) {
        if (copy) evaluate(k_mh_logd<true>, k_mh_thermal<true>, smc);
        else evaluate(k_mh_logd<false>, k_mh_thermal<false>, sm);
    }
    hip_check(hipGetLastError(), "multihist launch");
    hip_check(hipMemcpyAsync(f_out, f, (size_t)K * 8, hipMemcpyDeviceToHost, st), "hipMemcpyAsync");
    hip_check(hipStreamSynchronize(st), "hipStreamSynchronize");
    if (iters_out) *iters_out = now.iters;
}

}  // namespace hsim
