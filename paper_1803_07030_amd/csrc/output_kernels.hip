// Optional per-run outputs: the magnetisation of every site type after
// every MCS (each magnetic phase gets statistics of its own) and the spins at
// the end of every temperature/field step (the final states stored per
// step), both from the paper's feature list (section "VEGAS software
// package").
//
// Per-type sums are deterministic: a fixed chunk of sites per block, added in
// a fixed order inside the block, and the chunks in a fixed order.
#include "hsim_dev.h"

namespace hsim {

namespace {

constexpr int kOT = 256;        // threads of the per-type blocks
constexpr int kOChunk = 2048;   // sites per block (site and block layouts)

__device__ void tree3(double (&v)[3], double *lds)
{
    // sum of v over the block in a fixed tree, result in thread 0's v
#pragma unroll
    for (int c = 0; c < 3; ++c) lds[c * kOT + threadIdx.x] = v[c];
    __syncthreads();
    for (int s = kOT / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s)
#pragma unroll
            for (int c = 0; c < 3; ++c) lds[c * kOT + threadIdx.x] += lds[c * kOT + threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0)
#pragma unroll
        for (int c = 0; c < 3; ++c) v[c] = lds[c * kOT];
    __syncthreads();
}

// Site and block layouts, step 1: chunk b = blockIdx.x of replica r =
// blockIdx.y; for every type, the chunk's sum -> part[r][b][t][3].
template <typename T>
__global__ __launch_bounds__(kOT) void k_type_part_site(const RepDesc *reps, int nblk, RunArgs ra)
{
    __shared__ double lds[3 * kOT];
    const int r = blockIdx.y, b = blockIdx.x;
    const RepDesc &rd = reps[r];
    const T *S = (const T *)rd.spins;
    const int i0 = b * kOChunk, i1 = min(rd.n, i0 + kOChunk);
    for (int t = 0; t < ra.tm_types; ++t) {
        double v[3] = {0.0, 0.0, 0.0};
        for (int i = i0 + (int)threadIdx.x; i < i1; i += kOT) {
            if ((rd.type ? rd.type[i] : 0) != t) continue;
            v[0] += (double)S[i];
            v[1] += (double)S[rd.n_pad + i];
            v[2] += (double)S[2 * rd.n_pad + i];
        }
        tree3(v, lds);
        if (threadIdx.x == 0)
#pragma unroll
            for (int c = 0; c < 3; ++c) ra.tm_part[(((size_t)r * nblk + b) * ra.tm_types + t) * 3 + c] = v[c];
    }
}

// Replica layout, step 1, per MCS: the sum of one chunk of sites of one type
// (blockIdx.x) for a column of W replicas (blockIdx.y); the block's 256 / W
// slices take the chunk's sites in turn and are added in order.  Every spin
// row is read once (one pass per type over all sites, and a second launch
// that added the chunks one by one, took 31.8 us per MCS for three types on
// 4169 sites x 32 replicas; this takes 4.6 us, step 2 0.1 us).
template <int W>
__global__ __launch_bounds__(kOT) void k_type_sums_rep(RepLaneArgs a, TypeSums ts, int slot)
{
    constexpr int NS = kOT / W;
    __shared__ double lds[NS][3][W];
    const int lane = threadIdx.x % W, slice = threadIdx.x / W;
    const int r = lane + W * blockIdx.y;
    const int k1 = ts.chunk[blockIdx.x + 1];
    const float *S = a.spins + r;
    double v[3] = {0.0, 0.0, 0.0};
#pragma unroll 4
    for (int k = ts.chunk[blockIdx.x] + slice; k < k1; k += NS) {
        const size_t o = (size_t)ts.list[k] * a.ss;
        v[0] += (double)S[o];
        v[1] += (double)S[a.cs + o];
        v[2] += (double)S[2 * a.cs + o];
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) lds[slice][c][lane] = v[c];
    __syncthreads();
    for (int e = threadIdx.x; e < 3 * W; e += kOT) {
        const int c = e / W, l = e % W;
        double t = lds[0][c][l];
#pragma unroll
        for (int q = 1; q < NS; ++q) t += lds[q][c][l];
        ts.part[(((size_t)slot * ts.nchunk + blockIdx.x) * 3 + c) * a.Rp + l + W * blockIdx.y] = t;
    }
}

// Step 2, per window: MCS ctl->g + t_first + blockIdx.x, type blockIdx.y, a
// column of 64 replicas (blockIdx.z): the block's 16 waves add a fixed
// sixteenth of the type's chunks each, in order, then the sixteenths in
// order.
constexpr int kTFWaves = 16;
__global__ __launch_bounds__(kTFWaves * 64) void k_type_final_rep(RepLaneArgs a, TypeSums ts, int t_first,
                                                                  RunArgs ra)
{
    __shared__ double lds[kTFWaves][3][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, type = blockIdx.y;
    const int r = lane + 64 * blockIdx.z;
    const int t = t_first + (int)blockIdx.x;
    const uint32_t g = ra.ctl->g + (uint32_t)t;
    const int c0 = ts.first[type], nc = ts.first[type + 1] - c0;
    double v[3] = {0.0, 0.0, 0.0};
    if (r < a.R) {
        const double *p = ts.part + (((size_t)(t % ts.win) * ts.nchunk + c0) * 3) * a.Rp + r;
        const int k1 = nc * (w + 1) / kTFWaves;
#pragma unroll 4
        for (int k = nc * w / kTFWaves; k < k1; ++k)
#pragma unroll
            for (int c = 0; c < 3; ++c) v[c] += p[((size_t)k * 3 + c) * a.Rp];
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) lds[w][c][lane] = v[c];
    __syncthreads();
    if (w < 3 && r < a.R) {
        double s = lds[0][w][lane];
        for (int q = 1; q < kTFWaves; ++q) s += lds[q][w][lane];
        const uint32_t s_abs = g / (uint32_t)ra.M, m = g % (uint32_t)ra.M;
        ra.type_mag[((((size_t)r * ra.S_hist + s_abs) * ra.M + m) * ra.tm_types + type) * 3 + w] = s;
    }
}

// Step 2: per replica (blockIdx.x) and (type, component) (threads), the
// chunks in order, into type_mag[r][s][m][t][3] of MCS ctl->g + t_off.
__global__ void k_type_final(int nblk, int t_off, RunArgs ra)
{
    const int r = blockIdx.x;
    const uint32_t g = ra.ctl->g + (uint32_t)t_off;
    const uint32_t s_abs = g / (uint32_t)ra.M, m = g % (uint32_t)ra.M;
    for (int q = threadIdx.x; q < ra.tm_types * 3; q += blockDim.x) {
        double v = 0.0;
        for (int b = 0; b < nblk; ++b) v += ra.tm_part[((size_t)r * nblk + b) * ra.tm_types * 3 + q];
        ra.type_mag[(((size_t)r * ra.S_hist + s_abs) * ra.M + m) * ra.tm_types * 3 + q] = v;
    }
}

// Spins of every replica at the end of step g / M, user order, double, into
// snapshots[r][s][n_max][3].  check: copy only if MCS ctl->g + t_off ends a step.
template <typename T>
__global__ void k_snapshot_site(const RepDesc *reps, int t_off, int check, RunArgs ra)
{
    const uint32_t g = ra.ctl->g + (uint32_t)t_off;
    if (check && (g + 1) % (uint32_t)ra.M != 0) return;
    const RepDesc &rd = reps[blockIdx.y];
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= rd.n) return;
    const T *S = (const T *)rd.spins;
    double *o = ra.snapshots + (((size_t)blockIdx.y * ra.S_hist + g / (uint32_t)ra.M) * ra.snap_n +
                                rd.orig[i]) * 3;
    o[0] = (double)S[i];
    o[1] = (double)S[rd.n_pad + i];
    o[2] = (double)S[2 * rd.n_pad + i];
}

__global__ void k_snapshot_rep(RepLaneArgs a, int t_off, int check, RunArgs ra)
{
    const uint32_t g = ra.ctl->g + (uint32_t)t_off;
    if (check && (g + 1) % (uint32_t)ra.M != 0) return;
    const int i = blockIdx.x;
    const size_t plane = (size_t)a.cs;
    for (int r = threadIdx.x; r < a.R; r += blockDim.x) {
        const size_t src = (size_t)i * a.ss + r;
        double *o = ra.snapshots + (((size_t)r * ra.S_hist + g / (uint32_t)ra.M) * ra.snap_n +
                                    a.orig[i]) * 3;
        o[0] = (double)a.spins[src];
        o[1] = (double)a.spins[plane + src];
        o[2] = (double)a.spins[2 * plane + src];
    }
}

}  // namespace

int type_part_blocks(int max_n) { return (max_n + kOChunk - 1) / kOChunk; }

hipError_t launch_type_mag_site(hipStream_t st, bool f64, const RepDesc *reps, int R, int max_n,
                                int t_off, const RunArgs &ra)
{
    const int nblk = type_part_blocks(max_n);
    if (f64)
        hipLaunchKernelGGL(k_type_part_site<double>, dim3((unsigned)nblk, (unsigned)R), dim3(kOT), 0,
                           st, reps, nblk, ra);
    else
        hipLaunchKernelGGL(k_type_part_site<float>, dim3((unsigned)nblk, (unsigned)R), dim3(kOT), 0,
                           st, reps, nblk, ra);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_type_final, dim3((unsigned)R), dim3(64), 0, st, nblk, t_off, ra);
    return hipGetLastError();
}

hipError_t launch_type_sums_rep(hipStream_t st, const RepLaneArgs &a, const TypeSums &ts, int t_off)
{
    if (ts.nchunk <= 0) return hipSuccess;
    if (a.Rp % 64 == 0)
        hipLaunchKernelGGL(k_type_sums_rep<64>, dim3((unsigned)ts.nchunk, (unsigned)(a.Rp / 64)), dim3(kOT), 0,
                           st, a, ts, t_off % ts.win);
    else
        hipLaunchKernelGGL(k_type_sums_rep<32>, dim3((unsigned)ts.nchunk, (unsigned)(a.Rp / 32)), dim3(kOT), 0,
                           st, a, ts, t_off % ts.win);
    return hipGetLastError();
}

hipError_t launch_type_final_rep(hipStream_t st, const RepLaneArgs &a, const TypeSums &ts, int t_first,
                                 int count, const RunArgs &ra)
{
    if (count < 1 || count > ts.win) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_type_final_rep,
                       dim3((unsigned)count, (unsigned)ra.tm_types, (unsigned)((a.R + 63) / 64)),
                       dim3(kTFWaves * 64), 0, st, a, ts, t_first, ra);
    return hipGetLastError();
}

hipError_t launch_snapshot_site(hipStream_t st, bool f64, const RepDesc *reps, int R, int max_n,
                                int t_off, bool check, const RunArgs &ra)
{
    dim3 grid((unsigned)((max_n + 255) / 256), (unsigned)R);
    if (f64)
        hipLaunchKernelGGL(k_snapshot_site<double>, grid, dim3(256), 0, st, reps, t_off, check ? 1 : 0, ra);
    else
        hipLaunchKernelGGL(k_snapshot_site<float>, grid, dim3(256), 0, st, reps, t_off, check ? 1 : 0, ra);
    return hipGetLastError();
}

hipError_t launch_snapshot_rep(hipStream_t st, const RepLaneArgs &a, int t_off, bool check,
                               const RunArgs &ra)
{
    hipLaunchKernelGGL(k_snapshot_rep, dim3((unsigned)a.n), dim3(64), 0, st, a, t_off, check ? 1 : 0, ra);
    return hipGetLastError();
}

}  // namespace hsim
