// ali.hip -- field padding, partial-sum reduction, the operator-splitting
// update, Ng acceleration and convergence norms (gfx950).
//
// Operator splitting with a diagonal Lambda* (Sec. 2.2, eq. alo of the paper):
//   [1 - Lambda*(1-eps)] J_new = J_fs - Lambda*(1-eps) J_old
// written as the increment J_new = J_old + (J_fs - J_old) / (1 - (1-eps) Lambda*),
// then S = (1-eps) J_new + eps B.  All ALI state is double precision.
//
// Ng acceleration (Ng 1974; least-squares form of Auer 1987, not part of the
// paper): with the last four iterates x0 (newest) .. x3, d_i = x_i - x_{i+1},
// Q1 = d0 - d1, Q2 = d0 - d2 and weights 1/x0^2, (a, b) minimise
// sum w (d0 - a Q1 - b Q2)^2 and x <- (1-a-b) x0 + a x1 + b x2.
//
// Every reduction over voxels runs in a fixed order (per-block partials, then
// one block per wavelength), so results are bitwise reproducible; the only
// atomics are max-reductions of non-negative doubles, which are exact.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "ali.hpp"

namespace rt3d {

// ---------------------------------------------------------------------------
// Formal-solution input layout: for every wavelength a doubly periodic padded
// copy [k][y2][x2] (y2 < 2Ny, x2 < 2Nx) of the pair (chi, S), interleaved so a
// point's opacity and source are one 8- (16-) byte load:
//   dst[((l*Nz + k)*2Ny + y2)*2Nx + x2][comp] = src[l][k][y2 mod Ny][x2 mod Nx],
// comp 0 = chi, comp 1 = S (optionally minus an anchor), in the kernel type.
// Ny == 0 selects the voxel-major layout of the spherical grid, pairs
// [voxel][Nx][2] with Nx the wavelength stride (no periodic directions), so
// the wavelengths of one voxel are contiguous.
// ---------------------------------------------------------------------------
// Place of voxel v's first copy in the padded pairs of a wavelength.
__device__ __forceinline__ int64_t padded_offset(int64_t v, int64_t n_vox, int Nx, int Ny)
{
    if (n_vox <= 0xffffffffLL) {  // uniform: 32-bit divisions
        const uint32_t u = (uint32_t)v, r = u / (uint32_t)Nx, k = r / (uint32_t)Ny;
        return k * (4LL * Nx * Ny) + (int64_t)(r - k * (uint32_t)Ny) * (2 * Nx) + (u - r * (uint32_t)Nx);
    }
    const int64_t r = v / Nx, k = r / Ny;
    return k * (4LL * Nx * Ny) + (r - k * Ny) * (2 * Nx) + (v - r * Nx);
}

template <typename TD>
__device__ __forceinline__ void store_padded(TD *dst, int64_t l, int64_t n_vox, int64_t v, int Nx, int Ny, int comp,
                                             TD val)
{
    if (Ny == 0) {
        dst[2 * (v * Nx + l) + comp] = val;
        return;
    }
    TD *base = dst + 2 * (l * 4 * n_vox + padded_offset(v, n_vox, Nx, Ny)) + comp;
    const int64_t H = 2LL * Nx * Ny;
    base[0] = val;
    base[2 * Nx] = val;
    base[2 * H] = val;
    base[2 * (H + Nx)] = val;
}

template <typename TS, typename TD>
__global__ void pad_kernel(const TS *__restrict__ src, const double *__restrict__ anchor, TD *__restrict__ dst,
                           int Nx, int Ny, int64_t per_lambda, int64_t total, int comp)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    const int64_t l = i / per_lambda;
    const int64_t v = i - l * per_lambda;
    double val = (double)src[i];
    if (anchor) val -= anchor[i];
    store_padded<TD>(dst, l, per_lambda, v, Nx, Ny, comp, (TD)val);
}

template <typename TS, typename TD>
hipError_t pad_field(const TS *src, const double *anchor, TD *dst, int Nx, int Ny, int Nz, int n_lambda, int comp,
                     hipStream_t st)
{
    const int64_t per = Ny > 0 ? (int64_t)Nx * Ny * Nz : (int64_t)Nz;
    const int64_t total = per * n_lambda;
    if (total == 0) return hipSuccess;
    const int bs = 256;
    hipLaunchKernelGGL((pad_kernel<TS, TD>), dim3((unsigned)((total + bs - 1) / bs)), dim3(bs), 0, st, src, anchor,
                       dst, Nx, Ny, per, total, comp);
    return hipGetLastError();
}

// Both components of an input at once: whole pairs are written instead of
// every other word, and one launch does it (the call of a small grid is bound
// by its launches: with the joint reduction 9 x 9 x 8 x 32 directions, J and
// Lambda*, 37.6 -> 33.2 us).
template <typename T>
struct FieldPair {
    T chi, S;
};

template <typename T>
__global__ void __launch_bounds__(256) pad_pair_kernel(const T *__restrict__ chi, const T *__restrict__ S,
                                                       FieldPair<T> *__restrict__ dst, int Nx, int Ny, int64_t n_vox,
                                                       int n_lambda)
{
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v >= n_vox) return;
    const int64_t o = padded_offset(v, n_vox, Nx, Ny), H = 2LL * Nx * Ny;
    for (int l = blockIdx.y; l < n_lambda; l += gridDim.y) {
        const FieldPair<T> p{chi[l * n_vox + v], S[l * n_vox + v]};
        FieldPair<T> *d = dst + l * 4 * n_vox + o;
        d[0] = p;
        d[Nx] = p;
        d[H] = p;
        d[H + Nx] = p;
    }
}

// Voxel-major pairs [voxel][stride]: tiles of 64 voxels x 16 wavelengths are
// turned through LDS, so that both sides are read and written in runs (written
// straight from voxel-ordered threads, every word went to a line of its own:
// 2 x 29 us on 105105 voxels x 16 wavelengths, now 10 us).
template <typename T>
__global__ void __launch_bounds__(256) pad_pair_sphere_kernel(const T *__restrict__ chi, const T *__restrict__ S,
                                                              FieldPair<T> *__restrict__ dst, int stride,
                                                              int64_t n_vox, int n_lambda)
{
    constexpr int TV = 64, TL = 16;
    __shared__ FieldPair<T> tile[TL][TV + 1];
    const int64_t v0 = (int64_t)blockIdx.x * TV;
    for (int l0 = blockIdx.y * TL; l0 < n_lambda; l0 += gridDim.y * TL) {
        const int nl = min(TL, n_lambda - l0);
        for (int k = threadIdx.x; k < nl * TV; k += 256) {
            const int64_t v = v0 + k % TV, i = (int64_t)(l0 + k / TV) * n_vox + v;
            if (v < n_vox) tile[k / TV][k % TV] = FieldPair<T>{chi[i], S[i]};
        }
        __syncthreads();
        for (int k = threadIdx.x; k < nl * TV; k += 256) {
            const int q = k / nl, l = k - q * nl;
            if (v0 + q < n_vox) dst[(v0 + q) * stride + l0 + l] = tile[l][q];
        }
        __syncthreads();
    }
}

template <typename T>
hipError_t pad_pair(const T *chi, const T *S, T *dst, int Nx, int Ny, int Nz, int n_lambda, hipStream_t st)
{
    const int64_t per = Ny > 0 ? (int64_t)Nx * Ny * Nz : (int64_t)Nz;
    if (per == 0 || n_lambda == 0) return hipSuccess;
    FieldPair<T> *d = reinterpret_cast<FieldPair<T> *>(dst);
    if (Ny > 0)
        hipLaunchKernelGGL((pad_pair_kernel<T>), dim3((unsigned)((per + 255) / 256), (unsigned)std::min(n_lambda, 65535)),
                           dim3(256), 0, st, chi, S, d, Nx, Ny, per, n_lambda);
    else
        hipLaunchKernelGGL((pad_pair_sphere_kernel<T>),
                           dim3((unsigned)((per + 63) / 64), (unsigned)std::min((n_lambda + 15) / 16, 65535)), dim3(256), 0,
                           st, chi, S, d, Nx, per, n_lambda);
    return hipGetLastError();
}

template hipError_t pad_pair<float>(const float *, const float *, float *, int, int, int, int, hipStream_t);
template hipError_t pad_pair<double>(const double *, const double *, double *, int, int, int, int, hipStream_t);

template hipError_t pad_field<float, float>(const float *, const double *, float *, int, int, int, int, int,
                                             hipStream_t);
template hipError_t pad_field<float, double>(const float *, const double *, double *, int, int, int, int, int,
                                             hipStream_t);
template hipError_t pad_field<double, double>(const double *, const double *, double *, int, int, int, int, int,
                                             hipStream_t);
template hipError_t pad_field<double, float>(const double *, const double *, float *, int, int, int, int, int,
                                             hipStream_t);

// ---------------------------------------------------------------------------
// Sum of a voxel's partial slots (double accumulation).  The slots are cut into
// G contiguous runs, each added in order, and the G sums are added in order: a
// fixed order for a given grid, as G depends on the number of voxels alone, so
// that a wavelength's sum does not depend on the batch it is in.  The runs are
// shared by W wavefronts of a block over the same 64 voxels, with eight loads in
// flight each: a thread per voxel (W = 1) fills the chip only from about a
// quarter million voxels of the batch on; below that one wavefront walked 256
// slots on its own, which took 36-43 us on 33^3 voxels (37 MB of slots).  Beyond,
// more wavefronts only leave idle ones beside what follows the sum (an update of
// 58 x 101 x 9 voxels x 16 wavelengths of 16 slots in double: W = 16 164 us, 1
// 61).  With W > 1 the result is valid in the first wavefront (threads 0-63), one
// voxel a lane.
// ---------------------------------------------------------------------------
constexpr int slot_groups(int64_t n_vox) { return n_vox >= 262144 ? 1 : n_vox >= 65536 ? 4 : 16; }
constexpr int slot_waves(int64_t n_vox, int n_batch)
{
    const int W = slot_groups(n_vox * n_batch), G = slot_groups(n_vox);
    return W < G ? W : G;
}

template <typename TP>
__device__ __forceinline__ double slot_run(const TP *__restrict__ part, const int32_t *__restrict__ slot_ids, int s,
                                           int s1, int64_t n_vox, int64_t v)
{
    double acc = 0.0;
    constexpr int U = 8;
    for (; s + U <= s1; s += U) {
        TP x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = part[(int64_t)slot_ids[s + u] * n_vox + v];
#pragma unroll
        for (int u = 0; u < U; ++u) acc += (double)x[u];
    }
    for (; s < s1; ++s) acc += (double)part[(int64_t)slot_ids[s] * n_vox + v];
    return acc;
}

// All G runs by one thread: the loads go on over the ends of the (short) runs.
template <typename TP, int G>
__device__ __forceinline__ double slot_runs(const TP *__restrict__ part, const int32_t *__restrict__ slot_ids, int s0,
                                            int s1, int64_t n_vox, int64_t v)
{
    const int n = s1 - s0;
    double sum = 0.0, acc = 0.0;
    int g = 0, end = s0 + n / G;
    constexpr int U = 8;
    for (int s = s0; s < s1; s += U) {
        TP x[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (s + u < s1) x[u] = part[(int64_t)slot_ids[s + u] * n_vox + v];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (s + u < s1) {
                while (s + u == end) {  // run g ends here
                    sum += acc;
                    acc = 0.0;
                    ++g;
                    end = s0 + n * (g + 1) / G;
                }
                acc += (double)x[u];
            }
    }
    return sum + acc;
}

template <typename TP, int G, int W>
__device__ __forceinline__ double slot_sum(const TP *__restrict__ part, const int32_t *__restrict__ slot_begin,
                                           const int32_t *__restrict__ slot_ids, int b, int64_t n_vox, int64_t v)
{
    const int s0 = slot_begin[b], s1 = slot_begin[b + 1];
    if constexpr (G == 1) {
        return v < n_vox ? slot_run(part, slot_ids, s0, s1, n_vox, v) : 0.0;
    } else if constexpr (W == 1) {
        return v < n_vox ? slot_runs<TP, G>(part, slot_ids, s0, s1, n_vox, v) : 0.0;
    } else {
        __shared__ double sums[G][64];
        const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), n = s1 - s0;
        constexpr int R = G / W;  // runs a wavefront
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int g = w * R + r;
            sums[g][threadIdx.x % 64] =
                v < n_vox ? slot_run(part, slot_ids, s0 + n * g / G, s0 + n * (g + 1) / G, n_vox, v) : 0.0;
        }
        __syncthreads();
        double acc = 0.0;
        if (w == 0)
            for (int g = 0; g < G; ++g) acc += sums[g][threadIdx.x];
        return acc;
    }
}

// Voxel of this thread and whether it writes (blocks of 256 threads for
// W = 1, of W wavefronts over 64 voxels otherwise).
template <int W>
__device__ __forceinline__ int64_t slot_voxel()
{
    return W == 1 ? (int64_t)blockIdx.x * 256 + threadIdx.x : (int64_t)blockIdx.x * 64 + threadIdx.x % 64;
}

template <int W>
static dim3 slot_grid(int64_t n_vox, int n_batch)
{
    const int64_t per = W == 1 ? 256 : 64;
    return dim3((unsigned)((n_vox + per - 1) / per), (unsigned)n_batch);
}

// out[lambda_of[b]][v] = sum of the slots of batch entry b (grid row z: J, Lambda*)
template <typename TP, typename TO, int G, int W>
__global__ void __launch_bounds__(W == 1 ? 256 : 64 * W) reduce_kernel(const TP *__restrict__ part0,
                                                                       const TP *__restrict__ part1,
                                                                       const int32_t *__restrict__ slot_begin,
                                                                       const int32_t *__restrict__ slot_ids,
                                                                       const int32_t *__restrict__ lambda_of,
                                                                       TO *__restrict__ out0, TO *__restrict__ out1,
                                                                       int64_t n_vox)
{
    const TP *__restrict__ part = blockIdx.z ? part1 : part0;
    TO *__restrict__ out = blockIdx.z ? out1 : out0;
    const int b = blockIdx.y;
    const int64_t v = slot_voxel<W>();
    const double acc = slot_sum<TP, G, W>(part, slot_begin, slot_ids, b, n_vox, v);
    if (v < n_vox && (W == 1 || threadIdx.x < 64)) out[(int64_t)lambda_of[b] * n_vox + v] = (TO)acc;
}

template <typename TP, typename TO, int G, int W>
static hipError_t reduce_t(const TP *part, const TP *part2, const int32_t *slot_begin, const int32_t *slot_ids,
                           const int32_t *lambda_of, int n_batch, TO *out, TO *out2, int64_t n_vox, hipStream_t st)
{
    dim3 grid = slot_grid<W>(n_vox, n_batch);
    grid.z = part2 ? 2 : 1;
    hipLaunchKernelGGL((reduce_kernel<TP, TO, G, W>), grid, dim3(W == 1 ? 256 : 64 * W), 0, st, part, part2, slot_begin,
                       slot_ids, lambda_of, out, out2, n_vox);
    return hipGetLastError();
}

template <typename TP, typename TO>
hipError_t reduce_partials(const TP *part, const int32_t *slot_begin, const int32_t *slot_ids,
                           const int32_t *lambda_of, int n_batch, TO *out, int64_t n_vox, hipStream_t st,
                           bool one_slot, const TP *part2, TO *out2)
{
    if (n_batch == 0 || n_vox == 0) return hipSuccess;
    const int G = one_slot ? 1 : slot_groups(n_vox), W = slot_waves(n_vox, n_batch * (part2 ? 2 : 1));
#define RT_REDUCE(GV, WV) \
    return reduce_t<TP, TO, GV, WV>(part, part2, slot_begin, slot_ids, lambda_of, n_batch, out, out2, n_vox, st)
    if (G == 1) RT_REDUCE(1, 1);
    if (G == 4) {
        if (W == 1) RT_REDUCE(4, 1);
        RT_REDUCE(4, 4);
    }
    if (W == 1) RT_REDUCE(16, 1);
    if (W == 4) RT_REDUCE(16, 4);
    RT_REDUCE(16, 16);
#undef RT_REDUCE
}

template hipError_t reduce_partials<float, float>(const float *, const int32_t *, const int32_t *, const int32_t *, int,
                                                  float *, int64_t, hipStream_t, bool, const float *, float *);
template hipError_t reduce_partials<float, double>(const float *, const int32_t *, const int32_t *, const int32_t *, int,
                                                  double *, int64_t, hipStream_t, bool, const float *, double *);
template hipError_t reduce_partials<double, double>(const double *, const int32_t *, const int32_t *, const int32_t *, int,
                                                  double *, int64_t, hipStream_t, bool, const double *, double *);
template hipError_t reduce_partials<double, float>(const double *, const int32_t *, const int32_t *, const int32_t *, int,
                                                  float *, int64_t, hipStream_t, bool, const double *, float *);

template <typename TS, typename TD>
__global__ void cast_kernel(const TS *__restrict__ src, TD *__restrict__ dst, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = (TD)src[i];
}

template <typename TS, typename TD>
hipError_t cast_array(const TS *src, TD *dst, int64_t n, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL((cast_kernel<TS, TD>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, src, dst, n);
    return hipGetLastError();
}

template hipError_t cast_array<float, double>(const float *, double *, int64_t, hipStream_t);

// ---------------------------------------------------------------------------
// small fills (used instead of memset so the step can live in a graph)
// ---------------------------------------------------------------------------
__global__ void fill_u64_kernel(unsigned long long *p, unsigned long long v, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

hipError_t fill_u64(unsigned long long *p, unsigned long long v, int n, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_u64_kernel, dim3((n + 255) / 256), dim3(256), 0, st, p, v, n);
    return hipGetLastError();
}

// Stores the device's constant-rate wall clock: stream-ordered time stamps
// around a kernel inside a captured graph.
__global__ void wall_stamp_kernel(unsigned long long *p)
{
    if (threadIdx.x == 0) *p = (unsigned long long)wall_clock64();
}

hipError_t wall_stamp(unsigned long long *p, hipStream_t st)
{
    hipLaunchKernelGGL(wall_stamp_kernel, dim3(1), dim3(64), 0, st, p);
    return hipGetLastError();
}

__device__ __forceinline__ void atomic_max_nonneg(double *addr, double v)
{
    // non-negative doubles (and NaN, whose bits sort above +inf) order like
    // their bit patterns read as unsigned integers
    atomicMax(reinterpret_cast<unsigned long long *>(addr), (unsigned long long)__double_as_longlong(v));
}

template <int BS>
__device__ __forceinline__ double block_max(double v)
{
    __shared__ double red[BS / 64];
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    const int w = threadIdx.x / 64, ln = threadIdx.x % 64;
    if (ln == 0) red[w] = v;
    __syncthreads();
    if (threadIdx.x < 64) {
        v = threadIdx.x < BS / 64 ? red[threadIdx.x] : 0.0;
        for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    }
    return v;
}

// S = (1-eps) J + eps B, evaluated the same way (no contraction) wherever S
// is formed, so a source recomputed from a restored J is bitwise the one the
// update produced
__device__ __forceinline__ double source_value(double e, double j, double b)
{
#pragma clang fp contract(off)
    return (1.0 - e) * j + e * b;
}

// ---------------------------------------------------------------------------
// S = (1-eps) J + eps B and the padded formal-solution input (S - anchor)
// ---------------------------------------------------------------------------
template <typename G, typename TN>
__global__ void source_kernel(const double *__restrict__ J, const G *__restrict__ eps, const G *__restrict__ B,
                              double *__restrict__ S, const double *__restrict__ S_anchor, TN *__restrict__ next_pad,
                              int Nx, int Ny, int64_t n_vox, const int32_t *__restrict__ lambda_of)
{
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n_vox) return;
    const int64_t i = (int64_t)lambda_of[blockIdx.y] * n_vox + v;
    const double e = (double)eps[i];
    const double s = source_value(e, J[i], (double)B[i]);
    S[i] = s;
    const TN out = (TN)(S_anchor ? s - S_anchor[i] : s);
    store_padded<TN>(next_pad, lambda_of[blockIdx.y], n_vox, v, Nx, Ny, 1, out);
}

template <typename G, typename TN>
hipError_t source_update(const double *J, const G *eps, const G *B, double *S, const double *S_anchor, TN *next_pad,
                         int Nx, int Ny, int64_t n_vox, const int32_t *lambda_of, int n_batch, hipStream_t st)
{
    if (n_batch == 0 || n_vox == 0) return hipSuccess;
    const int bs = 256;
    dim3 grid((unsigned)((n_vox + bs - 1) / bs), (unsigned)n_batch);
    hipLaunchKernelGGL((source_kernel<G, TN>), grid, dim3(bs), 0, st, J, eps, B, S, S_anchor, next_pad, Nx, Ny, n_vox,
                       lambda_of);
    return hipGetLastError();
}

template hipError_t source_update<float, float>(const double *, const float *, const float *, double *,
                                                const double *, float *, int, int, int64_t, const int32_t *, int,
                                                hipStream_t);
template hipError_t source_update<double, double>(const double *, const double *, const double *, double *,
                                                  const double *, double *, int, int, int64_t, const int32_t *, int,
                                                  hipStream_t);
template hipError_t source_update<float, double>(const double *, const float *, const float *, double *,
                                                 const double *, double *, int, int, int64_t, const int32_t *, int,
                                                 hipStream_t);

// ---------------------------------------------------------------------------
// fused: J_fs = J_anchor + sum of partial slots; operator-splitting update;
// S; next padded input; Ng history; per-wavelength max |dJ/J|
// ---------------------------------------------------------------------------
template <typename TP, typename G, typename TN, int NG, int W>
__global__ void __launch_bounds__(W == 1 ? 256 : 64 * W) ali_update_kernel(AliUpdateArgs a)
{
    constexpr int BS = W == 1 ? 256 : 64 * W;
    const int b = blockIdx.y;
    const int lam = a.lambda_of[b];
    const int64_t v = slot_voxel<W>();
    const bool own = v < a.n_vox && (W == 1 || threadIdx.x < 64);  // this thread's voxel is written by it
    double rel = 0.0, res = 0.0, sum = 0.0;
    if (a.part && !a.rfs_in)  // uniform over the launch
        sum = slot_sum<TP, NG, W>(reinterpret_cast<const TP *>(a.part), a.slot_begin, a.slot_ids, b, a.n_vox, v);
    if (a.rfs_out) {  // uniform over the launch: no thread reaches the block reductions
        if (own) {
            const int64_t i = (int64_t)lam * a.n_vox + v;
            const double jfs = (a.J_anchor ? a.J_anchor[i] : 0.0) + sum;
            a.rfs_out[i] = jfs - a.J[i];
        }
        return;
    }
    if (own) {
        const int64_t i = (int64_t)lam * a.n_vox + v;
        const double jfs = a.rfs_in ? a.J[i] + a.rfs_in[i] : (a.J_anchor ? a.J_anchor[i] : 0.0) + sum;
        const double e = (double)reinterpret_cast<const G *>(a.eps)[i];
        const double L = (double)reinterpret_cast<const G *>(a.lstar)[i];
        const double Bv = (double)reinterpret_cast<const G *>(a.B)[i];
        const double jo = a.J[i];
        const double rr = (jfs - jo) / jo;
        res = fabs(rr);
        if (!(res <= 1.0e308)) res = __builtin_inf();
        if (a.net_r) a.net_r[i] = (float)rr;
        double den = 1.0 - (1.0 - e) * L;
        den = den < os_den_min<G>() ? os_den_min<G>() : den;
        const double jn = a.dJ ? jo + a.dJ[i] : jo + (jfs - jo) / den;
        a.J[i] = jn;
        if (a.hist) a.hist[i] = jn;
        const double dj = fabs(jn - jo);
        rel = dj == 0.0 ? 0.0 : dj / fabs(jn);
        if (!(rel <= 1.0e308)) rel = __builtin_inf();  // NaN or Inf: reported as non-finite
        const double s = source_value(e, jn, Bv);
        a.S[i] = s;
        const TN out = (TN)(a.S_anchor ? s - a.S_anchor[i] : s);
        store_padded<TN>(reinterpret_cast<TN *>(a.next_pad), lam, a.n_vox, v, a.Nx, a.Ny, 1, out);
    }
    rel = block_max<BS>(rel);
    if (threadIdx.x == 0) atomic_max_nonneg(&a.rel_change[lam], rel);
    if (a.resid) {
        __syncthreads();  // the reduction scratch of block_max is reused
        res = block_max<BS>(res);
        if (threadIdx.x == 0) atomic_max_nonneg(&a.resid[lam], res);
    }
}

template <typename TP, typename G, typename TN, int NG, int W>
static hipError_t ali_update_g(const AliUpdateArgs &a, int n_batch, hipStream_t st)
{
    hipLaunchKernelGGL((ali_update_kernel<TP, G, TN, NG, W>), slot_grid<W>(a.n_vox, n_batch),
                       dim3(W == 1 ? 256 : 64 * W), 0, st, a);
    return hipGetLastError();
}

template <typename TP, typename G, typename TN>
static hipError_t ali_update_t(const AliUpdateArgs &a, int n_batch, hipStream_t st)
{
    // launches that sum no slots, or one per voxel, need no groups
    const int NG = a.part && !a.rfs_in && !a.one_slot ? slot_groups(a.n_vox) : 1, W = slot_waves(a.n_vox, n_batch);
    if (NG == 1) return ali_update_g<TP, G, TN, 1, 1>(a, n_batch, st);
    if (NG == 4) return W == 1 ? ali_update_g<TP, G, TN, 4, 1>(a, n_batch, st) : ali_update_g<TP, G, TN, 4, 4>(a, n_batch, st);
    if (W == 1) return ali_update_g<TP, G, TN, 16, 1>(a, n_batch, st);
    return W == 4 ? ali_update_g<TP, G, TN, 16, 4>(a, n_batch, st) : ali_update_g<TP, G, TN, 16, 16>(a, n_batch, st);
}

hipError_t ali_update(const AliUpdateArgs &a, bool part_double, bool grid_double, bool next_double, int n_batch,
                      hipStream_t st)
{
    if (n_batch == 0 || a.n_vox == 0) return hipSuccess;
    if (grid_double) {
        if (part_double && next_double) return ali_update_t<double, double, double>(a, n_batch, st);
        return hipErrorInvalidValue;
    }
    if (next_double) return hipErrorInvalidValue;
    if (part_double) return ali_update_t<double, float, float>(a, n_batch, st);
    return ali_update_t<float, float, float>(a, n_batch, st);
}

// ---------------------------------------------------------------------------
// Ng: five weighted dot products per wavelength (per-block partials, then a
// fixed-order sum), the 2x2 solve, and the extrapolation
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) ng_dots_kernel(const double *__restrict__ x0, const double *__restrict__ x1,
                                                      const double *__restrict__ x2, const double *__restrict__ x3,
                                                      const int32_t *__restrict__ lambda_of, int64_t n_vox,
                                                      double *__restrict__ blk)
{
    const int b = blockIdx.y;
    const int64_t lam = lambda_of[b];
    double acc[5] = {0, 0, 0, 0, 0};
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n_vox; v += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = lam * n_vox + v;
        const double a0 = x0[i], a1 = x1[i], a2 = x2[i], a3 = x3[i];
        const double d0 = a0 - a1, d1 = a1 - a2, d2 = a2 - a3;
        const double q1 = d0 - d1, q2 = d0 - d2;
        const double w = 1.0 / (a0 * a0);
        acc[0] += w * q1 * q1;
        acc[1] += w * q1 * q2;
        acc[2] += w * q2 * q2;
        acc[3] += w * d0 * q1;
        acc[4] += w * d0 * q2;
    }
    __shared__ double red[5][4];
    const int wv = threadIdx.x / 64, ln = threadIdx.x % 64;
    for (int c = 0; c < 5; ++c) {
        double v = acc[c];
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if (ln == 0) red[c][wv] = v;
    }
    __syncthreads();
    if (threadIdx.x < 5) {
        const double s = ((red[threadIdx.x][0] + red[threadIdx.x][1]) + red[threadIdx.x][2]) + red[threadIdx.x][3];
        blk[((int64_t)b * gridDim.x + blockIdx.x) * 5 + threadIdx.x] = s;
    }
}

// The block sums of the five dot products: lane l adds the blocks l, l + 64, ...
// in order, then the lanes are added pairwise (a fixed order; one thread adding
// all blocks in turn took 45 us).
__global__ void __launch_bounds__(64) ng_solve_kernel(const double *__restrict__ blk, int nblk, double *__restrict__ coef)
{
    const int b = blockIdx.x;
    double A[5] = {0, 0, 0, 0, 0};
    for (int k = threadIdx.x; k < nblk; k += 64)
        for (int c = 0; c < 5; ++c) A[c] += blk[((int64_t)b * nblk + k) * 5 + c];
    for (int c = 0; c < 5; ++c)
        for (int o = 32; o > 0; o >>= 1) A[c] += __shfl_xor(A[c], o, 64);
    if (threadIdx.x != 0) return;
    const double det = A[0] * A[2] - A[1] * A[1];
    double ca = 0.0, cb = 0.0, ok = 0.0;
    if (det > 1e-10 * A[0] * A[2] && det == det && det < 1e300) {
        ca = (A[3] * A[2] - A[4] * A[1]) / det;
        cb = (A[4] * A[0] - A[3] * A[1]) / det;
        ok = 1.0;
    }
    coef[3 * b + 0] = ca;
    coef[3 * b + 1] = cb;
    coef[3 * b + 2] = ok;
}

template <typename G, typename TN>
__global__ void ng_apply_kernel(NgApplyArgs a)
{
    const int b = blockIdx.y;
    const int lam = a.lambda_of[b];
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= a.n_vox) return;
    if (a.coef[3 * b + 2] == 0.0) return;  // singular system: keep the plain iterate
    const double ca = a.coef[3 * b + 0], cb = a.coef[3 * b + 1];
    const int64_t i = (int64_t)lam * a.n_vox + v;
    const double jn = (1.0 - ca - cb) * a.x0[i] + ca * a.x1[i] + cb * a.x2[i];
    a.J[i] = jn;
    const double e = (double)reinterpret_cast<const G *>(a.eps)[i];
    const double s = source_value(e, jn, (double)reinterpret_cast<const G *>(a.B)[i]);
    a.S[i] = s;
    const TN out = (TN)(a.S_anchor ? s - a.S_anchor[i] : s);
    store_padded<TN>(reinterpret_cast<TN *>(a.next_pad), lam, a.n_vox, v, a.Nx, a.Ny, 1, out);
}

hipError_t ng_accelerate(const NgApplyArgs &a, double *blk, int nblk, int n_batch, bool grid_double, hipStream_t st)
{
    if (n_batch == 0 || a.n_vox == 0) return hipSuccess;
    hipLaunchKernelGGL(ng_dots_kernel, dim3(nblk, n_batch), dim3(256), 0, st, a.x0, a.x1, a.x2, a.x3, a.lambda_of,
                       a.n_vox, blk);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(ng_solve_kernel, dim3(n_batch), dim3(64), 0, st, blk, nblk, a.coef);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int bs = 256;
    dim3 grid((unsigned)((a.n_vox + bs - 1) / bs), (unsigned)n_batch);
    if (grid_double)
        hipLaunchKernelGGL((ng_apply_kernel<double, double>), grid, dim3(bs), 0, st, a);
    else
        hipLaunchKernelGGL((ng_apply_kernel<float, float>), grid, dim3(bs), 0, st, a);
    return hipGetLastError();
}

}  // namespace rt3d
