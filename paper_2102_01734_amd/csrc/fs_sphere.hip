// fs_sphere.hip -- formal solution on the spherical grid (gfx950).
//
// Characteristics of a spherical grid are not translates of one another, so
// every one is listed in the geometry cache (visits: voxel, path length,
// averaging weight), bundle-major: 64 characteristics of similar length per
// bundle, visit m of all 64 in one contiguous row.  One thread integrates one
// characteristic for one wavelength with the same per-point arithmetic as the
// box sweep (fs_point.hpp): entry half-segment with constant S, then the
// parabolic / linear recurrence.  The L lanes of a characteristic are L
// wavelengths: they share each cache entry (one broadcast load) and read the
// (chi, S) pairs of one voxel as one contiguous run (voxel-major field).  Each
// visit's w_v,d I_m (and w_v,d times the point's Lambda* term) is stored
// [entry][batch], w_v,d = w_d s_m / (sum of s over the visits of voxel v in
// direction d).  A second kernel sums these per voxel in a fixed CSR order, so
// J is bitwise reproducible and independent of how wavelengths are batched.
//
// Boundary intensities (Sec. 3.2 of the paper): characteristics entering
// from outside start with I_out plus the irradiation of the point source,
// J_sub times the characteristic's precomputed factor; characteristics that
// leave the opaque core start with I_core (the diffusion-limit value, B at
// the core for constant B).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "fs_point.hpp"
#include "fs_sphere.hpp"

namespace rt3d {

namespace {

template <typename T>
struct SPair {
    T chi, S;
};

// A lane's column of a bundle's rows of 64 entries: buffer loads with the row
// as a scalar offset.
template <typename E>
struct Rows {
    __amdgpu_buffer_rsrc_t rsrc;
    uint32_t col;
    __device__ __forceinline__ Rows(const E *p, int rows, uint32_t c)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<E *>(p), 0, rows * 64 * (int)sizeof(E), 0x00020000)), col(c * (uint32_t)sizeof(E))
    {
    }
    __device__ __forceinline__ E operator[](int m) const
    {
        const int so = m * 64 * (int)sizeof(E);
        if constexpr (sizeof(E) == 4)
            return __builtin_bit_cast(E, __builtin_amdgcn_raw_buffer_load_b32(rsrc, col, so, 0));
        else
            return __builtin_bit_cast(E, __builtin_amdgcn_raw_buffer_load_b64(rsrc, col, so, 0));
    }
};

}  // namespace

// Bound by instruction issue (79 vector instructions a visit, busy 84 % of the
// time) with memory not far behind: 4 GB of contributions, geometry and field
// lines a launch.  Two of them refine the reciprocal of the weights, without which
// thick steps lose their upwind weight (point_weights_pos): 2.24 -> 2.31 ms for the
// 16 wavelengths below.  The exponential of a step is the single-precision
// polynomial's, 2e-11 of itself.  What a lane adds to the box sweep's point is the walk through
// the cache.  The wavefront's bundle is known to be uniform, so a
// visit's row of the cache and of the outputs is a scalar base that advances by
// scalar adds, each lane's place in it a constant 32-bit offset, and a field
// pair (SMALL: below 4 GiB, voxel numbers below 2^24) one 24-bit multiply-add
// away.  Rows past a characteristic's end exist up to the bundle's longest, so
// the reads ahead need no mask, only a scalar clamp; they run a group of four
// visits ahead (two or one: 4 to 9 % slower at one wavelength, the same at 16).
// Measured on 49 x 33 x 65 voxels x 128 directions (57 M visits): 16 wavelengths
// in single 3.2 -> 2.4 ms; 25 x 17 x 34 x 32 directions, one wavelength, double,
// J and Lambda*: 74 -> 35 us.  Keeping neighbouring bundles on one XCD (runs of
// 8 to 128 blocks) changed nothing.
template <typename T, typename TG, bool WJ, bool WL, bool PARA, bool SMALL>
__global__ void __launch_bounds__(256) fs_sphere_kernel(FsSphereArgs a)
{
    // wavefront -> (bundle, batch group, slice of the bundle); lane -> (characteristic, batch entry)
    const uint32_t L = (uint32_t)a.L, C = 64 / L;
    const uint32_t nb = (uint32_t)a.n_batch;
    const uint32_t n_groups = (nb + L - 1) / L;
    const uint32_t wave = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t per_bundle = n_groups * L;
    const uint32_t bundle = wave / per_bundle;
    if (bundle >= (uint64_t)a.n_bundles) return;
    const uint32_t rem = wave - bundle * per_bundle;
    const uint32_t grp = rem / L, slice = rem - grp * L;
    const uint32_t c = (slice * C + lane / L) & 63;
    const uint32_t b = grp * L + lane % L;
    if (b >= nb) return;
    const int len = a.char_len[(int64_t)bundle * 64 + c];
    if (len <= 0) return;
    const int rows = a.char_len[(int64_t)bundle * 64];  // the bundle's longest characteristic comes first
    const int lam = a.lambda_of[b];
    const int64_t eb = a.bundle_begin[bundle];
    const Rows<TG> sv(reinterpret_cast<const TG *>(a.s) + eb, rows, c), wv(reinterpret_cast<const TG *>(a.w) + eb, rows, c);
    const Rows<int32_t> vx(a.vox + eb, rows, c);
    char *oJ = WJ ? reinterpret_cast<char *>(a.outJ) + eb * nb * (int64_t)sizeof(T) : nullptr;
    char *oL = WL ? reinterpret_cast<char *>(a.outL) + eb * nb * (int64_t)sizeof(T) : nullptr;
    const uint32_t oo = (c * nb + b) * (uint32_t)sizeof(T);
    const int64_t orow = 64 * (int64_t)nb * sizeof(T);  // bytes of a visit's row of outputs
    auto put = [&](char *o, T x) { *reinterpret_cast<T *>(o + oo) = x; };
    auto at = [&](int m) { return min(m, rows - 1); };
    constexpr int U = 4;
    constexpr uint32_t ES = sizeof(SPair<T>);
    const uint32_t stride = (uint32_t)a.lam_stride * ES, lam_off = (uint32_t)lam * ES;
    auto pair = [&](int32_t v) {
        if constexpr (SMALL)
            return *reinterpret_cast<const SPair<T> *>(reinterpret_cast<const char *>(a.field) +
                                                       (__umul24((uint32_t)v, stride) + lam_off));
        else
            return reinterpret_cast<const SPair<T> *>(a.field)[(int64_t)v * a.lam_stride + lam];
    };

    T I0 = T(0);
    if (WJ && a.I_bc) {
        const T *bc = reinterpret_cast<const T *>(a.I_bc) + 3 * lam;
        const double g = a.char_g[(int64_t)bundle * 64 + c];
        I0 = g < 0.0 ? bc[1] : bc[0] + bc[2] * T(g);
    }

    // software pipeline over groups of U visits: (chi, S) pairs, path lengths
    // and weights are read one group before they are used, voxel indices two
    SPair<T> f[U];   // points m + 1 ... m + U
    TG sl[U], w[U];  // their path lengths; the weights of points m ... m + U - 1
    int32_t vq[U];   // voxels of points m + U + 1 ... m + 2 U
    const SPair<T> f0 = pair(vx[0]), f1 = pair(vx[at(1)]);
    const TG s0 = sv[0], s1 = sv[at(1)], w0 = wv[0];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        f[u] = pair(vx[at(2 + u)]);
        sl[u] = sv[at(2 + u)];
        w[u] = wv[at(1 + u)];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) vq[u] = vx[at(2 + U + u)];

    // first point: entry half-segment with constant S
    const double t0 = seg_depth((double)f0.chi, (double)s0);
    T I, Sp = f0.S, Sc = f1.S;
    {
        T ex, e0w;
        entry_weights<T>(t0, ex, e0w);
        I = I0 * ex + f0.S * e0w;
        if (WJ) put(oJ, T(w0) * I);
        if (WL) put(oL, T(w0) * e0w);
    }
    auto step = [](double ta, double tb) {  // a vacuum step is taken at kMinStep; NaN propagates
        const double d = step_of(ta, tb);
        return d < kMinStep ? kMinStep : d;
    };
    double tc = seg_depth((double)f1.chi, (double)s1);
    double D = step(t0, tc);
    T gprev = T(0);
    for (int m0 = 1; m0 < len; m0 += U) {
        SPair<T> fx[U];
        TG sx[U], wx[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            fx[u] = pair(vq[u]);
            sx[u] = sv[at(m0 + U + 1 + u)];
            wx[u] = wv[at(m0 + U + u)];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) vq[u] = vx[at(m0 + 2 * U + 1 + u)];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int m = m0 + u;
            if (m >= len) break;
            const SPair<T> fn = f[u];  // point m + 1
            const double tn = seg_depth((double)fn.chi, (double)sl[u]);
            const bool last = m + 1 == len;
            const double Dp = last ? D : step(tc, tn);  // a padding row may hold any voxel
            const PointW<T> pw = point_weights_pos<T, false, WL && !PARA, true>(D, Dp, last);
            const T wk = T(w[u]);
            if (WJ) {
                I = I * pw.ex + pw.a * Sp + pw.b * Sc + (last ? T(0) : pw.g * fn.S);
                put(oJ + orow * m, wk * I);
            }
            if (WL) {
                T dloc;
                if (PARA) {
                    dloc = pw.b + gprev * pw.ex;
                    gprev = pw.g;
                } else {
                    dloc = pw.dlin;
                }
                put(oL + orow * m, wk * dloc);
            }
            Sp = Sc;
            Sc = fn.S;
            tc = tn;
            D = Dp;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            f[u] = fx[u];
            sl[u] = sx[u];
            w[u] = wx[u];
        }
    }
}

template <typename T, typename TG, bool WJ, bool WL, bool PARA>
static hipError_t launch_t(const FsSphereArgs &a, hipStream_t st)
{
    if (a.n_bundles == 0 || a.n_batch == 0) return hipSuccess;
    const int64_t n_groups = (a.n_batch + a.L - 1) / a.L;
    const int64_t waves = a.n_bundles * n_groups * a.L;
    if (waves > (int64_t)UINT32_MAX - 4 || 512 * (int64_t)a.n_batch > INT32_MAX) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((waves + 3) / 4));
    const int64_t stride = (int64_t)a.lam_stride * 2 * sizeof(T);
    const bool small = a.n_vox <= (1 << 24) && stride < (1 << 24) && a.n_vox * stride <= (int64_t)UINT32_MAX;
    if (small)
        hipLaunchKernelGGL((fs_sphere_kernel<T, TG, WJ, WL, PARA, true>), grid, dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL((fs_sphere_kernel<T, TG, WJ, WL, PARA, false>), grid, dim3(256), 0, st, a);
    return hipGetLastError();
}

template <typename T, typename TG>
static hipError_t launch_flags(const FsSphereArgs &a, bool wj, bool wl, bool para, hipStream_t st)
{
    if (wj && wl && para) return launch_t<T, TG, true, true, true>(a, st);
    if (wj && wl) return launch_t<T, TG, true, true, false>(a, st);
    if (wj) return launch_t<T, TG, true, false, false>(a, st);
    if (wl && para) return launch_t<T, TG, false, true, true>(a, st);
    if (wl) return launch_t<T, TG, false, true, false>(a, st);
    return hipErrorInvalidValue;
}

hipError_t fs_sphere_launch(const FsSphereArgs &a, bool is_double, bool gdouble, bool want_j, bool want_l,
                            bool parabolic_lstar, hipStream_t st)
{
    if (a.L != 1 && a.L != 2 && a.L != 4 && a.L != 8 && a.L != 16) return hipErrorInvalidValue;
    if (is_double && gdouble) return launch_flags<double, double>(a, want_j, want_l, parabolic_lstar, st);
    if (is_double) return launch_flags<double, float>(a, want_j, want_l, parabolic_lstar, st);
    if (!gdouble) return launch_flags<float, float>(a, want_j, want_l, parabolic_lstar, st);
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// fixed-order gather of the per-visit contributions into voxels
// ---------------------------------------------------------------------------
// A voxel's entries are cut into G runs of CSR order, each summed in order with
// sixteen loads in flight (the last ones masked: a tail one by one
// was half the time), and the G sums are added in order.  G depends on the
// number of voxels alone, so J does not depend on the batch a wavelength is in.
// Every run has a thread of its own while the batch leaves room: on 14450 voxels
// x 1 wavelength one thread had walked ~150 entries in 63 us, and 63 more for
// Lambda*; both now take 50 us in one launch.  With 16 wavelengths (64-byte rows,
// 2.1 GB in 0.69 ms) it runs at 3 TB/s of scattered reads, near memory's rate.
template <typename T>
__device__ __forceinline__ double gather_run(const T *__restrict__ src, const int32_t *__restrict__ idx, int32_t k,
                                             int32_t e, uint32_t nb, uint32_t b)
{
    double acc = 0.0;
    constexpr int U = 16;
    for (; k < e; k += U) {
        uint32_t i[U];
        T s[U];
#pragma unroll
        for (int u = 0; u < U; ++u) i[u] = (uint32_t)idx[min(k + u, e - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) s[u] = src[(uint64_t)i[u] * nb + b];
#pragma unroll
        for (int u = 0; u < U; ++u) acc += k + u < e ? (double)s[u] : 0.0;
    }
    return acc;
}

// Blocks of par runs x vpb voxels x nb batch entries, batch fastest (the entries
// of one voxel are read as contiguous rows), then voxels (whose k-th entries
// often are neighbours); a thread sums G / par runs.
template <typename T, int G>
__global__ void __launch_bounds__(256) sphere_gather_kernel(const T *__restrict__ srcJ, const T *__restrict__ srcL,
                                                            const int32_t *__restrict__ row,
                                                            const int32_t *__restrict__ idx, int64_t n_vox, uint32_t nb,
                                                            uint32_t vpb, int par, T *__restrict__ dstJ,
                                                            T *__restrict__ dstL, int accumulate)
{
    __shared__ double part[G > 1 ? 256 : 1];
    const T *__restrict__ src = blockIdx.y ? srcL : srcJ;
    T *__restrict__ dst = blockIdx.y ? dstL : dstJ;
    int64_t v;
    uint32_t b, g = 0;
    bool on;
    if (vpb > 0) {
        const uint32_t q = threadIdx.x / nb;
        g = q / vpb;
        b = threadIdx.x - q * nb;
        v = (int64_t)blockIdx.x * vpb + (q - g * vpb);
        on = g < (uint32_t)par && v < n_vox;
    } else {  // more batch entries than threads
        const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
        v = id / nb;
        b = (uint32_t)(id - v * nb);
        on = v < n_vox;
    }
    double acc = 0.0;
    if (on) {
        const int32_t k0 = row[v], n = row[v + 1] - k0;
        auto run = [&](int q) {
            const int32_t lo = k0 + (int32_t)((int64_t)n * q / G), hi = k0 + (int32_t)((int64_t)n * (q + 1) / G);
            return gather_run(src, idx, lo, hi, nb, b);
        };
        if (par == G) {
            acc = run((int)g);
        } else {
            for (int q = 0; q < G; ++q) acc += run(q);
        }
    }
    if (G > 1 && par == G) {
        part[threadIdx.x] = acc;
        __syncthreads();
        if (g != 0) return;
        for (int q = 1; q < G; ++q)
            if (on) acc += part[threadIdx.x + q * vpb * nb];
    }
    if (!on) return;
    T *d = dst + (int64_t)b * n_vox + v;
    *d = accumulate ? (T)((double)*d + acc) : (T)acc;
}

template <typename T, int G>
static hipError_t gather_t(const void *srcJ, const void *srcL, const int32_t *row, const int32_t *idx, int64_t n_vox,
                           int n_batch, void *dstJ, void *dstL, bool accumulate, hipStream_t st)
{
    const uint32_t nb = (uint32_t)n_batch;
    const int par = (int64_t)nb * G <= 256 ? G : 1;
    const uint32_t vpb = nb * (uint32_t)par <= 256 ? 256 / (nb * par) : 0;
    const int64_t blocks = vpb > 0 ? (n_vox + vpb - 1) / vpb : (n_vox * nb + 255) / 256;
    // one output: grid row 0 takes it as "J"
    const bool two = srcJ && srcL;
    hipLaunchKernelGGL((sphere_gather_kernel<T, G>), dim3((unsigned)blocks, two ? 2 : 1), dim3(256), 0, st,
                       reinterpret_cast<const T *>(srcJ ? srcJ : srcL), reinterpret_cast<const T *>(srcL), row, idx,
                       n_vox, nb, vpb, par, reinterpret_cast<T *>(srcJ ? dstJ : dstL), reinterpret_cast<T *>(dstL),
                       accumulate ? 1 : 0);
    return hipGetLastError();
}

hipError_t sphere_gather(const void *srcJ, const void *srcL, bool is_double, const int32_t *row, const int32_t *idx,
                         int64_t n_vox, int n_batch, void *dstJ, void *dstL, bool accumulate, hipStream_t st)
{
    if (n_vox == 0 || n_batch == 0 || (!srcJ && !srcL)) return hipSuccess;
    if (n_vox < 65536)
        return is_double ? gather_t<double, 8>(srcJ, srcL, row, idx, n_vox, n_batch, dstJ, dstL, accumulate, st)
                         : gather_t<float, 8>(srcJ, srcL, row, idx, n_vox, n_batch, dstJ, dstL, accumulate, st);
    if (n_vox < 524288)
        return is_double ? gather_t<double, 4>(srcJ, srcL, row, idx, n_vox, n_batch, dstJ, dstL, accumulate, st)
                         : gather_t<float, 4>(srcJ, srcL, row, idx, n_vox, n_batch, dstJ, dstL, accumulate, st);
    return is_double ? gather_t<double, 1>(srcJ, srcL, row, idx, n_vox, n_batch, dstJ, dstL, accumulate, st)
                     : gather_t<float, 1>(srcJ, srcL, row, idx, n_vox, n_batch, dstJ, dstL, accumulate, st);
}

}  // namespace rt3d
