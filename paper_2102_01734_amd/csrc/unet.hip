// unet.hip -- inference of the learned ALI correction network (gfx950).
//
// The 3^3 convolutions between feature maps of 16, 32 or 64 channels are
// implicit GEMMs on the matrix cores (v_mfma_f32_16x16x32_bf16): the
// reduction index k runs over (tap, input channel), 27 CI values padded to a
// multiple of 32, in tiles of 16 voxels times 16 output channels.  Per 32-wide
// k chunk a lane holds 8 consecutive input channels of one tap for its voxel
// (16 bytes, channels last; zero for the padding taps and for taps beyond the
// top or bottom layer) and 8 weights of one output channel (16 bytes);
// products accumulate in fp32.  Bias, ReLU and the U-Net skip addition are
// fused into the store, and the 1-channel head into the last convolution's.
// They stage their input in LDS (conv_tile_kernel).  The input layer (3 float
// features) and the upsampling are plain VALU kernels.
// Activations never leave HBM between layers; at 129^3 with 16 channels a
// level-0 map is 68 MB.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>

#include "unet.hpp"

namespace rt3d {

typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ uint16_t f2bf(float f)
{
    // round to nearest even (finite inputs)
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// Two at a time by the conversion instruction, which rounds the same way.
__device__ __forceinline__ uint32_t f2bf2(float a, float b)
{
    typedef float v2f __attribute__((ext_vector_type(2)));
    typedef __bf16 v2b __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f{a, b}), v2b));
}

static uint16_t f2bf_host(float f)
{
    uint32_t u;
    std::memcpy(&u, &f, 4);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ int wrap(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

struct Vol {
    int nx, ny, nz;
    __host__ __device__ int64_t n() const { return (int64_t)nx * ny * nz; }
};

// ---------------------------------------------------------------------------
// 3^3 convolutions on the matrix cores
// ---------------------------------------------------------------------------
struct ConvArgs {
    const uint16_t *in;
    Vol vi, vo;
    int stride;
    const uint16_t *w;     // [27][CO][CI] bf16
    const float *bias;     // [CO]
    const uint16_t *skip;  // [vo][CO] bf16 added after the ReLU, or null
    uint16_t *out;         // [vo][CO]
};

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

__device__ __forceinline__ v8bf load8(const uint16_t *p, bool ok)
{
    v4u u = ok ? *reinterpret_cast<const v4u *>(p) : v4u{0u, 0u, 0u, 0u};
    return __builtin_bit_cast(v8bf, u);
}

// ---------------------------------------------------------------------------
// the convolutions, from LDS
// ---------------------------------------------------------------------------
// A block computes TX x TY x TZ output voxels (TX <= TXM, evened out over the
// row) for all output channels from an LDS copy of their input with its halo,
// so that a voxel's channels come from L2 once or twice instead of 27 times:
// reading them from L1 per tap bounded the plain kernel (64 bytes a cycle and
// CU, 48 cycles of loads for 8 of matrix instructions).  LDS gives 128, of which
// 16 output channels use all (one 1 KB read per matrix instruction).  The 16-voxel
// tiles run over the block's voxels in flattened order, so rows of 129 waste
// no lanes; a wavefront keeps its tiles' sums in registers and walks the k
// chunks in the plain kernel's order (the sums are the same to the bit), whose
// weights it reads once per chunk.  Weights are the first operand, so a lane ends
// up with four consecutive channels of one voxel: 8-byte stores.  Two or three
// blocks fit a CU, so latency and the instructions around the products bound it:
// the next chunk's operands and the skip map are read ahead, the LDS copy is made
// by rows whose addresses are scalar, tiles are found by a multiplication (before
// that 2400 vector instructions a wavefront for 243 matrix ones: 97 and 190 us;
// without reading ahead 116 and 285 us).  TXM is a bound: a row is cut into as few
// pieces as it allows and evened out, so any width up to it occurs.  The bounds keep
// a block's copy at 18 to 81 KB, so that two and more fit a CU's 160 KB, and its sums
// in registers; other bounds (22 or 33, two or four layers) were 1 to 7 % slower at
// 129^3; neighbouring blocks on one XCD, and
// channels in separate planes against bank conflicts: no change.  Measured at
// 129^3: 16 -> 16 channels 170 -> 61 us, 32 -> 16 with the skip 382 -> 119 us; the
// network 1149 -> 550 us.
//
// Stride 2 (an eighth of the voxels, a halo of two and more inputs per output) and
// more output than input channels take smaller tiles, so that the copy and the
// sums fit.  Reading the inputs from L2 for every tap instead, as all of them once
// did: 16 -> 32 channels 42 us, 32 -> 32 27 us; now 34 and 14.
template <int CI, int CO, int S>
struct ConvTile {
    static constexpr bool kSmall = S == 2 || CO > CI;
    static constexpr int TXM = S == 2 && CI >= 32 ? 11 : kSmall || CI == 64 ? 22 : CI == 16 ? 44 : 33;
    static constexpr int TY = S == 2 && CI == 64 ? 2 : 4, TZ = CI == 32 && !kSmall ? 4 : 2;
    static constexpr int IX = S * (TXM - 1) + 3, IY = S * (TY - 1) + 3, IZ = S * (TZ - 1) + 3;
    static constexpr int kTiles = (TXM * TY * TZ + 15) / 16, kPerWave = (kTiles + 3) / 4;
    static constexpr size_t kBytes = (size_t)IX * IY * IZ * CI * 2;
};

// Block origin (x0, y0, z0) and width tx of the tiles of a volume.
__device__ __forceinline__ void tile_origin(Vol v, int txm, int ty, int tz, int &x0, int &y0, int &z0, int &tx)
{
    const int nbx = (v.nx + txm - 1) / txm, nby = (v.ny + ty - 1) / ty;
    tx = (v.nx + nbx - 1) / nbx;
    int b = blockIdx.x;
    const int q = b / nbx;
    x0 = (b - q * nbx) * tx;
    z0 = (q / nby) * tz;
    y0 = (q - (q / nby) * nby) * ty;
}

static unsigned tile_blocks(Vol v, int txm, int ty, int tz)
{
    const int64_t nbx = (v.nx + txm - 1) / txm, nby = (v.ny + ty - 1) / ty, nbz = (v.nz + tz - 1) / tz;
    return (unsigned)(nbx * nby * nbz);
}

struct HeadArgs {
    const float *w;     // [CO], null: no head, store the map
    const float *bias;  // [1]
    float *out;         // [vo]
};

template <int CI, int CO, int S>
__global__ void __launch_bounds__(256, 2) conv_tile_kernel(ConvArgs a, HeadArgs hd)
{
    using C = ConvTile<CI, CO, S>;
    constexpr int NB = CO / 16, NK = (27 * CI + 31) / 32, T = C::kPerWave;
    extern __shared__ __align__(16) unsigned char in[];  // [IZ][IY][IX][CI] bf16
    const Vol v = a.vo, vi = a.vi;
    int x0, y0, z0, tx;
    tile_origin(v, C::TXM, C::TY, C::TZ, x0, y0, z0, tx);
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), i = lane & 15, kq = (lane >> 4) * 8;
    // A wavefront copies whole rows: the row's address is scalar, and a lane's
    // 16-byte chunks lie at the same places in every row.  All rows' loads are in
    // flight together (one by one, their latency was most of the kernel).  Rows
    // and voxels outside the volume: neighbours across the period, zeros beyond
    // the top or bottom; what lies past the tile feeds only outputs that are not
    // stored.
    constexpr int kRow = C::IX * CI * 2, kChunks = kRow / 16, kPer = (kChunks + 63) / 64;  // bytes, chunks a row and lane
    constexpr int kRows = (C::IY * C::IZ + 3) / 4;  // rows a wavefront
    {
        uint32_t at[kPer];
#pragma unroll
        for (int n = 0; n < kPer; ++n) {
            const int k = lane + 64 * n, x = S * x0 + k / (CI / 8) - 1;
            at[n] = (uint32_t)((x > vi.nx ? 0 : wrap(x, vi.nx)) * (CI * 2) + k % (CI / 8) * 16);
        }
        v4u u[kRows][kPer];
#pragma unroll
        for (int m = 0; m < kRows; ++m) {
            const int r = wave + 4 * m, y = S * y0 + r % C::IY - 1, z = S * z0 + r / C::IY - 1;
            const bool in_vol = y <= vi.ny && z >= 0 && z < vi.nz;  // uniform
            const char *row = reinterpret_cast<const char *>(
                a.in + (in_vol ? ((int64_t)z * vi.ny + wrap(y, vi.ny)) * vi.nx * CI : 0));
#pragma unroll
            for (int n = 0; n < kPer; ++n) {
                u[m][n] = *reinterpret_cast<const v4u *>(row + at[n]);
                if (!in_vol) u[m][n] = v4u{0u, 0u, 0u, 0u};
            }
        }
#pragma unroll
        for (int m = 0; m < kRows; ++m)
#pragma unroll
            for (int n = 0; n < kPer; ++n)
                if ((C::IY * C::IZ % 4 == 0 || wave + 4 * m < C::IY * C::IZ) && lane + 64 * n < kChunks)
                    *reinterpret_cast<v4u *>(in + (wave + 4 * m) * kRow + (lane + 64 * n) * 16) = u[m][n];
    }
    const int P = tx * C::TY * C::TZ;
    // the lane's voxels (one per tile): LDS offset, place in the volume, whether it is stored
    const uint32_t inv = (65536u + (uint32_t)tx - 1) / (uint32_t)tx;  // q / tx for q < 1024, tx <= 44
    static_assert(C::kTiles * 16 < 1024 && C::TXM <= 44, "");
    int base[T];
    uint32_t place[T];
    bool store[T];
    uint2 sk[T][NB];
    v4f acc[T][NB];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int q0 = (wave + 4 * t) * 16 + i, q = min(q0, P - 1);
        const int r = (int)(((uint32_t)q * inv) >> 16), xl = q - r * tx;
        base[t] = S * (((r / C::TY) * C::IY + r % C::TY) * C::IX + xl) * (2 * CI) + 2 * (kq % CI & (CI == 16 ? 8 : 31));
        const int x = x0 + xl, y = y0 + r % C::TY, z = z0 + r / C::TY;
        store[t] = q0 < P && x < v.nx && y < v.ny && z < v.nz;
        place[t] = store[t] ? ((uint32_t)z * (uint32_t)v.ny + (uint32_t)y) * (uint32_t)v.nx + (uint32_t)x : 0u;
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) {
            acc[t][cb] = v4f{0.f, 0.f, 0.f, 0.f};
            sk[t][cb] = uint2{0u, 0u};
            if (a.skip) sk[t][cb] = *reinterpret_cast<const uint2 *>(a.skip + (int64_t)place[t] * CO + cb * 16 + kq / 2);
        }
    }
    __syncthreads();
    // k = 32 j + kq: with 16 channels a chunk spans two taps, else one
    auto weights = [&](int j, int cb) {
        const int k = j * 32 + kq;
        const int tap = k / CI, c0 = k % CI;
        const bool ok = CI != 16 || j + 1 < NK || tap < 27;
        return load8(a.w + ((int64_t)(ok ? tap : 0) * CO + cb * 16 + i) * CI + c0, ok);
    };
    auto tap_off = [](int t) { return ((t / 9 * C::IY + t / 3 % 3) * C::IX + t % 3) * (2 * CI); };
    auto voxels = [&](int j, int t) {
        // byte offset of the lane's tap from its voxel's corner (its channels are in base)
        const int off = CI == 16 ? ((kq & 16) ? tap_off(2 * j + 1 < 27 ? 2 * j + 1 : 26) : tap_off(2 * j))
                                 : tap_off(j * 32 / CI) + 2 * (j * 32 % CI);
        v4u u = *reinterpret_cast<const v4u *>(in + base[t] + off);
        if (CI == 16 && j + 1 == NK) u = (kq & 16) ? v4u{0u, 0u, 0u, 0u} : u;  // tap 27 does not exist
        return __builtin_bit_cast(v8bf, u);
    };
    // chunk j + 1's voxels and chunk j + 2's weights are read before chunk j's
    // products; the barriers keep the scheduler from moving them together again
    v8bf X[2][T], W[3][NB];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) {
        W[0][cb] = weights(0, cb);
        W[1][cb] = weights(1, cb);
    }
#pragma unroll
    for (int t = 0; t < T; ++t) X[0][t] = voxels(0, t);
#pragma unroll
    for (int j = 0; j < NK; ++j) {
        if (j + 2 < NK)
#pragma unroll
            for (int cb = 0; cb < NB; ++cb) W[(j + 2) % 3][cb] = weights(j + 2, cb);
        if (j + 1 < NK)
#pragma unroll
            for (int t = 0; t < T; ++t) X[(j + 1) % 2][t] = voxels(j + 1, t);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int cb = 0; cb < NB; ++cb)
                acc[t][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[j % 3][cb], X[j % 2][t], acc[t][cb], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    }
    // D layout: a lane holds channels 16 cb + kq/2 .. + 3 of voxel i
    v4f bias[NB], head[NB];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) {
        bias[cb] = *reinterpret_cast<const v4f *>(a.bias + cb * 16 + kq / 2);
        head[cb] = hd.w ? *reinterpret_cast<const v4f *>(hd.w + cb * 16 + kq / 2) : v4f{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int t = 0; t < T; ++t) {
        float dot = 0.f;
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) {
            float val[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                val[e] = fmaxf(acc[t][cb][e] + bias[cb][e], 0.f);
                if (a.skip) val[e] += bf2f((uint16_t)((e < 2 ? sk[t][cb].x : sk[t][cb].y) >> (16 * (e % 2))));
            }
            const uint2 h{f2bf2(val[0], val[1]), f2bf2(val[2], val[3])};
            if (hd.w) {
#pragma unroll
                for (int e = 0; e < 4; ++e) dot += head[cb][e] * bf2f((uint16_t)((e < 2 ? h.x : h.y) >> (16 * (e % 2))));
            } else if (store[t]) {
                *reinterpret_cast<uint2 *>(a.out + (int64_t)place[t] * CO + cb * 16 + kq / 2) = h;
            }
        }
        if (hd.w) {  // the four lanes of a voxel hold its channels between them
            dot += __shfl_xor(dot, 16, 64);
            dot += __shfl_xor(dot, 32, 64);
            if (store[t] && lane < 16) hd.out[place[t]] = dot + hd.bias[0];
        }
    }
}

template <int CI, int CO, int S>
static hipError_t conv_tile_t(const ConvArgs &a, const HeadArgs &hd, hipStream_t st)
{
    using C = ConvTile<CI, CO, S>;
    auto k = conv_tile_kernel<CI, CO, S>;
    hipError_t e = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::kBytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3(tile_blocks(a.vo, C::TXM, C::TY, C::TZ)), dim3(256), C::kBytes, st, a, hd);
    return hipGetLastError();
}

static hipError_t conv_tile(const ConvArgs &a, int ci, int co, const HeadArgs &hd, hipStream_t st)
{
#define RT_CONV_CASE(I, O) \
    if (ci == I && co == O) return a.stride == 1 ? conv_tile_t<I, O, 1>(a, hd, st) : conv_tile_t<I, O, 2>(a, hd, st);
    RT_CONV_CASE(16, 16) RT_CONV_CASE(16, 32) RT_CONV_CASE(16, 64)
    RT_CONV_CASE(32, 16) RT_CONV_CASE(32, 32) RT_CONV_CASE(32, 64)
    RT_CONV_CASE(64, 16) RT_CONV_CASE(64, 32) RT_CONV_CASE(64, 64)
#undef RT_CONV_CASE
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// input layer (3 features -> C channels), fp32 VALU
// ---------------------------------------------------------------------------
template <int CO>
__global__ void __launch_bounds__(256) conv_in_kernel(const float *__restrict__ f, Vol v, const float *__restrict__ w,
                                                      const float *__restrict__ bias, uint16_t *__restrict__ out)
{
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= v.n()) return;
    const int x = (int)(id % v.nx);
    const int64_t r = id / v.nx;
    const int y = (int)(r % v.ny);
    const int z = (int)(r / v.ny);
    float acc[CO];
#pragma unroll
    for (int c = 0; c < CO; ++c) acc[c] = bias[c];
    for (int dz = 0; dz < 3; ++dz) {
        const int zi = z + dz - 1;
        if (zi < 0 || zi >= v.nz) continue;
        for (int dy = 0; dy < 3; ++dy) {
            const int yi = wrap(y + dy - 1, v.ny);
            for (int dx = 0; dx < 3; ++dx) {
                const int xi = wrap(x + dx - 1, v.nx);
                const float *fp = f + (((int64_t)zi * v.ny + yi) * v.nx + xi) * 3;
                const float f0 = fp[0], f1 = fp[1], f2 = fp[2];
                const float *wt = w + ((dz * 3 + dy) * 3 + dx) * CO * 3;
#pragma unroll
                for (int c = 0; c < CO; ++c) acc[c] += wt[3 * c] * f0 + wt[3 * c + 1] * f1 + wt[3 * c + 2] * f2;
            }
        }
    }
#pragma unroll
    for (int c = 0; c < CO; ++c) out[id * CO + c] = f2bf(fmaxf(acc[c], 0.f));
}

// linear upsampling by 2 (align corners): fine index o takes the coarse
// point o/2 (o even) or the mean of (o-1)/2 and (o+1)/2 (o odd); the upper
// neighbour wraps in x, y and is clamped in z.  One thread per fine voxel
// and 8 channels (16-byte loads and stores; C is a multiple of 16), a block per
// row, so that rows are found without divisions (129^3 x 32 channels: 67 -> 51 us).
__global__ void __launch_bounds__(1024) upsample_kernel(const uint16_t *__restrict__ in, Vol vc, uint16_t *__restrict__ out,
                                                        Vol vf, int log_groups)
{
    const int groups = 1 << log_groups, C = 8 * groups;
    const int y = blockIdx.x, ys[2] = {y >> 1, (y & 1) ? wrap((y + 1) >> 1, vc.ny) : y >> 1};
    for (int z = blockIdx.y; z < vf.nz; z += gridDim.y) {
        const int zs[2] = {z >> 1, (z & 1) ? min((z + 1) >> 1, vc.nz - 1) : z >> 1};
        for (int i = threadIdx.x; i < vf.nx * groups; i += blockDim.x) {
            const int x = i >> log_groups, c0 = (i & (groups - 1)) * 8;
            const int xs[2] = {x >> 1, (x & 1) ? wrap((x + 1) >> 1, vc.nx) : x >> 1};
            float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int d = 0; d < 2; ++d) {
                        const v4u q = *reinterpret_cast<const v4u *>(
                            in + ((int64_t)zs[a] * vc.ny + ys[b]) * vc.nx * C + xs[d] * C + c0);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            acc[2 * e] += __uint_as_float(q[e] << 16);
                            acc[2 * e + 1] += __uint_as_float(q[e] & 0xffff0000u);
                        }
                    }
            v4u o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = f2bf2(0.125f * acc[2 * e], 0.125f * acc[2 * e + 1]);
            *reinterpret_cast<v4u *>(out + ((int64_t)z * vf.ny + y) * vf.nx * C + x * C + c0) = o;
        }
    }
}

// ---------------------------------------------------------------------------
// features and application of the correction
// ---------------------------------------------------------------------------
template <typename G>
__global__ void __launch_bounds__(256) features_kernel(const float *__restrict__ r, float inv_scale,
                                                       const G *__restrict__ chi, const G *__restrict__ eps, int64_t n,
                                                       float *__restrict__ f)
{
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    const float c = fmaxf((float)chi[v], 1e-30f), e = fmaxf((float)eps[v], 1e-30f);
    f[3 * v] = r[v] * inv_scale;
    f[3 * v + 1] = log10f(c) * 0.25f;
    f[3 * v + 2] = log10f(e) * (1.0f / 3.0f) + 1.0f;
}

template <typename G>
hipError_t unet_features(const float *r, double scale, const G *chi, const G *eps, int64_t n, float *features,
                         hipStream_t st)
{
    if (n == 0) return hipSuccess;
    const float inv = scale > 0.0 ? (float)(1.0 / scale) : 0.f;
    hipLaunchKernelGGL((features_kernel<G>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, r, inv, chi, eps, n,
                       features);
    return hipGetLastError();
}
template hipError_t unet_features<float>(const float *, double, const float *, const float *, int64_t, float *,
                                         hipStream_t);
template hipError_t unet_features<double>(const float *, double, const double *, const double *, int64_t, float *,
                                          hipStream_t);

__global__ void __launch_bounds__(256) apply_kernel(const float *__restrict__ out, double scale, double *__restrict__ J,
                                                    int64_t n)
{
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    double d = scale * (double)out[v];
    d = d < -0.5 ? -0.5 : (d > 1.0 ? 1.0 : d);
    J[v] *= 1.0 + d;
}

hipError_t unet_apply(const float *out, double scale, double *J, int64_t n, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(apply_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, out, scale, J, n);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
std::string parse_unet(const void *blob, size_t bytes, UNetSpec &out)
{
    out = UNetSpec();
    const unsigned char *p = static_cast<const unsigned char *>(blob);
    size_t off = 0;
    auto u32 = [&](uint32_t &v) {
        if (off + 4 > bytes) return false;
        std::memcpy(&v, p + off, 4);
        off += 4;
        return true;
    };
    if (bytes < 12 || std::memcmp(p, "RTUN", 4) != 0) return "not a network blob (magic)";
    off = 4;
    uint32_t ver = 0, L = 0;
    if (!u32(ver) || ver != 1) return "unsupported network blob version";
    if (!u32(L) || L < 1 || L > 6) return "number of levels must be 1..6";
    out.L = (int)L;
    for (uint32_t l = 0; l < L; ++l) {
        uint32_t c = 0;
        if (!u32(c) || (c != 16 && c != 32 && c != 64)) return "channel counts must be 16, 32 or 64";
        out.C.push_back((int)c);
    }
    auto conv = [&](int ci, int co, int taps) {
        UNetSpec::Conv cv;
        cv.ci = ci; cv.co = co; cv.taps = taps;
        const size_t nw = (size_t)taps * co * ci;
        if (off + 4 * (nw + co) > bytes) return false;
        cv.w.resize(nw);
        cv.b.resize(co);
        std::memcpy(cv.w.data(), p + off, 4 * nw);
        off += 4 * nw;
        std::memcpy(cv.b.data(), p + off, 4 * (size_t)co);
        off += 4 * (size_t)co;
        out.convs.push_back(std::move(cv));
        return true;
    };
    const auto &C = out.C;
    if (!conv(3, C[0], 27) || !conv(C[0], C[0], 27)) return "truncated blob";
    for (int l = 1; l < out.L; ++l)
        if (!conv(C[l - 1], C[l], 27) || !conv(C[l], C[l], 27)) return "truncated blob";
    for (int l = out.L - 1; l >= 1; --l)
        if (!conv(C[l], C[l - 1], 27) || !conv(C[l - 1], C[l - 1], 27)) return "truncated blob";
    if (!conv(C[0], 1, 1)) return "truncated blob";
    if (off != bytes) return "trailing bytes after the last layer";
    for (const auto &cv : out.convs)
        for (float x : cv.w)
            if (!std::isfinite(x)) return "non-finite weight";
    return "";
}

struct DevMem {
    void *p = nullptr;
    ~DevMem() { if (p) (void)hipFree(p); }
};

struct UNetDev {
    UNetSpec spec;
    std::vector<Vol> lv;                       // volume of each level
    std::vector<std::unique_ptr<DevMem>> mem;  // every allocation
    std::vector<const void *> w, b;            // per conv: weights (bf16 or fp32), biases (fp32)
    std::vector<uint16_t *> h, t;              // per level activations
    uint16_t *up = nullptr;                    // upsampled map (largest)
};

static hipError_t dev_alloc(UNetDev *u, size_t bytes, void **out)
{
    auto m = std::make_unique<DevMem>();
    hipError_t e = hipMalloc(&m->p, bytes > 0 ? bytes : 16);
    if (e != hipSuccess) return e;
    *out = m->p;
    u->mem.push_back(std::move(m));
    return hipSuccess;
}

UNetDev *unet_create(const UNetSpec &spec, int nx, int ny, int nz, std::string &err)
{
    auto u = std::make_unique<UNetDev>();
    u->spec = spec;
    Vol v{nx, ny, nz};
    for (int l = 0; l < spec.L; ++l) {
        if (l > 0) v = Vol{(v.nx + 1) / 2, (v.ny + 1) / 2, (v.nz + 1) / 2};
        u->lv.push_back(v);
    }
    hipError_t e = hipSuccess;
    for (size_t k = 0; k < spec.convs.size() && e == hipSuccess; ++k) {
        const auto &cv = spec.convs[k];
        const bool mfma = cv.taps == 27 && cv.ci >= 16;
        void *wp = nullptr, *bp = nullptr;
        if (mfma) {
            std::vector<uint16_t> wb(cv.w.size());
            for (size_t i = 0; i < wb.size(); ++i) wb[i] = f2bf_host(cv.w[i]);
            if ((e = dev_alloc(u.get(), wb.size() * 2, &wp)) == hipSuccess)
                e = hipMemcpy(wp, wb.data(), wb.size() * 2, hipMemcpyHostToDevice);
        } else {
            if ((e = dev_alloc(u.get(), cv.w.size() * 4, &wp)) == hipSuccess)
                e = hipMemcpy(wp, cv.w.data(), cv.w.size() * 4, hipMemcpyHostToDevice);
        }
        if (e == hipSuccess && (e = dev_alloc(u.get(), cv.b.size() * 4, &bp)) == hipSuccess)
            e = hipMemcpy(bp, cv.b.data(), cv.b.size() * 4, hipMemcpyHostToDevice);
        u->w.push_back(wp);
        u->b.push_back(bp);
    }
    size_t up_bytes = 0;
    for (int l = 0; l < spec.L && e == hipSuccess; ++l) {
        void *hp = nullptr, *tp = nullptr;
        const size_t bytes = (size_t)u->lv[l].n() * spec.C[l] * 2;
        if ((e = dev_alloc(u.get(), bytes, &hp)) == hipSuccess) e = dev_alloc(u.get(), bytes, &tp);
        u->h.push_back((uint16_t *)hp);
        u->t.push_back((uint16_t *)tp);
        if (l > 0) up_bytes = std::max(up_bytes, (size_t)u->lv[l - 1].n() * spec.C[l] * 2);
    }
    if (e == hipSuccess && spec.L > 1) {
        void *p = nullptr;
        e = dev_alloc(u.get(), up_bytes, &p);
        u->up = (uint16_t *)p;
    }
    if (e != hipSuccess) {
        err = std::string("network buffers: ") + hipGetErrorString(e);
        return nullptr;
    }
    return u.release();
}

void unet_destroy(UNetDev *u) { delete u; }

template <int C>
static hipError_t conv_in_t(const float *f, Vol v, const float *w, const float *b, uint16_t *out, hipStream_t st)
{
    hipLaunchKernelGGL((conv_in_kernel<C>), dim3((unsigned)((v.n() + 255) / 256)), dim3(256), 0, st, f, v, w, b, out);
    return hipGetLastError();
}

hipError_t unet_forward(UNetDev *u, const float *features, float *out, hipStream_t st)
{
    const UNetSpec &s = u->spec;
    const auto &C = s.C;
    size_t k = 0;  // conv index in blob order
    hipError_t e;
    const size_t last = s.convs.size() - 2;  // the convolution that the head follows
    auto conv = [&](const uint16_t *in, Vol vi, Vol vo, int stride, int ci, int co, const uint16_t *skip,
                    uint16_t *o) {
        ConvArgs a{in, vi, vo, stride, (const uint16_t *)u->w[k], (const float *)u->b[k], skip, o};
        HeadArgs hd{};
        if (k == last) hd = HeadArgs{(const float *)u->w[k + 1], (const float *)u->b[k + 1], out};
        ++k;
        return conv_tile(a, ci, co, hd, st);
    };
    // level 0 input layer
    const Vol v0 = u->lv[0];
    switch (C[0]) {
    case 16: e = conv_in_t<16>(features, v0, (const float *)u->w[0], (const float *)u->b[0], u->t[0], st); break;
    case 32: e = conv_in_t<32>(features, v0, (const float *)u->w[0], (const float *)u->b[0], u->t[0], st); break;
    default: e = conv_in_t<64>(features, v0, (const float *)u->w[0], (const float *)u->b[0], u->t[0], st); break;
    }
    if (e != hipSuccess) return e;
    k = 1;
    if ((e = conv(u->t[0], v0, v0, 1, C[0], C[0], nullptr, u->h[0])) != hipSuccess) return e;
    for (int l = 1; l < s.L; ++l) {
        if ((e = conv(u->h[l - 1], u->lv[l - 1], u->lv[l], 2, C[l - 1], C[l], nullptr, u->t[l])) != hipSuccess)
            return e;
        if ((e = conv(u->t[l], u->lv[l], u->lv[l], 1, C[l], C[l], nullptr, u->h[l])) != hipSuccess) return e;
    }
    for (int l = s.L - 1; l >= 1; --l) {
        const Vol vc = u->lv[l], vf = u->lv[l - 1];
        const int log_groups = C[l] == 16 ? 1 : C[l] == 32 ? 2 : 3;
        const int width = vf.nx << log_groups, turns = (width + 1023) / 1024;
        const int threads = ((width + turns - 1) / turns + 63) / 64 * 64;
        hipLaunchKernelGGL(upsample_kernel, dim3((unsigned)vf.ny, (unsigned)std::min(vf.nz, 65535)), dim3(threads), 0, st,
                           u->h[l], vc, u->up, vf, log_groups);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if ((e = conv(u->up, vf, vf, 1, C[l], C[l - 1], u->h[l - 1], u->t[l - 1])) != hipSuccess) return e;
        if ((e = conv(u->t[l - 1], vf, vf, 1, C[l - 1], C[l - 1], nullptr, u->h[l - 1])) != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace rt3d
