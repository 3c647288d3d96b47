// fs_box.hip -- formal solution on the x,y-periodic box (gfx950).
//
// One workgroup sweeps all characteristics of one (wavelength, direction)
// work item through the grid, layer by layer in the direction of travel
// (top to bottom for mu < 0).  Every thread carries the intensity of R rays in
// registers; all rays of a direction share the visit template, so at visit m
// every lane reads the same template entry (scalar loads) and ray r touches
// voxel r + offset_m.  At a fixed m that map is one-to-one, so with a
// workgroup barrier per visit step the layer's J (and Lambda*) tile in LDS is
// updated by plain read-add-write without collisions and in a fixed order
// (bitwise reproducible; no LDS atomics, whose queueing cost a third of the
// kernel time).
// When the template leaves a layer the tile is added into the workgroup's own
// partial-sum slot in HBM.
//
// Per point (Listing 1 of the paper): gather previous/current/next S and chi
// (step 1-2), optical steps (3), interpolation weights with the linear
// fallback (4) and vacuum fix-up (4a), Lambda* data (4b), exp(-dtau) and the
// intensity update (5).  Optical steps and weights are evaluated in double;
// the recurrence and the J accumulation run in the field type T.
//
// Fields are read from doubly periodic padded copies [Nz][2Ny][2Nx], so the
// address of ray r at visit m is base_r + offset_m with no wrap arithmetic.
//
// Band tiles (layers too wide for LDS): the rays of a direction are split
// into bundles of whole ray rows, and a workgroup's tile holds only the rows
// that its bundle reaches within the current layer.  Within one layer the
// template's row offsets span at most `span` rows (its horizontal travel per
// layer), so rays of origin rows [yb, yb + h) land in the h + span + 1 rows
// that start at yb + (lowest template row of the layer); the visit table
// carries each visit's row relative to that lowest row.  The tile index is
// then (origin row - yb + relative row) * Nx + x, and the flush maps tile
// word i to layer word (base * Nx + i) mod NxNy.  A band covers only part of
// a layer, so the first item of a slot also stores zeros to the rest of each
// layer that it flushes.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "fs_box.hpp"
#include "fs_point.hpp"

namespace rt3d {

// ---------------------------------------------------------------------------
// field loads: one raw buffer load per point fetches the (chi, S) pair; the
// per-ray byte offset sits in a VGPR, the per-visit byte offset in an SGPR,
// so there is no per-lane address arithmetic
// ---------------------------------------------------------------------------
__device__ __forceinline__ __amdgpu_buffer_rsrc_t field_rsrc(const void *base, uint32_t bytes, int stride)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)stride, (int)bytes, 0x00020000);
}

template <typename T>
struct Pair {
    T chi, S;
};

// Structured buffer load: byte address base + index * stride + soff.
typedef int v2i __attribute__((ext_vector_type(2)));
__device__ v2i struct_load_b64(__amdgpu_buffer_rsrc_t r, int index, int voff, int soff,
                               int aux) __asm("llvm.amdgcn.struct.ptr.buffer.load.v2i32");

template <typename T>
__device__ __forceinline__ Pair<T> ld_pair(__amdgpu_buffer_rsrc_t r, int voff, int soff);

template <>
__device__ __forceinline__ Pair<float> ld_pair<float>(__amdgpu_buffer_rsrc_t r, int voff, int soff)
{
    return __builtin_bit_cast(Pair<float>, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}

template <>
__device__ __forceinline__ Pair<double> ld_pair<double>(__amdgpu_buffer_rsrc_t r, int voff, int soff)
{
    return __builtin_bit_cast(Pair<double>, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}

// ---------------------------------------------------------------------------
// the sweep kernel
// ---------------------------------------------------------------------------
// Fused multiply-add in the recurrence type.
__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }

// A value that is the same in every lane, kept in a scalar register: the
// weight of a visit, formed by vector instructions from scalar inputs, then
// serves every ray of the thread as a scalar operand.  Double values stay
// as they are.
__device__ __forceinline__ float uniform(float v)
{
    // by an explicit v_readfirstlane (the builtin would be moved ahead of the
    // conversion to single precision, which is then redone per ray).  A
    // readlane of a VGPR that the previous VALU instruction wrote needs wait
    // states in between, which the compiler inserts only around its own
    // instructions: the s_nop gives them here.
    float s;
    asm("s_nop 1\n\tv_readfirstlane_b32 %0, %1" : "=s"(s) : "v"(v));
    return s;
}
__device__ __forceinline__ double uniform(double v) { return v; }

// A double loaded from the same address by every lane, in scalar registers (no
// instruction where the compiler already has it there).
__device__ __forceinline__ double scalar(double v)
{
    return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                            __builtin_amdgcn_readfirstlane(__double2loint(v)));
}

template <typename T, int LB, int R, bool WJ, bool WL, bool PARA, int OCC, bool BAND>
__global__ void __launch_bounds__(LB) __attribute__((amdgpu_waves_per_eu(OCC * LB / 256 > 0 ? OCC * LB / 256 : 1)))
fs_box_kernel(FsBoxArgs a)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int Nx = a.Nx, Ny = a.Ny;
    const int NxNy = Nx * Ny;
    const int tid = threadIdx.x;
    const int nthr = blockDim.x;
    // tiles of tile_words words plus one scratch word per thread (padding slots)
    const int TW = a.tile_words;
    T *tJ = reinterpret_cast<T *>(smem_raw);
    T *tL = tJ + (WJ ? TW + nthr : 0);
    constexpr int ES = 2 * (int)sizeof(T);  // bytes per (chi, S) pair
    // Single-precision band tiles of single-output sweeps are two layer rows
    // wide, like the padded field: a ray's column x0 + dx (below 2 Nx) then
    // needs no wrap, and the layer flush adds word x + Nx of a tile row to
    // column x.  (Two outputs at twice the width would leave room for fewer
    // rows per band.)
    constexpr bool WIDE = BAND && sizeof(T) == 4 && !(WJ && WL);
    // What is kept in registers besides the intensities and addresses, by what
    // the shape's waves per SIMD leave beside about kTmp temporaries of a point
    // (set so that no kernel spills that would not otherwise):
    //   CARRY  the state carried along a ray from visit to visit (see below)
    //   DEPTH  of it, the half depth of the current point (else its opacity)
    //   PRE    field pairs in flight, read this many rays ahead, past the barrier
    //          into the next visit (at most all of a thread's rays); 0: the next
    //          ray's pair, within the visit
    //   TPRE   a ray's tile words are read while the ray before it is computed,
    //          and the visit table two visits ahead
    constexpr int kWaves = OCC * LB / 256 > 0 ? OCC * LB / 256 : 1;
    constexpr int kRegs = kWaves > 2 ? (512 / kWaves) & ~7 : 256;
    constexpr int kWords = (int)sizeof(T) / 4;
    constexpr int kTmp = (sizeof(T) == 8 ? 84 : 74) + (WL ? 10 : 0);
    constexpr int kAddr = WIDE ? 1 : 2, kPara = WL && PARA ? kWords : 0;
    constexpr int kState = kAddr + 3 + (WJ ? 3 * kWords : 0) + kPara;
    constexpr bool CARRY = sizeof(T) == 4 || R * (kState + 1) + kTmp <= kRegs;
    constexpr bool DEPTH = CARRY && R * (kState + 1) + kTmp <= kRegs;
    constexpr int kUsed = CARRY ? R * (kState + DEPTH) + kTmp : R * (kAddr + (WJ ? kWords : 0) + kPara) + kTmp + 16;
    constexpr int kFree = kRegs > kUsed ? (kRegs - kUsed) / (2 * kWords) : 0;
    constexpr int PRE = !CARRY ? 0 : kFree < R ? kFree : R;
    constexpr bool TPRE = kUsed + 2 <= kRegs;
    // Words of a layer flush per thread whose slot reads are issued together: a
    // flush waits for memory once per such group, so as many as find room in the
    // registers that a visit's temporaries leave (eighteen beside eight rays and more
    // from 160 registers up, else eight).  Larger bands take more groups; the 98 rows
    // of 129 words of a 768-thread band take one, where groups of eight waited three
    // times at every layer.
    constexpr int FLUSH = WIDE && R >= 8 && kRegs >= 160 ? 18 : 8;
    // Wavefront priority by progress within a visit (see step): pays where a visit is
    // long and few waves share a SIMD, ten to twelve rays a thread (64.6 -> 62.0 ms
    // with the look-ahead at 768 x 11 on 129^3 x 2048 directions).  Neutral or slower
    // for shorter and longer visits, and with two outputs the registers around the rays'
    // blocks spill (the same, J and Lambda*: 88.8 ms with, 77.8 without).
    constexpr bool kPrio = R >= 10 && R <= 12 && !(WJ && WL);

    for (int i = tid; i < TW + nthr; i += nthr) {
        if (WJ) tJ[i] = T(0);
        if (WL) tL[i] = T(0);
    }

    // The rays of a direction may be split into bundles of consecutive ray
    // indices; workgroup w always sweeps bundle w mod n_bundles (its own layer
    // tile and partial slot), so smaller workgroups with fewer rays per thread
    // can share a CU.  Rays of this thread: local index l = tid + j*nthr of
    // the bundle, origin (x0, y0) of ray q_lo + l.  Slots past the bundle's
    // last ray repeat an earlier ray of the bundle and contribute exactly
    // zero.  The host admits a launch shape only if nthr * (R - 1) is below
    // the smallest bundle, so only the last slot (j = R - 1) of a thread can
    // be such a padding slot and the other R - 1 copies of the point body
    // carry no padding logic.
    const int bundle = a.n_bundles > 1 ? (int)(blockIdx.x % (unsigned)a.n_bundles) : 0;
    int q_lo, q_n, yb = 0, hb = 0;
    if (BAND) {
        yb = (int)(((int64_t)bundle * Ny) / a.n_bundles);
        hb = (int)(((int64_t)(bundle + 1) * Ny) / a.n_bundles) - yb;
        q_lo = yb * Nx;
        q_n = hb * Nx;
    } else {
        q_lo = bundle * a.bundle_rays;
        q_n = min(a.bundle_rays, NxNy - q_lo);
    }
    // Constants per ray j of this thread: vb[j], the byte offset of its origin
    // in the padded field (the per-visit part of the address is scalar), and
    // tw[j] = x0 << 19 | (tile word of its origin) * sizeof(T): its high field
    // decides the x wrap of a visit by one unsigned comparison with a scalar,
    // its low field (< 2^19: LDS bytes) is the tile address before the visit's
    // scalar offset.  Wide tiles have the pitch of the padded field, so one
    // number serves both: vb[j] is then the pair's index (structured loads
    // scale it by the pair size) and the tile address is 4 vb[j] + offset, and
    // tw is not kept.  Rows are relative to the bundle's first row yb for band
    // tiles.  Only the last slot of a thread can be a padding slot (padj).
    const uint32_t row_bytes = (uint32_t)(2 * Nx * ES);
    const uint32_t tpitch = WIDE ? 2u * (uint32_t)Nx : (uint32_t)Nx;
    const int gshift = BAND ? (int)((uint32_t)yb * row_bytes) : 0;
    constexpr uint32_t kTileMask = (1u << 19) - 1u;
    int vb[R];
    uint32_t tw[WIDE ? 1 : R];
    bool padj = false;
#pragma unroll
    for (int j = 0; j < R; ++j) {
        int l = tid + j * nthr;
        bool pad = false;
        while (l >= q_n) { l -= q_n; pad = true; }
        const int q = q_lo + l;
        const int y0 = q / Nx;
        const int x0 = q - y0 * Nx;
        const uint32_t yr = (uint32_t)(y0 - yb);
        if constexpr (WIDE) {
            vb[j] = (int)(yr * tpitch + (uint32_t)x0);
        } else {
            vb[j] = (int)(yr * row_bytes + (uint32_t)x0 * ES);
            tw[j] = ((uint32_t)x0 << 19) | ((yr * tpitch + (uint32_t)x0) * (uint32_t)sizeof(T));
        }
        if (j == R - 1) padj = pad;
    }
    unsigned char *const tJb = reinterpret_cast<unsigned char *>(tJ);
    unsigned char *const tLb = reinterpret_cast<unsigned char *>(tL);
    const uint32_t pad_addr = (uint32_t)(TW + tid) * (uint32_t)sizeof(T);
    const int f_row0 = tid / Nx, f_x0 = tid - f_row0 * Nx;    // flush position of this thread
    const int f_drow = nthr / Nx, f_dx = nthr - f_drow * Nx;  // and its step
    __syncthreads();

    const uint32_t slice_bytes = (uint32_t)(a.pad_stride * ES);
    const int it_end = a.wg_begin[blockIdx.x + 1];
    for (int it = a.wg_begin[blockIdx.x]; it < it_end; ++it) {
        const WorkItem item = a.items[it];
        const int lam = item.lambda;
        const int d = item.dir;
        const __amdgpu_buffer_rsrc_t rf = field_rsrc(
            reinterpret_cast<const T *>(a.field) + 2 * (int64_t)lam * a.pad_stride, slice_bytes, WIDE ? ES : 0);
        // the (chi, S) pair of ray j at scalar byte offset g
        auto field = [&](int j, int g) {
            if constexpr (WIDE) {
                const v2i v = struct_load_b64(rf, vb[j], 0, g, 0);
                return Pair<T>{__int_as_float(v.x), __int_as_float(v.y)};
            } else {
                return ld_pair<T>(rf, vb[j], g);
            }
        };
        T *__restrict__ pJ = WJ ? reinterpret_cast<T *>(a.partJ) + (int64_t)item.slot * a.n_vox : nullptr;
        T *__restrict__ pL = WL ? reinterpret_cast<T *>(a.partL) + (int64_t)item.slot * a.n_vox : nullptr;
        const bool first = item.first != 0;
        const int64_t vbeg = a.dir_vbegin[d];
        const int M = a.dir_M[d];
        const double wmu = a.dir_wmu[d];
        const bool down = a.dir_mu[d] < 0.0;
        const T Ibc = a.I_bc ? reinterpret_cast<const T *>(a.I_bc)[2 * lam + (down ? 0 : 1)] : T(0);
        const int32_t *__restrict__ goff = a.goff + vbeg;
        const uint32_t *__restrict__ dxy = a.dxy + vbeg;
        const double *__restrict__ sv = a.s + vbeg;
        const int32_t *__restrict__ brow = BAND ? a.brow + vbeg : nullptr;
        const int span = BAND ? a.dir_span[d] : 0;

        T I[R];
        T gprev[R];
        int layer = down ? 0 : a.Nz - 1;
        const int dlayer = down ? 1 : -1;

        // first item of a slot: zeros to the layer's words outside the band
        auto clear_rest = [&](T *__restrict__ part, int64_t lo, uint32_t g0, int n) {
            if (!first) return;
            for (int i = n + tid; i < NxNy; i += nthr) {
                const uint32_t gi = g0 + (uint32_t)i;
                part[lo + min(gi, gi - (uint32_t)NxNy)] = T(0);
            }
        };
        // w, r: offsets word and relative row of the layer's last visit
        auto flush_layer = [&](uint32_t w, int r) {
            const int64_t lo = (int64_t)layer * NxNy;
            if (BAND) {
                // tile row 0 is layer row yb + (lowest template row of the layer)
                int base = (yb + (int)((w >> kOffBits) & kOffMask) - r) % Ny;
                if (base < 0) base += Ny;
                const uint32_t g0 = (uint32_t)base * (uint32_t)Nx;
                const int n = (hb + span + 1) * Nx;
                if (WIDE) {
                    // output word i = row Nx + x takes tile words row 2Nx + x and
                    // row 2Nx + x + Nx; row and x advance without division.  A
                    // single-output sweep (one tile, one slot); FLUSH words of a
                    // thread at a time, their slot reads issued together
                    T *const tile = WJ ? tJ : tL;
                    T *__restrict__ const part = WJ ? pJ : pL;
                    int row = f_row0, x = f_x0;
                    auto layer_word = [&](int i) {
                        const uint32_t gi = g0 + (uint32_t)i;
                        return min(gi, gi - (uint32_t)NxNy);
                    };
                    constexpr int U = FLUSH;
                    for (int i = tid; i < n; i += U * nthr) {
                        T old[U];
                        // slots past the band end only the thread's last group
#pragma unroll
                        for (int u = 0; u < U; ++u)
                            if (i + u * nthr < n) old[u] = first ? T(0) : part[lo + layer_word(i + u * nthr)];
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            int k = i + u * nthr;
                            asm("" : "+v"(k));  // form the address again instead of keeping it from the read
                            if (k < n) {
                                T *const t0 = tile + (k + row * Nx);
                                const T v = t0[0] + t0[Nx];
                                t0[0] = T(0);
                                t0[Nx] = T(0);
                                part[lo + layer_word(k)] = old[u] + v;
                                x += f_dx;
                                row += f_drow;
                                if (x >= Nx) {
                                    x -= Nx;
                                    ++row;
                                }
                            }
                        }
                    }
                    clear_rest(part, lo, g0, n);
                    layer += dlayer;
                    __syncthreads();
                    return;
                }
                // some words of a thread at a time, their slot reads issued together
                constexpr int U = FLUSH / 2;
                for (int i = tid; i < n; i += U * nthr) {
                    uint32_t gi[U];
                    T oJ[U], oL[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        gi[u] = g0 + (uint32_t)(i + u * nthr);
                        gi[u] = min(gi[u], gi[u] - (uint32_t)NxNy);
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (i + u * nthr < n) {
                            if (WJ) oJ[u] = first ? T(0) : pJ[lo + gi[u]];
                            if (WL) oL[u] = first ? T(0) : pL[lo + gi[u]];
                        }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int k = i + u * nthr;
                        if (k < n) {
                            if (WJ) {
                                const T v = tJ[k];
                                tJ[k] = T(0);
                                pJ[lo + gi[u]] = oJ[u] + v;
                            }
                            if (WL) {
                                const T v = tL[k];
                                tL[k] = T(0);
                                pL[lo + gi[u]] = oL[u] + v;
                            }
                        }
                    }
                }
                if (WJ) clear_rest(pJ, lo, g0, n);
                if (WL) clear_rest(pL, lo, g0, n);
            } else {
                constexpr int U = 4;
                for (int i = tid; i < NxNy; i += U * nthr) {
                    T oJ[U], oL[U];
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (i + u * nthr < NxNy) {
                            if (WJ) oJ[u] = first ? T(0) : pJ[lo + i + u * nthr];
                            if (WL) oL[u] = first ? T(0) : pL[lo + i + u * nthr];
                        }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int k = i + u * nthr;
                        if (k < NxNy) {
                            if (WJ) {
                                const T v = tJ[k];
                                tJ[k] = T(0);
                                pJ[lo + k] = oJ[u] + v;
                            }
                            if (WL) {
                                const T v = tL[k];
                                tL[k] = T(0);
                                pL[lo + k] = oL[u] + v;
                            }
                        }
                    }
                }
            }
            layer += dlayer;
            __syncthreads();
        };
        // Scalar part of a visit's tile addresses: byte offset of the visit's
        // horizontal offsets (dx, and the relative row r or dy), the x-wrap
        // threshold (Nx - dx) << 19 on tw, and for layer tiles the y-wrap
        // threshold on the tile address.
        struct TileStep {
            uint32_t off, thx, thy;
        };
        auto tile_step = [&](uint32_t w, int r) {
            const uint32_t dx = w & kOffMask;
            TileStep s;
            s.thx = ((uint32_t)Nx - dx) << 19;
            if (BAND) {
                s.off = ((uint32_t)r * tpitch + dx) * (uint32_t)sizeof(T);
                s.thy = 0;
                // opaque, so that 4 vb + off stays one shift-and-add per ray
                s.off = (uint32_t)__builtin_amdgcn_readfirstlane((int)s.off);
                asm("" : "+s"(s.off));
            } else {
                const uint32_t dy = (w >> kOffBits) & kOffMask;
                s.off = (dy * (uint32_t)Nx + dx) * (uint32_t)sizeof(T);
                s.thy = ((uint32_t)Ny - dy) * (uint32_t)Nx * (uint32_t)sizeof(T);
            }
            return s;
        };
        // LDS byte address of ray j's voxel at a visit; padding slots go to
        // this thread's own word past the tile, so no two lanes ever update
        // the same word in one step
        auto tile_addr = [&](int j, const TileStep &s) {
            uint32_t a4;
            if constexpr (WIDE) {
                a4 = ((uint32_t)vb[j] << 2) + s.off;
            } else {
                const uint32_t base = tw[j] & kTileMask;
                a4 = base + s.off;
                a4 -= tw[j] >= s.thx ? (uint32_t)Nx * (uint32_t)sizeof(T) : 0u;
                if (!BAND) a4 -= base >= s.thy ? (uint32_t)NxNy * (uint32_t)sizeof(T) : 0u;
            }
            return (j == R - 1 && padj) ? pad_addr : a4;
        };
        // the visit weight, zero for a padding slot
        auto ray_weight = [&](int j, T cw) { return (j == R - 1 && padj) ? T(0) : cw; };
        auto tile_word = [&](unsigned char *tile, uint32_t addr) -> T & { return *reinterpret_cast<T *>(tile + addr); };

        // Carried along each ray from one visit to the next: the sources of the
        // previous and current points (Sp, Sc), the half depth of the current
        // point (tc; its opacity Xc where registers are short) and the optical
        // step from the previous point to the current one (Dc); each visit then
        // reads only the next point's (chi, S) pair.  Double sweeps with many rays per thread have no
        // registers for it and read the previous, current and next pairs at
        // every visit instead.
        T Sp[CARRY ? R : 1], Sc[CARRY ? R : 1];
        double tc[DEPTH ? R : 1], Dc[CARRY ? R : 1];
        T Xc[CARRY && !DEPTH ? R : 1];
        Pair<T> pf[PRE > 0 ? PRE : 1];  // queue of downwind pairs in flight
        int g_p = 0;
        double s_p = 0.0;

        // The visit table is read ahead of its use, so that no wave waits for
        // it right after a barrier: visit c is the current one, n the next, and
        // g_2, s_2, w_2, r_2 (g_3) belong to the visit(s) after it; past the
        // ray's end they repeat the last visit.  Path lengths are halved.
        const int i1 = min(1, M - 1), i2 = min(2, M - 1), i3 = min(3, M - 1);
        int g_c = goff[0] * ES + gshift, g_n = goff[i1] * ES + gshift, g_2 = goff[i2] * ES + gshift;
        int g_3 = PRE > 0 ? goff[i3] * ES + gshift : 0;
        double s_c = scalar(sv[0]), s_n = scalar(sv[i1]), s_2 = scalar(sv[i2]);
        uint32_t w_c = dxy[0], w_n = dxy[i1], w_2 = dxy[i2];
        int r_c = BAND ? brow[0] : 0, r_n = BAND ? brow[i1] : 0, r_2 = BAND ? brow[i2] : 0;
        // first point: entry half-segment with constant S; the second point's
        // pair is read too (the first optical step between points needs it)
        {
            const T cw = T(wmu * (2.0 * s_c));
            const TileStep ts = tile_step(w_c, r_c);
#pragma unroll
            for (int j = 0; j < R; ++j) {
                gprev[j] = T(0);
                const Pair<T> f0 = field(j, g_c);
                const double t0 = half_depth((double)f0.chi, s_c);
                T ex, e0;
                entry_weights<T>(t0, ex, e0);
                I[j] = WJ ? Ibc * ex + f0.S * e0 : T(0);
                const uint32_t ad = tile_addr(j, ts);
                const T cj = ray_weight(j, cw);
                if (WJ) tile_word(tJb, ad) += cj * I[j];
                if (WL) tile_word(tLb, ad) += cj * e0;
                if constexpr (CARRY) {
                    const Pair<T> f1 = field(j, g_n);
                    Sp[j] = f0.S;
                    Sc[j] = f1.S;
                    const double t1 = half_depth((double)f1.chi, s_n);
                    Dc[j] = step_of(t0, t1);
                    if constexpr (DEPTH) tc[j] = t1;
                    else Xc[j] = f1.chi;
                }
                if (j < PRE) pf[j] = field(j, g_2);
            }
            __syncthreads();
            if (w_c & kLayerEnd) flush_layer(w_c, r_c);
        }

        // one point of every ray of this thread; LAST: the final point, which
        // has no downwind neighbour
        auto step = [&](auto last_tag) {
            constexpr bool LAST = decltype(last_tag)::value;
            const T cw = uniform(T(wmu * (2.0 * s_c)));
            const TileStep ts = tile_step(w_c, r_c);
            // software pipeline over the rays of this thread and on into the
            // next visit: the loads of the next PRE rays are in flight while a
            // ray is computed, so that no wave waits for memory right after the
            // barrier, and a field larger than the caches (257^3) hides its HBM
            // latency (one pair in flight: 174 ms at ten rays a thread, 168
            // ms with three)
            const Pair<T> zero{T(0), T(0)};
            Pair<T> nn = LAST || PRE > 0 ? zero : field(0, g_n);
            Pair<T> np = CARRY ? zero : field(0, g_p);
            Pair<T> nc = CARRY ? zero : field(0, g_c);
            // so are its tile words: at one visit no two rays share a word
            uint32_t na = tile_addr(0, ts);
            T nJ = TPRE && WJ ? tile_word(tJb, na) : T(0), nL = TPRE && WL ? tile_word(tLb, na) : T(0);
#pragma unroll
            for (int j = 0; j < R; ++j) {
                // a wave that is behind its neighbours goes first, so that the
                // waves of a SIMD reach the barrier together instead of the last
                // one running alone
                if (kPrio) {
                    if (j == 0) __builtin_amdgcn_s_setprio(3);
                    else if (j == (R + 3) / 4) __builtin_amdgcn_s_setprio(2);
                    else if (j == (2 * R + 3) / 4) __builtin_amdgcn_s_setprio(1);
                    else if (j == (3 * R + 3) / 4) __builtin_amdgcn_s_setprio(0);
                }
                Pair<T> fn = nn;
                const Pair<T> fp = np, fc = nc;
                if constexpr (PRE > 0 && !LAST) {
                    fn = pf[0];
#pragma unroll
                    for (int k = 0; k + 1 < PRE; ++k) pf[k] = pf[k + 1];
                    pf[PRE - 1] = j + PRE < R ? field(j + PRE < R ? j + PRE : 0, g_n) : field(j + PRE < R ? 0 : j + PRE - R, g_2);
                }
                const uint32_t ad = TPRE ? na : tile_addr(j, ts);
                T oJ = nJ, oL = nL;
                if (j + 1 < R) {
                    if (TPRE) {
                        na = tile_addr(j + 1, ts);
                        if (WJ) nJ = tile_word(tJb, na);
                        if (WL) nL = tile_word(tLb, na);
                    }
                    if (!LAST && PRE == 0) nn = field(j + 1, g_n);
                    if (!CARRY) {
                        np = field(j + 1, g_p);
                        nc = field(j + 1, g_c);
                    }
                }
                double D, Dp = 0.0, tn = 0.0;
                T S_prev, S_cur;
                if constexpr (CARRY) {
                    D = Dc[j];
                    S_prev = Sp[j];
                    S_cur = Sc[j];
                    if (!LAST) {
                        tn = half_depth((double)fn.chi, s_n);
                        Dp = step_of(DEPTH ? tc[DEPTH ? j : 0] : half_depth((double)Xc[DEPTH ? 0 : j], s_c), tn);
                    }
                } else {
                    const double hc = half_depth((double)fc.chi, s_c);
                    D = step_of(half_depth((double)fp.chi, s_p), hc);
                    if (!LAST) Dp = step_of(hc, half_depth((double)fn.chi, s_n));
                    S_prev = fp.S;
                    S_cur = fc.S;
                }
                const PointW<T> pw = point_weights_pos<T, LAST, WL && !PARA>(D, Dp);
                if (WJ) {
                    // accumulated in place: I ex, then the three source terms
                    T Ij = I[j] * pw.ex;
                    Ij = fma_t(pw.a, S_prev, Ij);
                    Ij = fma_t(pw.b, S_cur, Ij);
                    if (!LAST) Ij = fma_t(pw.g, fn.S, Ij);
                    I[j] = Ij;
                }
                const T cj = ray_weight(j, cw);
                if (!TPRE && WJ) oJ = tile_word(tJb, ad);
                if (!TPRE && WL) oL = tile_word(tLb, ad);
                if (WJ) tile_word(tJb, ad) = oJ + cj * I[j];
                if (WL) {
                    T dloc;
                    if (PARA) {
                        dloc = pw.b + gprev[j] * pw.ex;
                        gprev[j] = pw.g;
                    } else {
                        dloc = pw.dlin;
                    }
                    tile_word(tLb, ad) = oL + cj * dloc;
                }
                if constexpr (CARRY && !LAST) {
                    Sp[j] = Sc[j];
                    Sc[j] = fn.S;
                    if constexpr (DEPTH) tc[j] = tn;
                    else Xc[j] = fn.chi;
                    Dc[j] = Dp;
                }
            }
            __syncthreads();
            if (w_c & kLayerEnd) flush_layer(w_c, r_c);
        };

        // the final point is taken after the loop, so that the loop body has a
        // single path (no merge of the carried per-ray state)
        auto advance = [&](int m) {
            g_p = g_c;
            s_p = s_c;
            g_c = g_n;
            s_c = s_n;
            w_c = w_n;
            r_c = r_n;
            const int m2 = min(m + 2, M - 1);
            if constexpr (!TPRE) {
                const int m1 = min(m + 1, M - 1);
                g_n = goff[m1] * ES + gshift;
                s_n = scalar(sv[m1]);
                w_n = dxy[m1];
                if (BAND) r_n = brow[m1];
                if (PRE > 0) g_2 = goff[m2] * ES + gshift;
                return;
            }
            g_n = g_2;
            s_n = s_2;
            w_n = w_2;
            r_n = r_2;
            s_2 = scalar(sv[m2]);
            w_2 = dxy[m2];
            if (BAND) r_2 = brow[m2];
            if (PRE > 0) {
                g_2 = g_3;
                g_3 = goff[min(m + 3, M - 1)] * ES + gshift;
            } else {
                g_2 = goff[m2] * ES + gshift;
            }
        };
        for (int m = 1; m + 1 < M; ++m) {
            advance(m);
            step(std::false_type{});
        }
        if (M > 1) {
            advance(M - 1);
            step(std::true_type{});
        }
    }
}

// ---------------------------------------------------------------------------
// host-side dispatch
//
// Launch shapes: (threads per workgroup bound LB, rays per thread R).  All
// output combinations exist for LB = 1024; the other shapes exist for the
// J-only kernel, which runs every ALI step and is the one the autotuner
// (rt_autotune) times.
// ---------------------------------------------------------------------------
// Launch shapes (threads bound LB, rays per thread R, workgroups per CU OCC).
// OCC = 2 shapes split each direction's rays into two bundles so that two
// workgroups (two layer tiles) share a CU: twice the resident waves to hide
// the latency of the double-precision point arithmetic.  Band-tile shapes
// serve layers too wide for a whole-layer tile (and grids that ask for band
// tiles); their bundle count follows from the LDS left per workgroup.
#define RT_FS_SHAPES_FULL(X)                                                                                 \
    X(1024, 1, 1) X(1024, 2, 1) X(1024, 4, 1) X(1024, 8, 1) X(1024, 12, 1) X(1024, 17, 1) X(1024, 24, 1) \
        X(768, 6, 1) X(768, 11, 1)
#define RT_FS_SHAPES_TUNE(X)                                                                                     \
    X(768, 2, 1) X(768, 8, 1) X(768, 22, 1) X(768, 32, 1) X(512, 33, 1) X(256, 5, 1) X(256, 17, 1) X(256, 34, 1) \
        X(512, 3, 2) X(512, 7, 2) X(512, 9, 2) X(512, 17, 2)
#define RT_FS_SHAPES_BAND_FULL(X)                                                                            \
    X(1024, 1, 1) X(1024, 2, 1) X(1024, 4, 1) X(1024, 8, 1) X(1024, 12, 1) X(1024, 17, 1) X(768, 6, 1) \
        X(768, 11, 1)
#define RT_FS_SHAPES_BAND_TUNE(X) \
    X(768, 8, 1) X(768, 10, 1) X(896, 10, 1) X(768, 22, 1) X(512, 6, 2) X(512, 7, 2) X(512, 9, 2) X(512, 17, 2)

static const FsShape kShapes[] = {
#define RT_LIST(lb, r, o) {lb, r, true, o, false},
    RT_FS_SHAPES_FULL(RT_LIST)
#undef RT_LIST
#define RT_LIST(lb, r, o) {lb, r, false, o, false},
    RT_FS_SHAPES_TUNE(RT_LIST)
#undef RT_LIST
#define RT_LIST(lb, r, o) {lb, r, true, o, true},
    RT_FS_SHAPES_BAND_FULL(RT_LIST)
#undef RT_LIST
#define RT_LIST(lb, r, o) {lb, r, false, o, true},
    RT_FS_SHAPES_BAND_TUNE(RT_LIST)
#undef RT_LIST
};

int fs_box_shapes(const FsShape **out)
{
    *out = kShapes;
    return (int)(sizeof(kShapes) / sizeof(kShapes[0]));
}

template <typename T, int LB, int R, bool WJ, bool WL, bool PARA, int OCC, bool BAND>
static hipError_t launch_one(const FsBoxArgs &a, int n_wg, int nthr, size_t lds, hipStream_t st)
{
    auto k = fs_box_kernel<T, LB, R, WJ, WL, PARA, OCC, BAND>;
    hipError_t e = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3(n_wg), dim3(nthr), lds, st, a);
    return hipGetLastError();
}

// Resident workgroups per CU; negative when the compiled kernel spills
// registers to scratch memory (the host then prefers other shapes).  Up to five
// words are tolerated: they are set-up values parked once per work item, and
// such shapes time like their neighbours without any.
template <typename T, int LB, int R, bool WJ, bool WL, bool PARA, int OCC, bool BAND>
static int occ_one(int nthr, size_t lds)
{
    const auto k = fs_box_kernel<T, LB, R, WJ, WL, PARA, OCC, BAND>;
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k, nthr, lds) != hipSuccess) return 0;
    hipFuncAttributes attr{};
    if (hipFuncGetAttributes(&attr, (const void *)k) != hipSuccess) return 0;
    return attr.localSizeBytes > 20 ? -n : n;
}

template <typename T, int LB, int R, int OCC, bool BAND>
static hipError_t launch_flags(const FsBoxArgs &a, bool wj, bool wl, bool para, int n_wg, int nthr, size_t lds,
                               hipStream_t st)
{
    if (wj && wl && para) return launch_one<T, LB, R, true, true, true, OCC, BAND>(a, n_wg, nthr, lds, st);
    if (wj && wl) return launch_one<T, LB, R, true, true, false, OCC, BAND>(a, n_wg, nthr, lds, st);
    if (wj) return launch_one<T, LB, R, true, false, false, OCC, BAND>(a, n_wg, nthr, lds, st);
    if (wl && para) return launch_one<T, LB, R, false, true, true, OCC, BAND>(a, n_wg, nthr, lds, st);
    if (wl) return launch_one<T, LB, R, false, true, false, OCC, BAND>(a, n_wg, nthr, lds, st);
    return hipSuccess;
}

template <typename T, int LB, int R, int OCC, bool BAND>
static int occ_flags(bool wj, bool wl, bool para, int nthr, size_t lds)
{
    if (wj && wl && para) return occ_one<T, LB, R, true, true, true, OCC, BAND>(nthr, lds);
    if (wj && wl) return occ_one<T, LB, R, true, true, false, OCC, BAND>(nthr, lds);
    if (wj) return occ_one<T, LB, R, true, false, false, OCC, BAND>(nthr, lds);
    if (wl && para) return occ_one<T, LB, R, false, true, true, OCC, BAND>(nthr, lds);
    if (wl) return occ_one<T, LB, R, false, true, false, OCC, BAND>(nthr, lds);
    return 0;
}

template <typename T>
static hipError_t launch_t(const FsBoxArgs &a, bool wj, bool wl, bool para, bool band, int lb, int R, int n_wg,
                           int nthr, size_t lds, hipStream_t st)
{
    const bool j_only = wj && !wl;
    if (!band) {
#define RT_CASE(LBv, Rv, Ov) \
    if (lb == LBv && R == Rv) return launch_flags<T, LBv, Rv, Ov, false>(a, wj, wl, para, n_wg, nthr, lds, st);
        RT_FS_SHAPES_FULL(RT_CASE)
#undef RT_CASE
        if (!j_only) return hipErrorInvalidValue;
#define RT_CASE(LBv, Rv, Ov) \
    if (lb == LBv && R == Rv) return launch_one<T, LBv, Rv, true, false, false, Ov, false>(a, n_wg, nthr, lds, st);
        RT_FS_SHAPES_TUNE(RT_CASE)
#undef RT_CASE
    } else {
#define RT_CASE(LBv, Rv, Ov) \
    if (lb == LBv && R == Rv) return launch_flags<T, LBv, Rv, Ov, true>(a, wj, wl, para, n_wg, nthr, lds, st);
        RT_FS_SHAPES_BAND_FULL(RT_CASE)
#undef RT_CASE
        if (!j_only) return hipErrorInvalidValue;
#define RT_CASE(LBv, Rv, Ov) \
    if (lb == LBv && R == Rv) return launch_one<T, LBv, Rv, true, false, false, Ov, true>(a, n_wg, nthr, lds, st);
        RT_FS_SHAPES_BAND_TUNE(RT_CASE)
#undef RT_CASE
    }
    return hipErrorInvalidValue;
}

template <typename T>
static int occ_t(bool wj, bool wl, bool para, bool band, int lb, int R, int nthr, size_t lds)
{
    const bool j_only = wj && !wl;
    if (!band) {
#define RT_CASE(LBv, Rv, Ov) \
    if (lb == LBv && R == Rv) return occ_flags<T, LBv, Rv, Ov, false>(wj, wl, para, nthr, lds);
        RT_FS_SHAPES_FULL(RT_CASE)
#undef RT_CASE
        if (!j_only) return 0;
#define RT_CASE(LBv, Rv, Ov) \
    if (lb == LBv && R == Rv) return occ_one<T, LBv, Rv, true, false, false, Ov, false>(nthr, lds);
        RT_FS_SHAPES_TUNE(RT_CASE)
#undef RT_CASE
    } else {
#define RT_CASE(LBv, Rv, Ov) \
    if (lb == LBv && R == Rv) return occ_flags<T, LBv, Rv, Ov, true>(wj, wl, para, nthr, lds);
        RT_FS_SHAPES_BAND_FULL(RT_CASE)
#undef RT_CASE
        if (!j_only) return 0;
#define RT_CASE(LBv, Rv, Ov) \
    if (lb == LBv && R == Rv) return occ_one<T, LBv, Rv, true, false, false, Ov, true>(nthr, lds);
        RT_FS_SHAPES_BAND_TUNE(RT_CASE)
#undef RT_CASE
    }
    return 0;
}

hipError_t fs_box_launch(const FsBoxArgs &a, bool is_double, bool want_j, bool want_l, bool para, bool band, int lb,
                         int R, int n_wg, int nthr, size_t lds, hipStream_t st)
{
    if (n_wg <= 0) return hipSuccess;
    return is_double ? launch_t<double>(a, want_j, want_l, para, band, lb, R, n_wg, nthr, lds, st)
                     : launch_t<float>(a, want_j, want_l, para, band, lb, R, n_wg, nthr, lds, st);
}

int fs_box_occupancy(bool is_double, bool want_j, bool want_l, bool para, bool band, int lb, int R, int nthr,
                     size_t lds)
{
    return is_double ? occ_t<double>(want_j, want_l, para, band, lb, R, nthr, lds)
                     : occ_t<float>(want_j, want_l, para, band, lb, R, nthr, lds);
}

}  // namespace rt3d
