// Conversion of the weights, done once when they are loaded (Section 3.1: one set of constants per column
// of W): fp16 W [h x o] -> tiled codes and column constants, absmax (Section 2.1) and zeropoint (Eq. 1-3).
//
// The constants need every row of a column before its first code.  Where the columns of a tile fit a workgroup's
// registers W is read once (weight_strip_kernel, 3 bytes per weight over HBM), else twice (5 bytes), which bounds these kernels.
#include <mutex>

#include "common.h"

namespace llmint8 {

typedef unsigned int u4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// Column ranges over a slab of rows, for the zeropoint constants (the absmax ones come from
// colmax_partial_kernel): keys of the smallest and largest entry, as colmax_partial_kernel walks the matrix:
// one workgroup = 512 columns x rows_per_slab rows, its four waves taking every fourth row, eight rows in
// flight per lane.  A column per lane and one 2-byte load at a time took 171 us on a 5 120 x 20 480 W.
// ---------------------------------------------------------------------------
__device__ __forceinline__ us8 f16_key8(us8 v)  // f16_key() of eight values
{
    typedef short ss8 __attribute__((ext_vector_type(8)));
    const us8 sign = (us8)((ss8)v >> 15);
    return v ^ (sign | (us8)((unsigned short)0x8000));
}

__global__ void __launch_bounds__(256) zp_colrange_partial_kernel(const unsigned short* __restrict__ W, int h, int o,
                                                                  unsigned short* __restrict__ pmin,
                                                                  unsigned short* __restrict__ pmax, int rows_per_slab)
{
    __shared__ us8 red[2][4][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int c0 = blockIdx.x * 512 + lane * 8;
    const int r0 = blockIdx.y * rows_per_slab, r1 = min(h, r0 + rows_per_slab);
    us8 mn = (us8)((unsigned short)0xffff), mx = (us8)((unsigned short)0);
    scan_rows<true>(W, h, o, c0, blockIdx.x * 512 + 512 > o, r0, r1, w, [&](us8 v) {
        const us8 k = f16_key8(v);
        mn = __builtin_elementwise_min(mn, k);
        mx = __builtin_elementwise_max(mx, k);
    });
    red[0][w][lane] = mn;
    red[1][w][lane] = mx;
    __syncthreads();
    if (w < 2) {  // wave 0: minima, wave 1: maxima
        us8 m = red[w][0][lane];
#pragma unroll
        for (int q = 1; q < 4; q++)
            m = w == 0 ? __builtin_elementwise_min(m, red[0][q][lane]) : __builtin_elementwise_max(m, red[1][q][lane]);
        store8((w == 0 ? pmin : pmax) + (size_t)blockIdx.y * o, c0, o, m);
    }
}

// ---------------------------------------------------------------------------
// Slab maxima (or the keys of slab ranges) -> column constants.  256 columns x 4 groups of slabs per
// workgroup, eight loads in flight per thread (one slab after the other, one thread per column: 13.3 us on
// 52 slabs of 20 480 columns).
// ---------------------------------------------------------------------------
template <bool ZP>
__global__ void __launch_bounds__(1024) colconst_kernel(const unsigned short* __restrict__ part,
                                                        const unsigned short* __restrict__ pmin, int nslab, int cols,
                                                        unsigned short* __restrict__ cw, int4* __restrict__ zc)
{
    __shared__ unsigned short rmax[4][256], rmin[ZP ? 4 : 1][256];
    const int c = threadIdx.x & 255, g = threadIdx.x >> 8;
    const int j = blockIdx.x * 256 + c, jj = j < cols ? j : 0;
    unsigned mx = 0, mn = 0xffffu;
    for (int sl = g; sl < nslab; sl += 32) {
        unsigned short a[8], b[8];
#pragma unroll
        for (int u = 0; u < 8; u++) {  // unconditional: a slab that does not exist reads this group's first again
            const size_t at = (size_t)(sl + 4 * u < nslab ? sl + 4 * u : sl) * cols + jj;
            a[u] = part[at];
            if constexpr (ZP) b[u] = pmin[at];
        }
#pragma unroll
        for (int u = 0; u < 8; u++) {
            mx = a[u] > mx ? a[u] : mx;
            if constexpr (ZP) mn = b[u] < mn ? b[u] : mn;
        }
    }
    rmax[g][c] = (unsigned short)mx;
    if constexpr (ZP) rmin[g][c] = (unsigned short)mn;
    __syncthreads();
    if (g == 0 && j < cols) {
#pragma unroll
        for (int q = 1; q < 4; q++) {
            mx = rmax[q][c] > mx ? rmax[q][c] : mx;
            if constexpr (ZP) mn = rmin[q][c] < mn ? rmin[q][c] : mn;
        }
        if constexpr (ZP) zc[j] = make_const(mn, mx); else cw[j] = (unsigned short)mx;
    }
}

constexpr int codes_waves(bool ahead) { return ahead ? 8 : 4; }

// ---------------------------------------------------------------------------
// Codes in the tiled layout (tile rows = output columns, tile K = features), and for the zeropoint variant
// each workgroup's part of the column sums of the codes.
//
// One workgroup = 512 output columns x 64 * steps features, one wave = 512 columns x 16 features per step.  A lane
// holds 8 columns x 16 features (16 loads of 16 bytes in flight), so the 16 codes that make up a 16-byte piece
// of a tile meet in one lane and are packed in registers; LDS only swaps pieces between lanes, private to
// the wave (no barrier), so that the stores leave as 512-byte runs.  The pieces are placed at
// column ^ (lane & 7) within a lane's eight, which keeps both sides free of bank conflicts.
// Measured on 5 120 x 20 480 (105 MB of codes from 210 MB of weights): 53 us (absmax) = 5.9 TB/s and 67 us
// (zeropoint: the arithmetic in double); with the codes put into LDS byte by byte, from one 2-byte (zeropoint)
// or 16-byte load per row at a time, 178 and 219 us.  W is streamed past the caches (102 us for both passes
// together if not, 89 so); the codes are not (103 us).
// ---------------------------------------------------------------------------
// AHEAD (zeropoint): eight waves (the sums of a column's codes are kept per workgroup in the scratch that the ranges had, which
// limits how many workgroups there can be), and a wave requests the features of its next step before it codes these: two waves
// per SIMD are all that the registers allow, and neither covers the other's loads otherwise.  5 120 x 20 480 67 -> 57 us.
template <bool ZP, bool AHEAD>
__global__ void __launch_bounds__(64 * codes_waves(AHEAD), ZP ? 2 : 4) weight_codes_kernel(const unsigned short* __restrict__ W, int h, int o,
                                                           const unsigned short* __restrict__ cw, const int4* __restrict__ zc,
                                                           int8_t* __restrict__ Wq, int KT, int JT, int steps,
                                                           int* __restrict__ psum)
{
    constexpr int NW = codes_waves(AHEAD);
    __shared__ u4 stage[NW][512];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int jb = blockIdx.x * 512, j0 = jb + lane * 8;
    const bool ragged = jb + 512 > o;  // some lanes of this block hold columns that do not exist
    const int jl = j0 < o ? j0 : 0;    // they read column 0; their constants make all codes 0

    // column constants
    float kup[ZP ? 1 : 8];
    double zf[ZP ? 8 : 1];
    int z[ZP ? 8 : 1], sum[ZP ? 8 : 1];
    if constexpr (ZP) {
#pragma unroll
        for (int e = 0; e < 8; e++) {
            const int4 r = zc[j0 + e < o ? j0 + e : 0];
            zf[e] = j0 + e < o ? zp_factor(zp_range((unsigned)r.x)) : 0.0;
            z[e] = j0 + e < o ? r.y : 0;
            sum[e] = 0;
        }
    } else {
        us8 c;
#pragma unroll
        for (int e = 0; e < 8; e++) c[e] = cw[j0 + e < o ? j0 + e : 0];
#pragma unroll
        for (int e = 0; e < 8; e++) kup[e] = j0 + e < o ? code_factor(f16_bits_to_float(c[e])) : 0.0f;
    }

    u4* mine = stage[w];
    const int k_end = KT * 32;
    int k = (blockIdx.y * steps * NW + w) * 16;
    us8 v[16], ahead[AHEAD ? 16 : 1];
    // rows past h: the last row again, zeroed below
    auto load = [&](us8* to, int k) {
        if (!ragged || (k + 15 < h - 1 && h >= 16 && o >= 8)) {
            const unsigned short* p = W + jl;
#pragma unroll
            for (int i = 0; i < 16; i++) to[i] = load8_once(p + (size_t)(k + i < h ? k + i : h - 1) * o);
        } else {
#pragma unroll
            for (int i = 0; i < 16; i++)
#pragma unroll
                for (int e = 0; e < 8; e++)
                    to[i][e] = W[(size_t)(k + i < h ? k + i : h - 1) * o + (jl + e < o ? jl + e : o - 1)];
        }
    };
    if (AHEAD && k < k_end) load(v, k);
    for (int it = 0; it < steps && k < k_end; it++, k += 16 * NW) {  // uniform in a wave; no barrier in the loop
        if constexpr (AHEAD) {
            if (it + 1 < steps && k + 16 * NW < k_end) load(ahead, k + 16 * NW);
        } else {
            load(v, k);
        }
        if (k + 16 > h) {
#pragma unroll
            for (int i = 0; i < 16; i++)
                if (k + i >= h) v[i] = (us8)((unsigned short)0);
        }
#pragma unroll
        for (int e = 0; e < 8; e++) {
            unsigned q[4];
#pragma unroll
            for (int b = 0; b < 4; b++) {
                unsigned t[4];
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    if constexpr (ZP) t[i] = zp_u_bits(v[4 * b + i][e], zf[e]) - (unsigned)z[e];
                    else t[i] = code_bits(v[4 * b + i][e], kup[e]);
                }
                q[b] = pack_low_bytes(t[0], t[1], t[2], t[3]);
            }
            if constexpr (ZP) {
                if (k + 16 > h) {  // a padding row's u(0) = 0 is not its code: padding is 0 whatever the zeropoint
#pragma unroll
                    for (int b = 0; b < 4; b++)
#pragma unroll
                        for (int i = 0; i < 4; i++)
                            if (k + 4 * b + i >= h) q[b] &= ~(0xffu << (8 * i));
                }
#pragma unroll
                for (int b = 0; b < 4; b++) sum[e] = __builtin_amdgcn_sdot4((int)q[b], 0x01010101, sum[e], false);
            }
            mine[lane * 8 + (e ^ (lane & 7))] = u4{q[0], q[1], q[2], q[3]};
        }
        // read back by other lanes of the same wave only: LDS serves a wave's requests in order, the compiler
        // just must not reorder them
        asm volatile("" ::: "memory");
        int8_t* out = Wq + ((size_t)(blockIdx.x * 16) * KT + (k >> 5)) * TILE_BYTES + ((k >> 4) & 1) * 512 + (lane & 31) * 16;
#pragma unroll
        for (int i = 0; i < 8; i++) {
            const int c = i * 64 + lane;  // column of the block
            const u4 piece = mine[(c & ~7) + ((c & 7) ^ ((c >> 3) & 7))];
            const int jt = 2 * i + (lane >> 5);
            if (blockIdx.x * 16 + jt < JT) *(u4*)(out + (size_t)jt * KT * TILE_BYTES) = piece;
        }
        asm volatile("" ::: "memory");  // the next step's pieces stay behind these reads
        if constexpr (AHEAD) {
#pragma unroll
            for (int i = 0; i < 16; i++) v[i] = ahead[i];
        }
    }
    if constexpr (ZP) {
        // the waves' sums meet in LDS; a workgroup stores its own, zp_colsum_kernel adds them up
        __syncthreads();
        int* s_sum = (int*)stage;
#pragma unroll
        for (int e = 0; e < 8; e++) s_sum[w * 512 + e * 64 + lane] = sum[e];
        __syncthreads();
        for (int q = threadIdx.x; q < 512; q += 64 * NW) {
            int t = 0;
#pragma unroll
            for (int x = 0; x < NW; x++) t += s_sum[x * 512 + (q & 7) * 64 + (q >> 3)];
            if (jb + q < o) psum[(size_t)blockIdx.y * o + jb + q] = t;
        }
    }
}

// Column sums of the codes into the records.  (Added there by weight_codes_kernel with one global addition per column
// and workgroup, 40 to a record, that kernel took 110 us instead of 68 on a 5 120 x 20 480 W.)
__global__ void __launch_bounds__(1024) zp_colsum_kernel(const int* __restrict__ psum, int n, int o, int4* __restrict__ zc)
{
    __shared__ int red[4][256];
    const int c = threadIdx.x & 255, g = threadIdx.x >> 8;
    const int j = blockIdx.x * 256 + c, jj = j < o ? j : 0;
    int t = 0;
    for (int b = g; b < n; b += 32) {
        int v[8];
#pragma unroll
        for (int u = 0; u < 8; u++) v[u] = psum[(size_t)(b + 4 * u < n ? b + 4 * u : b) * o + jj];
#pragma unroll
        for (int u = 0; u < 8; u++) t += b + 4 * u < n ? v[u] : 0;
    }
    red[g][c] = t;
    __syncthreads();
    if (g == 0 && j < o) zc[j].z = red[0][c] + red[1][c] + red[2][c] + red[3][c];
}

// ---------------------------------------------------------------------------
// The whole conversion of 32 output columns (one row tile of the codes) in one workgroup, W read once: the columns stay
// in registers between their constants and their codes, so 3 bytes per weight move instead of 5.
//
// A lane holds 8 columns x 16 features per unit (16 loads of 16 bytes; four lanes side by side cover the 64 bytes that
// the tile has in a row), a wave 256 features, so that the 16 codes of a 16-byte piece meet in one lane as in
// weight_codes_kernel; wave w of the nw takes the units w, w + nw, ... (U of them).  What fits in registers is 16 waves
// of one unit, 12 of two (absmax, above 2 048 features: 150 registers) or 8 of three (zeropoint, above 4 096: 253), up to 6 144
// features in all; LDS swaps pieces between lanes, 8 KiB to a wave.
// Two tiles side by side share the 128-byte lines of W, and rows of 4 096 bytes or a multiple send all of a tile to one
// L2 channel: each XCD takes a run of tiles side by side (neighbours alternating between the XCDs: 100.7 us instead of 85.1 on
// 5 120 x 20 480).  What bounds it: the memory while all workgroups load; loading, coding and storing follow one
// another in a workgroup.  Against the two passes, W from memory, us:
// 5 120 x 20 480 82.5 / 88.5, 4 096 x 8 192 28.1 / 33.0, 2 048 x 49 152 67.2 / 85.4; zeropoint 30.5 / 44.0 and 74.3 / 98.3 on the latter two.
// ---------------------------------------------------------------------------
constexpr int STRIP_WAVES = 16, STRIP_STAGE = 512 * 16;
constexpr int strip_max_waves(int units) { return units == 1 ? 16 : units == 2 ? 12 : 8; }

template <int U, bool ZP>
__global__ void __launch_bounds__(64 * strip_max_waves(U))
    weight_strip_kernel(const unsigned short* __restrict__ W, int h, int o, unsigned short* __restrict__ cw,
                        int4* __restrict__ zc, int8_t* __restrict__ Wq, int KT, int JT)
{
    extern __shared__ u4 stage[];  // 512 pieces for each wave
    __shared__ us8 rmax[STRIP_WAVES][4], rmin[ZP ? STRIP_WAVES : 1][4];
    __shared__ float s_kup[32];
    __shared__ double s_zf[ZP ? 32 : 1];
    __shared__ int s_z[ZP ? 32 : 1], s_sum[ZP ? STRIP_WAVES : 1][32];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
    const int b = blockIdx.x;
    const int jt = (b & 7) * (JT >> 3) + min(b & 7, JT & 7) + (b >> 3);
    const int oct = (lane & 3) * 8, j0 = jt * 32 + oct, g16 = (lane >> 2) * 16;
    const unsigned short* p = W + (j0 + 8 <= o ? j0 : o - 8);  // (chunk_fix() below moves the row's last columns into place)
    us8 v[U][16];
#pragma unroll
    for (int u = 0; u < U; u++) {
        const int k0 = (u * nw + w) * 256;
        if (k0 + 256 <= h) {
            const unsigned short* q = p + (size_t)(k0 + g16) * o;
#pragma unroll
            for (int i = 0; i < 16; i++) v[u][i] = load8(q + (size_t)i * o);
        } else {  // rows past h: the last row again, which changes no extreme; zeroed below
#pragma unroll
            for (int i = 0; i < 16; i++) v[u][i] = load8(p + (size_t)(k0 + g16 + i < h ? k0 + g16 + i : h - 1) * o);
        }
    }
    if (jt * 32 + 32 > o) {  // uniform
#pragma unroll
        for (int u = 0; u < U; u++)
#pragma unroll
            for (int i = 0; i < 16; i++) v[u][i] = chunk_fix(v[u][i], j0, o);  // columns that do not exist: all zero
    }
    // ---- the columns' extremes
    us8 mx = (us8)((unsigned short)0), mn = (us8)((unsigned short)0xffff);
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
        for (int i = 0; i < 16; i++) {
            if constexpr (ZP) {
                const us8 k = f16_key8(v[u][i]);
                mn = __builtin_elementwise_min(mn, k);
                mx = __builtin_elementwise_max(mx, k);
            } else {
                mx = __builtin_elementwise_max(mx, v[u][i] & (unsigned short)0x7fff);
            }
        }
#pragma unroll
    for (int d = 4; d <= 32; d <<= 1) {
        u4 a = __builtin_bit_cast(u4, mx), c = __builtin_bit_cast(u4, mn);
#pragma unroll
        for (int q = 0; q < 4; q++) {
            a[q] = (unsigned)__shfl_xor((int)a[q], d);
            if constexpr (ZP) c[q] = (unsigned)__shfl_xor((int)c[q], d);
        }
        mx = __builtin_elementwise_max(mx, __builtin_bit_cast(us8, a));
        if constexpr (ZP) mn = __builtin_elementwise_min(mn, __builtin_bit_cast(us8, c));
    }
    if (lane < 4) {
        rmax[w][lane] = mx;
        if constexpr (ZP) rmin[w][lane] = mn;
    }
    __syncthreads();
    if (tid < 32) {
        unsigned kx = 0, kn = 0xffffu;
        for (int q = 0; q < nw; q++) {
            const unsigned x = rmax[q][tid >> 3][tid & 7];
            kx = x > kx ? x : kx;
            if constexpr (ZP) {
                const unsigned n = rmin[q][tid >> 3][tid & 7];
                kn = n < kn ? n : kn;
            }
        }
        const int j = jt * 32 + tid;
        if constexpr (ZP) {
            const int4 r = make_const(kn, kx);
            if (j < o) {
                zc[j].x = r.x;
                zc[j].y = r.y;
                zc[j].w = 0;
            }
            s_zf[tid] = zp_factor(zp_range((unsigned)r.x));
            s_z[tid] = r.y;
        } else {
            if (j < o) cw[j] = (unsigned short)kx;
            s_kup[tid] = code_factor(f16_bits_to_float((unsigned short)kx));
        }
    }
    __syncthreads();
    // ---- codes
    u4* mine = stage + w * 512;
    int sum[ZP ? 8 : 1];
    if constexpr (ZP) {
#pragma unroll
        for (int e = 0; e < 8; e++) sum[e] = 0;
    }
#pragma unroll
    for (int u = 0; u < U; u++) {
        const int unit = u * nw + w, k = unit * 256 + g16;
        if (unit * 8 >= KT) break;  // uniform in a wave
        if (k + 16 > h) {
#pragma unroll
            for (int i = 0; i < 16; i++)
                if (k + i >= h) v[u][i] = (us8)((unsigned short)0);
        }
#pragma unroll
        for (int e = 0; e < 8; e++) {
            const float f = ZP ? 0.0f : s_kup[oct + e];
            const double zf = ZP ? s_zf[oct + e] : 0.0;
            const unsigned z = ZP ? (unsigned)s_z[oct + e] : 0u;
            unsigned q[4];
#pragma unroll
            for (int c = 0; c < 4; c++) {
                unsigned t[4];
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    if constexpr (ZP) t[i] = zp_u_bits(v[u][4 * c + i][e], zf) - z;
                    else t[i] = code_bits(v[u][4 * c + i][e], f);
                }
                q[c] = pack_low_bytes(t[0], t[1], t[2], t[3]);
            }
            if constexpr (ZP) {
                if (k + 16 > h) {  // a padding row's u(0) - zp is not its code: padding is 0 whatever the zeropoint
#pragma unroll
                    for (int c = 0; c < 4; c++)
#pragma unroll
                        for (int i = 0; i < 4; i++)
                            if (k + 4 * c + i >= h) q[c] &= ~(0xffu << (8 * i));
                }
#pragma unroll
                for (int c = 0; c < 4; c++) sum[e] = __builtin_amdgcn_sdot4((int)q[c], 0x01010101, sum[e], false);
            }
            mine[lane * 8 + (e ^ (lane & 7))] = u4{q[0], q[1], q[2], q[3]};
        }
        // (wave-private, as in weight_codes_kernel)
        asm volatile("" ::: "memory");
        int8_t* out = Wq + ((size_t)jt * KT + unit * 8) * TILE_BYTES;
#pragma unroll
        for (int i = 0; i < 8; i++) {
            const int c = i * 64 + lane;  // piece of the unit, in the order of the tiles
            const u4 piece = mine[(c & ~7) + ((c & 7) ^ ((c >> 3) & 7))];
            if (unit * 8 + i < KT) *(u4*)(out + (size_t)c * 16) = piece;
        }
        asm volatile("" ::: "memory");
    }
    if constexpr (ZP) {
#pragma unroll
        for (int d = 4; d <= 32; d <<= 1)
#pragma unroll
            for (int e = 0; e < 8; e++) sum[e] += __shfl_xor(sum[e], d);
        if (lane < 4) {
#pragma unroll
            for (int e = 0; e < 8; e++) s_sum[w][oct + e] = sum[e];
        }
        __syncthreads();
        if (tid < 32 && jt * 32 + tid < o) {
            int t = 0;
            for (int q = 0; q < nw; q++) t += s_sum[q][tid];
            zc[jt * 32 + tid].z = t;
        }
    }
}

// Waves of a workgroup of weight_strip_kernel and units per wave; 0: the kernels that read W twice take the call.
// Where the line lies was measured with W from memory (copies of W in turn; strips / two passes, us).
// At most one strip to a compute unit: a unit takes its strip in at 20 to 30 GB/s and then codes it, however few strips
// there are, while two passes spread over all units.  So tall strips need many of them: 5 120 x 2 048 26.4 / 18.2, x 4 096
// 28.2 / 22.5, x 6 144 32.3 / 31.7, x 7 168 33.8 / 36.7 (zeropoint 35.9 / 25.7, 38.1 / 32.9, 39.7 / 39.7, 40.7 / 51.6); 3 072 x 2 048
// 13.2 / 14.3, x 3 072 1.15 times the two passes.  That holds for rows of whole KiB (o a multiple of 512), which the two passes read in whole
// blocks of 512 columns and which crowd a strip's loads on few memory channels.  With others strips are ahead (5 120 x 5 000 0.65
// times the two passes, zeropoint 0.77) down to few of them, where it depends on how much of the last block of 512 columns
// the two passes do for nothing (5 467 x 1 608 1.17, x 1 928 0.95, x 560 1.17, x 1 000 0.86; zeropoint 1.22, 1.03, 1.19, 0.94):
// there the line is within 10 % of the faster one, elsewhere within 5 %.
// More strips than units, up to 2 048 features, where a unit holds two workgroups: strips, but where the share of 1 or 2
// to a unit is most uneven and the rows are whole KiB (2 048 x 9 216 24.0 / 23.3, x 10 240 25.1 / 23.5, x 12 288 24.8 / 24.9; zeropoint 24.8 / 30.9).
// Above, the time is that of whole rounds of the units (absmax, 5 120 features: 28.3 us a round, the two passes 0.139 us per strip), which have to be
// four fifths full; that up to 3 072 features two workgroups fit (absmax: 150 registers, 6 waves) changes little (2 560 x 10 240
// 31.8 / 28.0, x 12 288 31.2 / 31.1, x 14 336 32.7 / 35.5).  Zeropoint there: only where all strips are one round (5 120 x 20 480,
// where the codes take longer, 108.9 / 106.1).
static int strip_waves(int h, int o, bool zeropoint, int cus, int* units)
{
    const int n = (h + 255) / 256, JT = row_tiles(o);
    *units = n <= 8 || (zeropoint && n <= strip_max_waves(1)) ? 1 : zeropoint ? 3 : 2;
    const int nw = (n + *units - 1) / *units;
    if (o < 8 || nw > strip_max_waves(*units)) return 0;
    const bool kib_rows = o % 512 == 0;
    bool take = true;
    if (JT <= cus) {  // (lines in sixteenths of the compute units)
        if (kib_rows) {
            const int least = zeropoint ? (n > 20 ? 11 : n > 16 ? 13 : n > 12 ? 9 : 0) : n > 12 || n == 10 ? 13 : n > 10 ? 11 : 0;
            take = 16 * JT >= least * cus || (!zeropoint && n <= 12 && 4 * JT <= cus);
        } else if (n > (zeropoint ? 16 : 14)) {
            const int many = zeropoint ? 6 : n > 20 ? 5 : 2, few = zeropoint ? 1 : 0;
            take = 16 * JT >= many * cus || (16 * JT > few * cus && o % 512 >= 288);
        }
    } else if (n <= 8) {
        take = zeropoint || !kib_rows || n < 7 || 16l * JT >= 21l * cus;
    } else {
        take = !zeropoint && 5l * JT >= 4l * ((JT + cus - 1) / cus) * cus;
    }
    return take ? nw : 0;
}

template <int U, bool ZP>
static hipError_t launch_weight_strip(const void* W, int h, int o, unsigned short* cw, int4* zc, int8_t* Wq, int nw, hipStream_t st)
{
    const int JT = row_tiles(o);
    weight_strip_kernel<U, ZP><<<JT, nw * 64, nw * STRIP_STAGE, st>>>((const unsigned short*)W, h, o, cw, zc, Wq, k_tiles(h), JT);
    return hipGetLastError();
}

// Once per device, for the conversions: the dynamic LDS of weight_strip_kernel's instantiations and the compute units (as
// prefill_device_setup(), which calls this, does it for the tiled kernel: a program that only converts need not wait for
// its 36 instantiations, 2 ms in all).
hipError_t weights_device_setup(int* cus)
{
    constexpr int MAX_DEVICES = 64;
    static std::atomic<int> done[MAX_DEVICES];  // 0: not set up yet; else the device's compute units
    static std::mutex lock;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const bool cached = dev >= 0 && dev < MAX_DEVICES;
    if (cached && (*cus = done[dev].load(std::memory_order_acquire)) > 0) return hipSuccess;
    std::lock_guard<std::mutex> hold(lock);
    const void* k[4] = {(const void*)weight_strip_kernel<1, false>, (const void*)weight_strip_kernel<1, true>,
                        (const void*)weight_strip_kernel<2, false>, (const void*)weight_strip_kernel<3, true>};
    const int waves[4] = {strip_max_waves(1), strip_max_waves(1), strip_max_waves(2), strip_max_waves(3)};
    for (int i = 0; i < 4; i++)
        if ((e = hipFuncSetAttribute(k[i], hipFuncAttributeMaxDynamicSharedMemorySize, waves[i] * STRIP_STAGE)) != hipSuccess) return e;
    if (hipDeviceGetAttribute(cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || *cus < 1) *cus = 256;
    if (cached) done[dev].store(*cus, std::memory_order_release);
    return hipSuccess;
}

// how often a conversion reads W
int weight_reads(int h, int o, bool zeropoint)
{
    int units, cus = 256;
    if (weights_device_setup(&cus) != hipSuccess) cus = 256;
    return strip_waves(h, o, zeropoint, cus, &units) ? 1 : 2;
}

// At most n slabs of rows, of 32 rows (one pass of a workgroup over eight rows per wave) or a multiple of that
static int whole_pass_slabs(int h, int n)
{
    const int rps = ((h + n - 1) / n + 31) & ~31;
    return (h + rps - 1) / rps;
}

hipError_t launch_quantize_weight(const void* W, int h, int o, unsigned short* part, int shared, unsigned short* cw,
                                  int8_t* Wq, hipStream_t st)
{
    int units, cus;
    hipError_t e = weights_device_setup(&cus);
    if (e != hipSuccess) return e;
    if (const int nw = shared ? 0 : strip_waves(h, o, false, cus, &units))
        return units == 1 ? launch_weight_strip<1, false>(W, h, o, cw, nullptr, Wq, nw, st)
                          : launch_weight_strip<2, false>(W, h, o, cw, nullptr, Wq, nw, st);
    const int nslab = whole_pass_slabs(h, colmax_slabs(h, o));
    e = launch_colmax_partial(W, h, o, part, nslab, true, st);
    if (e != hipSuccess) return e;
    colconst_kernel<false><<<(o + 255) / 256, 1024, 0, st>>>(part, nullptr, nslab, o, cw, nullptr);
    e = hipGetLastError();
    if (e == hipSuccess && shared) e = launch_spread_max(cw, o, st);
    if (e != hipSuccess) return e;
    // one step per workgroup: 88.7 us for the whole conversion of a 5 120 x 20 480 W, 91.8 with two, 96.1 with four
    const int KT = k_tiles(h), JT = row_tiles(o);
    weight_codes_kernel<false, false><<<dim3((JT + 15) / 16, KT / 2), 256, 0, st>>>((const unsigned short*)W, h, o, cw, nullptr, Wq,
                                                                            KT, JT, 1, nullptr);
    return hipGetLastError();
}

int zp_colrange_slabs(int h, int o)
{
    const int colblocks = (o + 255) / 256;
    int n = (2048 + colblocks - 1) / colblocks;
    const int maxslab = (h + 31) / 32;
    if (n > maxslab) n = maxslab;
    if (n > 64) n = 64;
    return n < 1 ? 1 : n;
}

hipError_t launch_zp_quantize_weight(const void* W, int h, int o, int8_t* Wq, int4* zc, unsigned short* part,
                                     hipStream_t st)
{
    int units, cus;
    hipError_t e = weights_device_setup(&cus);
    if (e != hipSuccess) return e;
    if (const int nw = strip_waves(h, o, true, cus, &units))
        return units == 1 ? launch_weight_strip<1, true>(W, h, o, nullptr, zc, Wq, nw, st)
                          : launch_weight_strip<3, true>(W, h, o, nullptr, zc, Wq, nw, st);
    const int nslab = whole_pass_slabs(h, zp_colrange_slabs(h, o));
    const int rps = ((h + nslab - 1) / nslab + 31) & ~31;
    unsigned short* pmin = part;
    unsigned short* pmax = part + (size_t)nslab * o;
    zp_colrange_partial_kernel<<<dim3((o + 511) / 512, nslab), 256, 0, st>>>((const unsigned short*)W, h, o, pmin, pmax,
                                                                            rps);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    colconst_kernel<true><<<(o + 255) / 256, 1024, 0, st>>>(pmax, pmin, nslab, o, nullptr, zc);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    // a workgroup's sums take the place of the ranges of a slab in the scratch (4 bytes per column): no more of them than slabs
    const int KT = k_tiles(h), JT = row_tiles(o), most = zp_colrange_slabs(h, o), nx = (JT + 15) / 16;
    // With the next step requested ahead, steps of 16 features per wave so that rounds of the compute units (one workgroup
    // each) times steps are as few as can be.  Us, so / four waves and no request ahead: 5 120 x 20 480 96.5 / 105.2, 10 000 x
    // 10 240 98.0 / 105.3, 8 486 x 2 944 36.8 / 46.1, 9 216 x 9 216 84.3 / 85.6, 21 632 x 2 392 66.7 / 75.4, 49 152 x 2 048 91.9 / 93.9; but
    // 12 288 x 8 192 101.9 / 95.1, x 4 096 54.0 / 52.7, x 1 000 34.4 / 32.4, 16 264 x 3 584 63.3 / 62.0 (12 288 x 8 200 104.8 / 109.1),
    // and where less than half of the compute units would have a workgroup.  (Between 10 240 and 20 480 features the loop without the request
    // stays for the sizes that lose; 12 288 x 8 192 against x 8 200 says that the pitch of W's rows has a part in it, what part is not known.)
    constexpr int nw = codes_waves(true);
    int steps = 0, ny = 0;
    long least = 0;
    for (int n = 1; n <= 64 || !steps; n++) {
        const int y = (2 * KT + n * nw - 1) / (n * nw);
        if (y > most) continue;
        const long cost = (long)((nx * y + cus - 1) / cus) * (n + 1);
        if (!steps || cost < least) { least = cost; steps = n; ny = y; }
    }
    const bool ahead = (h <= 10240 || h > 20480) && 2 * nx * ny >= cus;
    if (!ahead) {
        steps = (KT / 2 + most - 1) / most;
        ny = (KT / 2 + steps - 1) / steps;
    }
    if (ahead)
        weight_codes_kernel<true, true><<<dim3(nx, ny), 64 * nw, 0, st>>>((const unsigned short*)W, h, o, nullptr, zc, Wq, KT, JT,
                                                                          steps, (int*)part);
    else
        weight_codes_kernel<true, false><<<dim3(nx, ny), 256, 0, st>>>((const unsigned short*)W, h, o, nullptr, zc, Wq, KT, JT,
                                                                       steps, (int*)part);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    zp_colsum_kernel<<<(o + 255) / 256, 1024, 0, st>>>((const int*)part, ny, o, zc);
    return hipGetLastError();
}

}  // namespace llmint8
