// Conversion of the weights, done once when they are loaded (Section 3.1: one set of constants per column
// of W): fp16 W [h x o] -> tiled codes and column constants, absmax (Section 2.1) and zeropoint (Eq. 1-3).
//
// W is read twice (the constants need every row of a column before its first code), the codes are written
// once: 5 bytes per weight over HBM, which is what bounds both kernels.
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
template <bool ZP>
__global__ void __launch_bounds__(256, ZP ? 2 : 4) weight_codes_kernel(const unsigned short* __restrict__ W, int h, int o,
                                                           const unsigned short* __restrict__ cw, const int4* __restrict__ zc,
                                                           int8_t* __restrict__ Wq, int KT, int JT, int steps,
                                                           int* __restrict__ psum)
{
    __shared__ u4 stage[4][512];
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
    int k = (blockIdx.y * steps * 4 + w) * 16;
    for (int it = 0; it < steps && k < k_end; it++, k += 64) {  // uniform in a wave; no barrier in the loop
        us8 v[16];
        // rows past h: the last row again, zeroed below
        if (!ragged || (k + 15 < h - 1 && h >= 16 && o >= 8)) {
            const unsigned short* p = W + jl;
#pragma unroll
            for (int i = 0; i < 16; i++) v[i] = load8_once(p + (size_t)(k + i < h ? k + i : h - 1) * o);
        } else {
#pragma unroll
            for (int i = 0; i < 16; i++)
#pragma unroll
                for (int e = 0; e < 8; e++)
                    v[i][e] = W[(size_t)(k + i < h ? k + i : h - 1) * o + (jl + e < o ? jl + e : o - 1)];
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
    }
    if constexpr (ZP) {
        // the four waves' sums meet in LDS; a workgroup stores its own, zp_colsum_kernel adds them up
        __syncthreads();
        int* s_sum = (int*)stage;
#pragma unroll
        for (int e = 0; e < 8; e++) s_sum[w * 512 + e * 64 + lane] = sum[e];
        __syncthreads();
        for (int q = threadIdx.x; q < 512; q += 256) {
            const int at = (q & 7) * 64 + (q >> 3);
            if (jb + q < o)
                psum[(size_t)blockIdx.y * o + jb + q] = s_sum[at] + s_sum[512 + at] + s_sum[1024 + at] + s_sum[1536 + at];
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

// At most n slabs of rows, of 32 rows (one pass of a workgroup over eight rows per wave) or a multiple of that
static int whole_pass_slabs(int h, int n)
{
    const int rps = ((h + n - 1) / n + 31) & ~31;
    return (h + rps - 1) / rps;
}

hipError_t launch_quantize_weight(const void* W, int h, int o, unsigned short* part, int shared, unsigned short* cw,
                                  int8_t* Wq, hipStream_t st)
{
    const int nslab = whole_pass_slabs(h, colmax_slabs(h, o));
    hipError_t e = launch_colmax_partial(W, h, o, part, nslab, true, st);
    if (e != hipSuccess) return e;
    colconst_kernel<false><<<(o + 255) / 256, 1024, 0, st>>>(part, nullptr, nslab, o, cw, nullptr);
    e = hipGetLastError();
    if (e == hipSuccess && shared) e = launch_spread_max(cw, o, st);
    if (e != hipSuccess) return e;
    // one step per workgroup: 88.7 us for the whole conversion of a 5 120 x 20 480 W, 91.8 with two, 96.1 with four
    const int KT = k_tiles(h), JT = row_tiles(o);
    weight_codes_kernel<false><<<dim3((JT + 15) / 16, KT / 2), 256, 0, st>>>((const unsigned short*)W, h, o, cw, nullptr, Wq,
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
    const int nslab = whole_pass_slabs(h, zp_colrange_slabs(h, o));
    const int rps = ((h + nslab - 1) / nslab + 31) & ~31;
    unsigned short* pmin = part;
    unsigned short* pmax = part + (size_t)nslab * o;
    zp_colrange_partial_kernel<<<dim3((o + 511) / 512, nslab), 256, 0, st>>>((const unsigned short*)W, h, o, pmin, pmax,
                                                                            rps);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    colconst_kernel<true><<<(o + 255) / 256, 1024, 0, st>>>(pmax, pmin, nslab, o, nullptr, zc);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    // a workgroup's sums take the place of the ranges of a slab in the scratch (4 bytes per column): no more of them than slabs
    const int KT = k_tiles(h), JT = row_tiles(o), most = zp_colrange_slabs(h, o);
    const int steps = (KT / 2 + most - 1) / most, ny = (KT / 2 + steps - 1) / steps;
    weight_codes_kernel<true><<<dim3((JT + 15) / 16, ny), 256, 0, st>>>((const unsigned short*)W, h, o, nullptr, zc, Wq, KT, JT,
                                                                       steps, (int*)part);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    zp_colsum_kernel<<<(o + 255) / 256, 1024, 0, st>>>((const int*)part, ny, o, zc);
    return hipGetLastError();
}

}  // namespace llmint8
