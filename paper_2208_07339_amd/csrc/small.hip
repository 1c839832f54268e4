// A whole call in one kernel, for a few tokens of few features (s * h up to 32 768): outlier scan, row constants,
// codes (Section 3.2, 2.1, 3.1) and the product (Eq. 7 + Eq. 8).
#include <type_traits>

#include "common.h"

namespace llmint8 {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef unsigned int u2 __attribute__((ext_vector_type(2)));
typedef unsigned short us2 __attribute__((ext_vector_type(2)));

#define FENCE() __builtin_amdgcn_sched_barrier(0)

// ---------------------------------------------------------------------------
// What bounds such a call is not the pre-pass's work but its launches: three kernels of 4.5 us each for 0.2 MB
// (8 x 256 x 512), 10 us in front of a 15 us weight stream (1 x 5120 x 20480).  So there is one launch, and every
// workgroup makes the codes of X for itself: X is at most 64 KiB, comes from L2, and the first two batches of the
// workgroup's weights travel meanwhile.
//
// One workgroup = 4 waves, one tile of 32 output columns, K split over the waves, as in gemm_decode_kernel; the
// codes of X are read from LDS instead of memory, which leaves registers for three workgroups per compute unit.
// Row r of X belongs to 256 / sp threads (sp: s rounded up to a power of two), each holding XC chunks of 8
// features in registers from the first load to the codes.  A column is an outlier when any of its entries says
// so: those entries set bits of a bitmap in LDS, whose population counts place the columns in order.
//
// Outputs are those of the separate calls bit for bit.  Where llmint8_matmul takes the tiled kernel for these sizes, the
// outlier product therefore comes from the matrix unit, as there.
//
// Every workgroup also writes its share of the codes; workgroup 0 writes idx, count, status, c_x and Xo.
// ---------------------------------------------------------------------------
struct SmallArgs {
    const unsigned short* X;
    int s, h, o, KT, lg_tpr;  // lg_tpr: log2 of the threads per row
    unsigned thr;
    const int8_t* Wq;
    const unsigned short* cw;
    const unsigned short* Wf;  // [h x o] fp16 weights, or NULL: outlier rows rebuilt from the codes
    int32_t* idx;
    int cap, opad;
    int32_t* count;
    int32_t* status;
    int8_t* Xq;
    unsigned short* cx;
    unsigned short* Xo;
    _Float16* Out;
    int tiled_order;  // llmint8_matmul takes the tiled kernel for these sizes: add up in its order
};

constexpr int SSLOTS = 32;  // outlier slots whose operands are fetched before the weight stream goes on

// T = 16 (up to 16 tokens): a workgroup has half a tile, 16 columns, and 16 x 16 x 64 MFMAs; the waves take the pairs of k-tiles
// in turn.  Twice as many workgroups reach more compute units, or share them more evenly (half_tiles() has the figures).
// Four loads to a batch leave registers for five workgroups per compute unit up to 4 chunks (with eight, four of them and 640
// column tiles in two rounds: 1 x 5120 x 20480 21 us instead of 17); at 8 chunks long sums want eight (2 x 8192 x 11000 16.2 / 17.6).
template <int XC, int T>
__global__ void __launch_bounds__(256, XC <= 4 ? (T == 16 ? 5 : 4) : 3) linear_small_kernel(const SmallArgs a)
{
    constexpr int U = T == 16 && XC != 8 ? 4 : 8;  // loads per batch: k-tiles, or halves of pairs of them
    constexpr int NG = 256 / T, NQ = T * T / 64;  // threads per column, accumulators per lane
    typedef std::conditional_t<T == 16, v4i, v16i> acc_t;
    extern __shared__ __attribute__((aligned(16))) int8_t xq[];  // codes [KT][2][sp][16], then 16 zero bytes
    __shared__ int red[4][NQ][64];
    __shared__ unsigned bitmap[XC * 64];       // outlier columns, 32 per word
    __shared__ int s_idx[JOB_MAX_CAP];
    __shared__ unsigned s_row[32];             // row constants, fp16 bits
    __shared__ int s_wsum[4];
    __shared__ unsigned short s_xo[SSLOTS][32], s_wo[SSLOTS][32];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int s = a.s, h = a.h, o = a.o, KT = a.KT;
    const int lg = a.lg_tpr, tpr = 1 << lg, sp = 256 >> lg;
    const int r = tid >> lg, g = tid & (tpr - 1);  // this thread's row, its first chunk
    const unsigned short* row = a.X + (size_t)(r < s ? r : 0) * h;

    // ---- X first, then the weights: loads are waited for in the order of issue
    us8 v[XC];
#pragma unroll
    for (int m = 0; m < XC; m++) {
        const int c = g + (m << lg);
        v[m] = load8(row + (8 * c + 8 <= h ? 8 * c : 0));  // h >= 8; what does not exist is replaced below
    }
    const int jj = tid & (T - 1), ig = tid / T;
    const int jt = T == 16 ? blockIdx.x >> 1 : blockIdx.x, jr = (T == 16 ? (blockIdx.x & 1) * 16 : 0) + jj, j = jt * 32 + jr;
    const unsigned short cwb = a.cw[j < o ? j : 0];
    const int kq = T == 16 ? (KT / 2 - w + 3) >> 2 : KT / 4;  // this wave's loads (KT is a multiple of 4)
    const v4i* wp = T == 16 ? (const v4i*)(a.Wq + ((size_t)jt * KT + 2 * w) * TILE_BYTES) + (blockIdx.x & 1) * 16 + (lane >> 4) * 32 + (lane & 15)
                            : (const v4i*)(a.Wq + ((size_t)jt * KT + (size_t)w * kq) * TILE_BYTES) + lane;
    if (T == 16 && kq == 0) wp -= 2 * w * 64;  // (no pair for this wave: the first one, not used)
    v4i wv[2][U];
    auto load = [&](int B, int kt) {
#pragma unroll
        for (int u = 0; u < U; u++)
            wv[B][u] = __builtin_nontemporal_load(wp + (size_t)(kt + u < kq ? kt + u : T == 16 ? max(0, kq - 1) : kq - 1) * (T == 16 ? 512 : 64));
    };
    FENCE();
    load(0, 0);
    if (XC <= 8) load(1, U);  // 16 chunks of X take its registers
    FENCE();

    // ---- outlier columns
    for (int q = tid; q < XC * 64; q += 256) bitmap[q] = 0;
    if (tid < 32) s_row[tid] = 0;
    if (tid < 4) ((int*)(xq + sp * KT * 32))[tid] = 0;
    __syncthreads();
    if (h & 7) {
#pragma unroll
        for (int m = 0; m < XC; m++) {
            const int c = g + (m << lg);
            if (8 * c < h && 8 * c + 8 > h)
#pragma unroll
                for (int e = 0; e < 8; e++) v[m][e] = 8 * c + e < h ? row[8 * c + e] : (unsigned short)0;
        }
    }
#pragma unroll
    for (int m = 0; m < XC; m++) {
        const int c = g + (m << lg);
        if (r >= s || 8 * c >= h) v[m] = (us8)(0);
        unsigned f = 0;
        const us8 mag = v[m] & (unsigned short)0x7fff;
        const us2 a2 = __builtin_elementwise_max(__builtin_elementwise_max(mag.s01, mag.s23),
                                                 __builtin_elementwise_max(mag.s45, mag.s67));
        if ((a2.x > a2.y ? a2.x : a2.y) >= a.thr && r < s) {
#pragma unroll
            for (int e = 0; e < 8; e++)
                if (8 * c + e < h && (unsigned)mag[e] >= a.thr) f |= 1u << e;
        }
        if (f) atomicOr(&bitmap[c >> 2], f << (8 * (c & 3)));
    }
    __syncthreads();
    // positions of the columns: a thread has the words 4 tid .. 4 tid + 3
    int cnt;
    {
        unsigned b[4];
        int n = 0;
#pragma unroll
        for (int q = 0; q < 4; q++) {
            b[q] = 4 * tid + q < XC * 64 ? bitmap[4 * tid + q] : 0u;
            n += __popc(b[q]);
        }
        int incl = n;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int t = __shfl_up(incl, d);
            if (lane >= d) incl += t;
        }
        if (lane == 63) s_wsum[w] = incl;
        __syncthreads();
        int pos = incl - n, total = 0;
#pragma unroll
        for (int q = 0; q < 4; q++) {
            if (q < w) pos += s_wsum[q];
            total += s_wsum[q];
        }
        cnt = total < a.cap ? total : a.cap;
        if (n) {
#pragma unroll
            for (int q = 0; q < 4; q++) {
                unsigned left = b[q];
                while (left) {
                    const int bit = __ffs((int)left) - 1;
                    left &= left - 1;
                    if (pos < cnt) s_idx[pos] = 32 * (4 * tid + q) + bit;
                    else b[q] &= ~(1u << bit);  // more columns than the buffer takes: ordinary ones from here on
                    pos++;
                }
                if (total > cnt) bitmap[4 * tid + q] = b[q];
            }
        }
        if (blockIdx.x == 0 && tid == 0) {
            *a.count = cnt;
            if (a.status) *a.status = total > a.cap ? 1 : 0;
        }
    }
    __syncthreads();

    // ---- this workgroup's outlier operands: slots ig, ig + NG, .. of column jj, and of the tokens
    unsigned short wo[SSLOTS / NG], xo[SSLOTS / NG];
#pragma unroll
    for (int q = 0; q < SSLOTS / NG; q++) {
        const int t = ig + NG * q;
        wo[q] = xo[q] = 0;
        if (t < cnt) {
            const int k = s_idx[t];
            xo[q] = a.X[(size_t)(jj < s ? jj : 0) * h + k];
            if (a.Wf)
                wo[q] = a.Wf[(size_t)k * o + (j < o ? j : 0)];
            else
                wo[q] = (unsigned char)a.Wq[((size_t)jt * KT + (k >> 5)) * TILE_BYTES + tile_byte(jr, k & 31)];
        }
    }

    // ---- row constants and codes
    us8 mx = (us8)(0);
    unsigned bits[XC];
#pragma unroll
    for (int m = 0; m < XC; m++) {
        const int c = g + (m << lg);
        bits[m] = c < 4 * KT ? (bitmap[c >> 2] >> (8 * (c & 3))) & 0xffu : 0u;
        if (bits[m]) {
#pragma unroll
            for (int e = 0; e < 8; e++)
                if ((bits[m] >> e) & 1u) v[m][e] = 0;
        }
        mx = __builtin_elementwise_max(mx, v[m] & (unsigned short)0x7fff);
    }
    {
        const us2 a2 = __builtin_elementwise_max(__builtin_elementwise_max(mx.s01, mx.s23),
                                                 __builtin_elementwise_max(mx.s45, mx.s67));
        unsigned m1 = a2.x > a2.y ? a2.x : a2.y;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1)
            if (d < tpr) {
                const unsigned t = (unsigned)__shfl_xor((int)m1, d);
                m1 = t > m1 ? t : m1;
            }
        if ((g & 63) == 0) atomicMax(&s_row[r], m1);
    }
    __syncthreads();
    {
        const float f = code_factor(f16_bits_to_float((unsigned short)s_row[r]));
#pragma unroll
        for (int m = 0; m < XC; m++) {
            const int c = g + (m << lg);
            unsigned t[8];
#pragma unroll
            for (int e = 0; e < 8; e++) t[e] = code_bits(v[m][e], f);
            const u2 pk = {pack_low_bytes(t[0], t[1], t[2], t[3]), pack_low_bytes(t[4], t[5], t[6], t[7])};
            if (c < 4 * KT) *(u2*)(xq + (((c >> 1) * sp + r) * 16 + (c & 1) * 8)) = pk;
        }
    }
    __syncthreads();
    const int lr = lane & (T - 1);
    const int8_t* xb = lr < sp ? xq + ((lane / T) * sp + lr) * 16 : xq + sp * KT * 32;
    const int xstep = lr < sp ? (T == 16 ? 256 : 32) * sp : 0;  // from one load of this wave to the next

    // ---- the stream goes on
    if (XC > 8) load(1, U);
    acc_t acc;
#pragma unroll
    for (int q = 0; q < NQ; q++) acc[q] = 0;
    const int8_t* xw = T == 16 ? (lr < sp ? xb + w * 64 * sp : xb) : xb + w * kq * xstep;
    auto mfma = [&](v4i p, v4i x) {
        if constexpr (T == 16) acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(p, x, acc, 0, 0, 0);
        else acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(p, x, acc, 0, 0, 0);
    };
    auto mm = [&](int B, int kt) {
        v4i x[U];
#pragma unroll
        for (int u = 0; u < U; u++) x[u] = *(const v4i*)(xw + (kt + u) * xstep);
#pragma unroll
        for (int u = 0; u < U; u++) mfma(wv[B][u], x[u]);
    };
    auto mm_rest = [&](int B, int kt) {
#pragma unroll
        for (int u = 0; u < U; u++)
            if (kt + u < kq) mfma(wv[B][u], *(const v4i*)(xw + (kt + u) * xstep));
    };
    int kt = 0;
    for (; kt + 2 * U <= kq; kt += 2 * U) {
        mm(0, kt);
        FENCE();
        if (kt + 2 * U < kq) load(0, kt + 2 * U);
        FENCE();
        mm(1, kt + U);
        FENCE();
        if (kt + 3 * U < kq) load(1, kt + 3 * U);
        FENCE();
    }
    mm_rest(0, kt);
    mm_rest(1, kt + U);

    // ---- this workgroup's share of the outputs of the pre-pass
    // (whole tiles: the lane's own address again; as with the clamp of load(), the general form cost them 0.7 of 17.4 us at
    // 4 x 4096 x 22000)
    for (int t = blockIdx.x * 4 + w; t < KT; t += gridDim.x * 4)
        *((v4i*)(a.Xq + (size_t)t * TILE_BYTES) + lane) =
            *(const v4i*)(T == 32 ? xb + t * xstep : (lane & 31) < sp ? xq + ((2 * t + (lane >> 5)) * sp + (lane & 31)) * 16 : xq + sp * KT * 32);
    if (blockIdx.x == 0) {
        for (int q = tid; q < cnt; q += 256) a.idx[q] = s_idx[q];
        for (int q = tid; q < s * a.opad; q += 256) {
            const int i = q / a.opad, t = q - i * a.opad;
            a.Xo[q] = t < cnt ? a.X[(size_t)i * h + s_idx[t]] : (unsigned short)0;
        }
        if (tid < s) a.cx[tid] = (unsigned short)s_row[tid];
    }

    // ---- the four partial sums meet in LDS; token i, column jj of the tile: register 4 (jj / 8) + jj % 4 of lane
    // i + 32 ((jj / 4) % 2), or jj % 4 of lane i + 16 (jj / 4)
#pragma unroll
    for (int q = 0; q < NQ; q++) red[w][q][lane] = acc[q];
#pragma unroll
    for (int q = 0; q < SSLOTS / NG; q++) {
        s_xo[ig + NG * q][jj] = xo[q];
        s_wo[ig + NG * q][jj] = a.Wf ? wo[q] : dequant_bits((int)(int8_t)wo[q], cwb);
    }
    __syncthreads();
    __shared__ float s_t[16][64];  // the outlier product, laid out as the sums
    if (a.tiled_order) {
        if (w == 0) {
            const int gl = lane >> 5, ll = lane & 31;
            v16f t = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int ks = 0; ks < SSLOTS / 16; ks++) {
                if (16 * ks >= cnt) continue;
                v8h wa, xa;
#pragma unroll
                for (int e = 0; e < 8; e++) {
                    wa[e] = __builtin_bit_cast(_Float16, s_wo[16 * ks + 8 * gl + e][ll]);
                    xa[e] = __builtin_bit_cast(_Float16, s_xo[16 * ks + 8 * gl + e][ll]);
                }
                t = __builtin_amdgcn_mfma_f32_32x32x16_f16(wa, xa, t, 0, 0, 0);
            }
#pragma unroll
            for (int q = 0; q < 16; q++) s_t[q][lane] = t[q];
        }
        __syncthreads();
    }
    if (j >= o) return;
    const int rr = 4 * (jj >> 3) + (jj & 3), l0 = 32 * ((jj >> 2) & 1);
    const int rq = T == 16 ? jj & 3 : rr, lq = T == 16 ? 16 * (jj >> 2) : l0;
    const float cwj = f16_bits_to_float(cwb);
    for (int i = ig; i < s; i += NG) {
        const int l = l0 + i;
        const int c = red[0][rq][lq + i] + red[1][rq][lq + i] + red[2][rq][lq + i] + red[3][rq][lq + i];
        if (a.tiled_order) {
            const float sx = f16_bits_to_float((unsigned short)s_row[i]) * (1.0f / 16129.0f);
            a.Out[(size_t)i * o + j] = (_Float16)__builtin_fmaf((float)c * sx, cwj, s_t[rr][l]);
            continue;
        }
        // Eq. 7 dequantization, then the outlier product of Eq. 8 accumulated in fp32
        float d = (float)c * (f16_bits_to_float((unsigned short)s_row[i]) * (1.0f / 16129.0f)) * cwj;
        for (int t = 0; t < (cnt < SSLOTS ? cnt : SSLOTS); t++)
            d = __builtin_fmaf(f16_bits_to_float(s_xo[t][i]), f16_bits_to_float(s_wo[t][jj]), d);
        for (int t = SSLOTS; t < cnt; t++) {  // more outlier columns than were fetched: rare
            const int k = s_idx[t];
            const unsigned short wk =
                a.Wf ? a.Wf[(size_t)k * o + j]
                     : dequant_bits((int)a.Wq[((size_t)jt * KT + (k >> 5)) * TILE_BYTES + tile_byte(jr, k & 31)], cwb);
            d = __builtin_fmaf(f16_bits_to_float(a.X[(size_t)i * h + k]), f16_bits_to_float(wk), d);
        }
        a.Out[(size_t)i * o + j] = (_Float16)d;
    }
}

// log2 of the threads per row, and the chunks of 8 features per thread (0: X too large for this path)
static int small_chunks(int s, int h, int cap, int* lg)
{
    if (s > 32 || h < 8 || cap > JOB_MAX_CAP) return 0;
    int l = 8;
    while ((256 >> l) < s) l--;
    *lg = l;
    const int n = (4 * k_tiles(h) + (1 << l) - 1) >> l;
    return n <= 16 ? n : 0;
}

static bool tiled_order(int s, int h, int o) { return !ksplit_takes(s, h, o) && !decode_kernel_takes(s, h, o, false); }

// Where one kernel is the better way, per call against the separate kernels.  Every workgroup repeats the
// pre-pass, about 1 200 vector instructions per wave at 16 chunks, so its price grows with the chunks, with the tokens and
// with the workgroups that share a compute unit; what it saves is two launches and two short kernels, 6 to 10 us.
//   up to 8 chunks, up to two workgroups per compute unit, or up to 8 tokens: 8 x 256 x 512 10.2 against 15.3 us, 2 x 4096 x
//     4096 10.2 / 17.0, 1 x 5120 x 20480 18.4 / 29.1, 8 x 2048 x 49152 28.9 / 29.6, 32 x 512 x 16384 15.1 / 17.8
//   more workgroups, where llmint8_matmul takes the tiled kernel: 16 x 1024 x 20480 16.6 / 19.9 (640 column tiles), 16 x 512 x
//     28672 16.3 / 17.3 (4 chunks), but 16 x 1024 x 28672 22.2 / 20.7, 32 x 384 x 28672 23.2 / 16.6, 32 x 512 x 20480 17.7 / 16.9
//   more workgroups, where it takes the weight-streaming kernel: as long as K is too short for a full batch of loads there:
//     12 x 768 x 49152 26.2 / 31.1, 16 x 896 x 36864 24.6 / 31.3, 32 x 384 x 36864 28.9 / 31.0, but 16 x 1024 x 49152 30.2 / 25.9,
//     32 x 512 x 40960 30.5 / 28.4, and with its two full rounds of 2 x 4 tiles 32 x 384 x 32768 26.5 / 23.1
//   9 to 16 chunks: 1 x 32768 x 4096 32.6 / 44.8, 8 x 4096 x 12288 18.9 / 21.7 (384 column
//     tiles), but 1 x 32768 x 16384 94.9 / 92.9 (512) and 32 x 1024 x 32768 35.5 / 27.5 (1 024): taken up to
//     one and a half workgroups per compute unit
//   13 and more of them, against separate kernels that read X once: 1 x 20480 x 4096 23.8 / 31.0, 8 x 4096 x 4096 14.5 / 14.7, but
//     16 x 2048 x 4096 14.5 / 13.7, 32 x 1024 x 1024 15.8 / 13.6, 20 x 1024 x 8192 14.5 / 13.0: not from 16 tokens on
bool linear_small_takes(int s, int h, int o, int cap)
{
    int lg, cus = 0;
    if (g_decode_cfg.load(std::memory_order_relaxed) >= 0) return false;  // test hook: the separate kernels
    const int n = small_chunks(s, h, cap, &lg);
    if (n == 0) return false;
    if (cap > SSLOTS && tiled_order(s, h, o)) return false;
    if (prefill_device_setup(&cus) != hipSuccess) cus = 256;
    const int JT = row_tiles(o);
    if (n > 8) return 2 * JT <= 3 * cus && (s < 16 || n <= 12);
    if (JT <= 2 * cus || s <= 8) return true;
    if (tiled_order(s, h, o)) return 2 * JT <= 5 * cus ? s <= 16 || n <= 4 : s <= 16 && n <= 4;
    const int kq = k_tiles(h) / 4;  // k-tiles per wave there
    if (s <= 16) return kq < 8;
    return JT > 4 * cus ? kq < 4 : n <= 4;
}

// Whether a workgroup takes half a tile.  Us per call, half / whole tiles:
//   up to 4 chunks: while all workgroups are resident, five to a compute unit: 1 x 4096 x 4096 7.6 / 9.2, 1 x 5120 x 20480 on int8 rows
//     17.1 / 18.2, 8 x 512 x 16384 9.0 / 9.3, 1 x 8192 x 20480 26.4 / 29.2; but 1 x 5120 x 25600 23.4 / 22.3, 3 x 768 x 40960 16.9 / 15.6
//   8: three: 1 x 12288 x 4096 12.3 / 16.7, 2 x 8192 x 11000 16.2 / 20.1, 1 x 16384 x 12288 31.0 / 38.7, 8 x 2048 x 8192 11.3 / 11.3; but
//     4 x 4096 x 16384 19.0 / 15.2, 8 x 2048 x 20480 20.8 / 16.1
//   16: one: 1 x 32768 x 4096 27.5 / 32.0, 8 x 4096 x 2048 13.0 / 14.6; but 1 x 20480 x 5120 25.7 / 24.3
static bool half_tiles(int s, int o, int n)
{
    int cus = 0;
    if (prefill_device_setup(&cus) != hipSuccess) cus = 256;
    const int JT = row_tiles(o);
    return s <= 16 && 2 * JT <= (n <= 4 ? 5 : n <= 8 ? 3 : 1) * cus;
}

hipError_t launch_linear_small(const void* X, int s, int h, unsigned thr, const int8_t* Wq, const unsigned short* cw,
                               const unsigned short* Wf, int o, int32_t* idx, int cap, int32_t* count, int32_t* status,
                               int8_t* Xq, unsigned short* cx, unsigned short* Xo, unsigned short* Out, hipStream_t st)
{
    int lg = 0;
    const int n = small_chunks(s, h, cap, &lg);
    if (n == 0) return hipErrorInvalidValue;
    const int KT = k_tiles(h);
    const SmallArgs a = {(const unsigned short*)X, s, h, o, KT, lg, thr, Wq, cw, Wf, idx, cap, opad_of(cap), count, status,
                         Xq, cx, Xo, (_Float16*)Out, tiled_order(s, h, o) ? 1 : 0};
    const size_t shm = (size_t)(256 >> lg) * KT * 32 + 16;
    const bool half = half_tiles(s, o, n);
    const int grid = row_tiles(o) * (half ? 2 : 1);
#define SMALL(XC)                                               \
    do {                                                        \
        if (half)                                               \
            linear_small_kernel<XC, 16><<<grid, 256, shm, st>>>(a); \
        else                                                    \
            linear_small_kernel<XC, 32><<<grid, 256, shm, st>>>(a); \
    } while (0)
    if (n <= 1)
        SMALL(1);
    else if (n <= 4)
        SMALL(4);
    else if (n <= 8)
        SMALL(8);
    else
        SMALL(16);
#undef SMALL
    return hipGetLastError();
}

}  // namespace llmint8
