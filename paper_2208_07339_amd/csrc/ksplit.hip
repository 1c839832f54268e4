// Eq. 7 + Eq. 8 for products that are too small to fill the chip with the tiles of gemm.hip.
#include <type_traits>

#include "common.h"

namespace llmint8 {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef _Float16 v4h __attribute__((ext_vector_type(4)));

#define FENCE() __builtin_amdgcn_sched_barrier(0)

constexpr int KSLOTS = 32;  // outlier slots kept in LDS at a time

struct KsplitArgs {
    const int8_t* Wq;
    const int8_t* Xq;
    int KT, JT, RT, nP, nQ;
    const unsigned short* cw;
    const unsigned short* cx;
    const unsigned short* Wf;
    int rows_are_slots, wrows;
    const int32_t* idx;
    const unsigned short* Xo;
    const int32_t* count;
    int cap, opad;
    _Float16* Out;
    int32_t* Cdbg;
    int s, h, o;
    ZpArgs zp;
};

// ---------------------------------------------------------------------------
// A tile of 128 or more columns per workgroup leaves most compute units without work when the product is small, and
// one compute unit pulls only so much: about 30 KB/us of W from memory (48 from the last-level cache), 60 to 85 in
// all.  So the tiles here are 32 NJ columns x 32 NI tokens, and the eight waves of a workgroup split K among
// them (wave w takes the k-tiles w, w + 8, ..), each with all NJ x NI accumulators.  Operands go straight into
// registers, R k-tiles in flight per wave, with no barrier in the K loop.  The eight sums meet in LDS, token tile by
// token tile (32-bit integers: the same in any order).  The kernel alone, against the tiles of gemm.hip, on a W from
// memory / from the last-level cache: 53 x 9856 x 4480 39.6 -> 22.0 / 29.3 -> 16.0 us, 48 x 14336 x 4096 57.5 -> 20.3 /
// 39.3 -> 13.7, 128 x 12288 x 8192 58.9 -> 35.4 / 36.3 -> 23.7, 64 x 4096 x 4096 15.7 -> 9.4, 96 x 12288 x 12288 57.6 ->
// 46.8 / 35.9 -> 29.6.
//
// Measured and left out: batches of several k-tiles instead of a ring, contiguous parts of K per wave, and starting
// points in K that differ from workgroup to workgroup (all the same time); W streamed past the caches (96 x 5120 x
// 15360 26.5 -> 23.3 us from memory, but 19.4 -> 22.0 from the last-level cache).
//
// T = 16 (one column tile, up to 16 tokens): half a column tile and 16 x 16 x 64 MFMAs, the waves take pairs of k-tiles.
//
// ZP: zeropoint constants, as in gemm.hip.
// ---------------------------------------------------------------------------
template <int NJ, int NI, int R, int T, bool ZP>
__global__ void __launch_bounds__(512, 2) gemm_ksplit_kernel(const KsplitArgs a)
{
    static_assert(T == 32 || (NJ == 1 && NI == 1), "half tiles come alone");
    constexpr int NW = 8, NC = T * NJ, NTK = T * NI, NM = T == 16 ? 1 : NJ * 4, STEP = NW * (T == 16 ? 128 : 64);
    typedef std::conditional_t<T == 16, v4i, v16i> acc_t;
    __shared__ v4i red[4][NM][64];                      // [wave][4 columns of a tile][token + 32 half, swizzled]
    __shared__ unsigned short s_wo[KSLOTS][NC];
    __shared__ __attribute__((aligned(16))) unsigned short s_xo[NTK][KSLOTS];
    __shared__ float s_sx[ZP ? 1 : NTK];
    __shared__ double s_zc[ZP ? 3 : 1][ZP ? NC : 1];
    __shared__ int4 s_zx[ZP ? NTK : 1];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int s = a.s, o = a.o, KT = a.KT;
    // consecutive workgroups go round-robin to the 8 XCDs; each XCD gets a contiguous run of the tiles, column block by
    // column block, so that the token blocks of one column block share its part of W in one L2
    const int total = a.nP * a.nQ, xcd = blockIdx.x & 7, more = total & 7;
    const int tile = xcd * (total >> 3) + (xcd < more ? xcd : more) + (blockIdx.x >> 3);
    const int cb = tile / a.nQ, tb = tile - cb * a.nQ;
    const int J0 = cb * NC, I0 = tb * NTK;

    // ---- epilogue operands
    int cnt = *a.count;
    constexpr int TPC = 512 / NC;          // threads per column: a thread has slots q TPC + tid / NC of column tid % NC
    constexpr int NS = KSLOTS / TPC;
    const int jc = tid % NC, t0 = tid / NC;
    unsigned short wo[NS], cx_raw = 0;
    int kk[NS];
#pragma unroll
    for (int q = 0; q < NS; q++) {
        const int t = t0 + q * TPC;
        kk[q] = a.rows_are_slots ? t : a.idx[t < a.cap ? t : 0];
    }
    us8 xo = (us8)(0);
    int4 zx = make_int4(0, 0, 0, 0);
    double zc[3] = {0, 0, 0};
    const int xs = (tid & 3) * 8;  // this thread's first slot of token tid / 4
    if (tid < 4 * NTK && xs < a.opad) {
        const int i = I0 + (tid >> 2);
        xo = *(const us8*)(a.Xo + (size_t)(i < s ? i : s - 1) * a.opad + xs);
    }
    if (tid < NTK) {
        const int i = I0 + tid;
        if constexpr (ZP) zx = a.zp.zcx[i < s ? i : s - 1]; else cx_raw = a.cx[i < s ? i : s - 1];
    }
    // this thread's outputs: token il of a tile, columns jl .. jl + 3
    const int il = tid / (NC / 4), ch = tid % (NC / 4), jl = 4 * ch, j = J0 + jl;
    if constexpr (ZP) {
        if (tid < NC) {
#pragma unroll
            for (int q = 0; q < 3; q++) zc[q] = a.zp.colc[(size_t)q * a.zp.pitch + J0 + tid];
        }
    }
    FENCE();

    // ---- this wave's part of K
    const int n = ((T == 16 ? KT / 2 : KT) - w + NW - 1) / NW;  // k-tiles (or pairs) w, w + 8, ..; none in a short K
    const int k0 = n > 0 ? (T == 16 ? 2 * w : w) : 0;
    const int half = T == 16 ? (lane >> 4) * 32 + (lane & 15) : lane;  // this lane's piece
    const v4i *wp[NJ], *xp[NI];
#pragma unroll
    for (int c = 0; c < NJ; c++) {
        const int jt = T == 16 ? cb >> 1 : cb * NJ + c < a.JT ? cb * NJ + c : a.JT - 1;
        wp[c] = (const v4i*)(a.Wq + ((size_t)jt * KT + k0) * TILE_BYTES) + half + (T == 16 ? (cb & 1) * 16 : 0);
    }
#pragma unroll
    for (int t = 0; t < NI; t++) {
        const int rt = tb * NI + t < a.RT ? tb * NI + t : a.RT - 1;
        // lane -> token lane % 32 of the tile; for tokens that do not exist the first one again, so that their zeros are not
        // fetched (unused: nothing is stored for them)
        xp[t] = (const v4i*)(a.Xq + ((size_t)rt * KT + k0) * TILE_BYTES) + (NI > 1 || 32 * rt + (lane & (T - 1)) < s ? half : half & ~(T - 1));
    }
    acc_t acc[NJ][NI];
#pragma unroll
    for (int c = 0; c < NJ; c++)
#pragma unroll
        for (int t = 0; t < NI; t++)
#pragma unroll
            for (int q = 0; q < T * T / 64; q++) acc[c][t][q] = 0;
    v4i wv[R][NJ], xv[R][NI];
    auto load = [&](int r, int kt) {
        int k = kt < n ? kt : n - 1;
        k = k > 0 ? k : 0;
#pragma unroll
        for (int c = 0; c < NJ; c++) wv[r][c] = wp[c][(size_t)k * STEP];
#pragma unroll
        for (int t = 0; t < NI; t++) xv[r][t] = xp[t][(size_t)k * STEP];
    };
    auto mm = [&](int r) {
#pragma unroll
        for (int c = 0; c < NJ; c++)
#pragma unroll
            for (int t = 0; t < NI; t++) {
                if constexpr (T == 16) acc[c][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wv[r][c], xv[r][t], acc[c][t], 0, 0, 0);
                else acc[c][t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wv[r][c], xv[r][t], acc[c][t], 0, 0, 0);
            }
    };
#pragma unroll
    for (int r = 0; r < R; r++) {
        load(r, r);
        FENCE();
    }
    cnt = cnt < 0 ? 0 : (cnt > a.cap ? a.cap : cnt);
#pragma unroll
    for (int q = 0; q < NS; q++) {
        const unsigned k = (unsigned)kk[q];
        const bool ok = k < (unsigned)a.wrows && t0 + q * TPC < cnt && J0 + jc < o;
        wo[q] = a.Wf[(size_t)(ok ? k : 0u) * o + (J0 + jc < o ? J0 + jc : 0)];
        if (!ok) wo[q] = 0;
    }
    FENCE();
    int kt = 0;
    for (; kt + R <= n; kt += R) {
#pragma unroll
        for (int r = 0; r < R; r++) {
            mm(r);
            FENCE();
            load(r, kt + R + r);
            FENCE();
        }
    }
#pragma unroll
    for (int r = 0; r < R; r++)
        if (kt + r < n) mm(r);

    // ---- epilogue operands into LDS
#pragma unroll
    for (int q = 0; q < NS; q++)
        s_wo[t0 + q * TPC][jc] = wo[q];
    if (tid < 4 * NTK) *(us8*)&s_xo[tid >> 2][xs] = xo;
    if (tid < NTK) {
        if constexpr (ZP) s_zx[tid] = zx; else s_sx[tid] = f16_bits_to_float(cx_raw) * (1.0f / 16129.0f);
    }
    if constexpr (ZP) {
        if (tid < NC) {
#pragma unroll
            for (int q = 0; q < 3; q++) s_zc[q][tid] = zc[q];
        }
    }
    // More outlier columns than fit: a chunk of slots in LDS after the other, the next one's operands on their way meanwhile;
    // their product comes first, or last up to 32 tokens.  Calls with 200 columns, 128 x 12288 x 8192: 56 us; with every column's
    // operands from memory for each output 180, with the tiles of gemm.hip 93.  Products of few tokens with 200, so / from memory
    // for each output / with the weight-streaming kernel: 8 x 8192 x 4096 12.7 / 66.9 / 40.2, 16 x 4096 x 4096 9.9 / 44.9 / 66.1, 32 x
    // 4096 x 2048 11.8 / 47.2, zeropoint 8 x 12288 x 4096 33.7 / 92 / 65.4.
    const bool many = cnt > KSLOTS;
    float od[NI][4];
#pragma unroll
    for (int t = 0; t < NI; t++)
#pragma unroll
        for (int e = 0; e < 4; e++) od[t][e] = 0.0f;
    auto chunks = [&]() {  // by all threads; od goes on from what it holds
        auto rows_of = [&](int q0) {  // the rows of this thread's slots of a chunk
#pragma unroll
            for (int q = 0; q < NS; q++) {
                const int t = q0 + t0 + q * TPC;
                kk[q] = a.rows_are_slots ? t : a.idx[t < cnt ? t : 0];
            }
        };
        rows_of(KSLOTS);
        for (int q0 = 0;; q0 += KSLOTS) {
            const int q1 = q0 + KSLOTS;
            if (q1 < cnt) {
#pragma unroll
                for (int q = 0; q < NS; q++) {
                    const unsigned k = (unsigned)kk[q];
                    const bool ok = k < (unsigned)a.wrows && q1 + t0 + q * TPC < cnt && J0 + jc < o;
                    wo[q] = a.Wf[(size_t)(ok ? k : 0u) * o + (J0 + jc < o ? J0 + jc : 0)];
                    if (!ok) wo[q] = 0;
                }
                if (tid < 4 * NTK && q1 + xs < a.opad) {
                    const int i = I0 + (tid >> 2);
                    xo = *(const us8*)(a.Xo + (size_t)(i < s ? i : s - 1) * a.opad + q1 + xs);
                }
                rows_of(q1 + KSLOTS);
            }
            __syncthreads();  // the chunk is in LDS
            const int ns = cnt - q0 < KSLOTS ? cnt - q0 : KSLOTS;
            if (il < T)
                for (int q = 0; q < ns; q++) {
                    float wf[4];
#pragma unroll
                    for (int e = 0; e < 4; e++) wf[e] = f16_bits_to_float(s_wo[q][jl + e]);
#pragma unroll
                    for (int t = 0; t < NI; t++) {
                        const float x = f16_bits_to_float(s_xo[T * t + il][q]);
#pragma unroll
                        for (int e = 0; e < 4; e++) od[t][e] = __builtin_fmaf(x, wf[e], od[t][e]);
                    }
                }
            if (q1 >= cnt) break;
            __syncthreads();
#pragma unroll
            for (int q = 0; q < NS; q++) s_wo[t0 + q * TPC][jc] = wo[q];
            if (tid < 4 * NTK) *(us8*)&s_xo[tid >> 2][xs] = xo;
        }
    };
    if (T == 32 && __builtin_expect(many && s > 32, 0)) chunks();  // uniform
    float cwj[4] = {0, 0, 0, 0};
    if constexpr (!ZP) {
#pragma unroll
        for (int e = 0; e < 4; e++) cwj[e] = f16_bits_to_float(a.cw[j + e < o ? j + e : 0]);
    }
#pragma unroll
    for (int t = 0; t < NI; t++) {
        if (t > 0) __syncthreads();
        // waves 4 .. 7 hand their sums to waves 0 .. 3
        if (w >= 4) {
#pragma unroll
            for (int m = 0; m < NM; m++) {
                const v4i v = {acc[m >> 2][t][4 * (m & 3)], acc[m >> 2][t][4 * (m & 3) + 1], acc[m >> 2][t][4 * (m & 3) + 2],
                               acc[m >> 2][t][4 * (m & 3) + 3]};
                red[w - 4][m][lane ^ ((m & 7) << 2)] = v;
            }
        }
        __syncthreads();
        if (w < 4) {
#pragma unroll
            for (int m = 0; m < NM; m++) {
                v4i v = red[w][m][lane ^ ((m & 7) << 2)];
#pragma unroll
                for (int e = 0; e < 4; e++) v[e] += acc[m >> 2][t][4 * (m & 3) + e];
                red[w][m][lane ^ ((m & 7) << 2)] = v;
            }
        }
        __syncthreads();
        const int i = I0 + T * t + il;
        const bool mine = il < T && i < s && j < o;
        float p[4] = {0, 0, 0, 0}, d[4] = {0, 0, 0, 0};
        if (mine) {
            const int m = T == 16 ? 0 : ch >> 1, l = T == 16 ? il + 16 * ch : (il + 32 * (ch & 1)) ^ ((m & 7) << 2);
            const v4i c = red[0][m][l] + red[1][m][l] + red[2][m][l] + red[3][m][l];
            if (a.Cdbg) {
#pragma unroll
                for (int e = 0; e < 4; e++)
                    if (j + e < o) a.Cdbg[(size_t)i * o + j + e] = c[e];
            }
            // Eq. 7 (zeropoint: Eq. 5), to which Eq. 8 adds the outlier product: that sum first, as in gemm.hip, or, up
            // to 32 tokens, last, as in the weight-streaming kernel (the one-call path there gives the same bits)
            if constexpr (ZP) {
                const int4 rec = s_zx[T * t + il];
                const double sa = zp_range((unsigned)rec.x) * (1.0 / 254.0), za = (double)rec.y, rs = (double)rec.z;
#pragma unroll
                for (int e = 0; e < 4; e++)
                    p[e] = (float)(sa * __builtin_fma((double)c[e], s_zc[0][jl + e],
                                                      __builtin_fma(rs, s_zc[1][jl + e], za * s_zc[2][jl + e])));
            } else {
#pragma unroll
                for (int e = 0; e < 4; e++) p[e] = (float)c[e] * s_sx[T * t + il];
            }
            if (s <= 32) {
#pragma unroll
                for (int e = 0; e < 4; e++) d[e] = ZP ? p[e] : p[e] * cwj[e];
            }
        }
        if constexpr (NJ == 1 && NI == 1) {  // (the only shape of up to 32 tokens)
            if (__builtin_expect(many && s <= 32, 0)) {  // uniform
#pragma unroll
                for (int e = 0; e < 4; e++) od[t][e] = d[e];
                chunks();
            }
        }
        if (mine) {
            if (many) {
#pragma unroll
                for (int e = 0; e < 4; e++) d[e] = od[t][e];
            }
            const int ns = many ? 0 : cnt;
            for (int q = 0; q < ns; q++) {
                const float x = f16_bits_to_float(s_xo[T * t + il][q]);
#pragma unroll
                for (int e = 0; e < 4; e++) d[e] = __builtin_fmaf(x, f16_bits_to_float(s_wo[q][jl + e]), d[e]);
            }
            if (s > 32) {
#pragma unroll
                for (int e = 0; e < 4; e++) d[e] = ZP ? d[e] + p[e] : __builtin_fmaf(p[e], cwj[e], d[e]);
            }
            const v4h hv = {(_Float16)d[0], (_Float16)d[1], (_Float16)d[2], (_Float16)d[3]};
            _Float16* out = a.Out + (size_t)i * o + j;
            if (j + 4 <= o) {
                __builtin_memcpy(out, &hv, 8);
            } else {
#pragma unroll
                for (int e = 0; e < 4; e++)
                    if (j + e < o) out[e] = hv[e];
            }
        }
    }
}

// R, RZ: k-tiles in flight per wave, absmax and zeropoint
template <int NJ, int NI, int R, int RZ, int T = 32>
static hipError_t launch(KsplitArgs& a, bool zp, hipStream_t st)
{
    a.nP = T == 16 ? 2 * a.JT : (a.JT + NJ - 1) / NJ;
    a.nQ = (a.RT + NI - 1) / NI;
    const int grid = a.nP * a.nQ;
    if (zp)
        gemm_ksplit_kernel<NJ, NI, RZ, T, true><<<grid, 512, 0, st>>>(a);
    else
        gemm_ksplit_kernel<NJ, NI, R, T, false><<<grid, 512, 0, st>>>(a);
    return hipGetLastError();
}

// Estimated time of a tile grid in us, without what every launch costs: the bytes a compute unit pulls, of W and
// in all, and the bytes that all of them pull together (13 TB/s).  two: two workgroups fit a compute unit.
static double pull_time(int s, int h, int o, int cols, int toks, int cus, bool two, double rate)
{
    const double tiles = (double)((o + cols - 1) / cols) * ((s + toks - 1) / toks);
    double rounds = tiles / cus;
    if (!two || rounds < 1) rounds = (double)(long)((tiles + cus - 1) / cus);
    const double w = 1e-3 * h * cols, all = 1e-3 * h * (cols + toks);
    const double t_w = rounds * w / ((double)h * o > 40e6 ? 38.0 : 48.0), t_all = rounds * all / rate;
    const double t_l2 = tiles * all / 13000.0;
    const double t = t_w > t_all ? t_w : t_all;
    return t > t_l2 ? t : t_l2;
}

constexpr int KS_SHAPES = 4;
static const int ks_nj[KS_SHAPES] = {1, 2, 2, 2}, ks_ni[KS_SHAPES] = {1, 1, 2, 3};

// The shape for a product, or -1 where the other kernels are the better ones.  Products whose tiles in gemm.hip
// fill the chip stay there (512 x 4096 x 4096 17.0 against 17.6 us at best, 630 x 13824 x 6528 68 against 103); the
// others come here if the estimate says that they gain 8 % with the launch counted (it is within a third of
// the measured times on 25 products of 33 to 1 094 tokens, and low for these kernels rather than for those).
// It counts a W of up to 40 MB as cached; on a W from memory the choice is the faster one all the same: 33 x 4096 x 4096 20.9
// us there, 8.9 here, 128 x 12288 x 8192 56.5 / 35.4, 1000 x 8192 x 768 37.0 / 21.3, 96 x 5120 x 9000 27.2 / 23.4, 96 x 12288 x
// 12288 56.6 / 46.2.
// Up to 16 tokens half a column tile to a workgroup: twice the compute units that whole tiles reach, per call half tiles here / the
// weight-streaming kernel or whole tiles here: 3 x 37120 x 640 22.8 / 30.7 us, 16 x 12288 x 2048 16.1 / 18.6, 16 x 4096 x 4096 13.2 /
// 16.0, 12 x 20480 x 4096 25.0 / 32.8, 6 x 7793 x 5000 18.7 / 20.3, 4 x 20480 x 5120 30.1 / 32.0; at 8 x 8192 x 6000 21.5 / 21.2.
// From a pair of k-tiles for each wave on.  Up to 8 tokens with at most 128 k-tiles and an eighth of the compute units' column tiles
// keep the weight-streaming kernel.  That is not the faster one on any size measured: zeropoint calls on a W from memory, half tiles /
// weight-streaming, 8 x 4096 x 1024 15.1 / 16.4 us, 8 x 2048 x 512 14.2 / 15.2, 8 x 1024 x 1024 14.9 / 15.2, and past the line 8 x 6144 x
// 1024 16.1 / 18.6, 2 x 5120 x 640 16.3 / 18.1.  It keeps what llmint8_debug_kernel_for says of these products, at up to 1.3 us a call.
// 17 to 32 tokens: the weight-streaming kernel keeps every W that gives a quarter of the compute units a column tile; below that
// 8 waves per column tile pull more than 4; the matmul alone there / here on a W from memory: 32 x 2048 x 2048 7.3 / 7.0 us,
// 24 x 8192 x 512 12.0 / 11.8.
int ksplit_shape(int s, int h, int o)
{
    if (g_decode_cfg.load(std::memory_order_relaxed) >= 0 || g_force_cfg.load(std::memory_order_relaxed) >= 0)
        return -1;  // test hooks: the other kernels
    int cus = 0;
    if (prefill_device_setup(&cus) != hipSuccess) cus = 256;
    if (s <= 16) return 8 * row_tiles(o) <= 5 * cus && k_tiles(h) >= 16 && (s > 8 || k_tiles(h) > 128 || 8 * row_tiles(o) > cus) ? 0 : -1;
    if (s <= 32) return 4 * row_tiles(o) <= cus ? 0 : -1;
    int cols, toks;
    prefill_tile_size(s, h, o, &cols, &toks);
    if ((long)((o + cols - 1) / cols) * ((s + toks - 1) / toks) >= cus) return -1;
    // (a launch with next to nothing to do takes 5.5 us there, 4.5 us here and 0.6 us more per token tile of a
    // workgroup: 384 x 700 x 4800 8.9 us there and 11.1 here)
    double best = 0.92 * (pull_time(s, h, o, cols, toks, cus, false, 85.0) + 5.5);
    int shape = -1;
    for (int c = 0; c < KS_SHAPES; c++) {
        const double t = pull_time(s, h, o, 32 * ks_nj[c], 32 * ks_ni[c], cus, ks_ni[c] == 1, 65.0) +
                         4.5 + 0.6 * ks_ni[c];
        if (t < best) {
            best = t;
            shape = c;
        }
    }
    return shape;
}

hipError_t launch_gemm_ksplit(const int8_t* Xq, const unsigned short* cx, const unsigned short* Xo,
                              const int32_t* count, int cap, const int8_t* Wq, const unsigned short* cw,
                              const unsigned short* Wf, int rows_are_slots, const int32_t* idx, int s, int h, int o,
                              unsigned short* Out, int32_t* Cdbg, hipStream_t st, const ZpArgs* zp)
{
    KsplitArgs a = {Wq, Xq, k_tiles(h), row_tiles(o), row_tiles(s), 0, 0, cw, cx, Wf, rows_are_slots,
                    rows_are_slots ? opad_of(cap) : h, idx, Xo, count, cap, opad_of(cap), (_Float16*)Out, Cdbg, s, h, o,
                    zp ? *zp : ZpArgs{nullptr, nullptr, 0}};
    switch (ksplit_shape(s, h, o)) {
        case 0: return s <= 16 ? launch<1, 1, 8, 8, 16>(a, zp, st) : launch<1, 1, 8, 8>(a, zp, st);
        case 1: return launch<2, 1, 6, 5>(a, zp, st);  // two workgroups per compute unit
        case 2: return launch<2, 2, 6, 6>(a, zp, st);
        case 3: return launch<2, 3, 4, 4>(a, zp, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace llmint8
