// Hidden states: constants and codes with X read once.
//
// row_codes_kernel     a workgroup holds a few whole rows in registers.  Inside the one-call entry points the outlier
//                      columns are not known yet: the kernel takes its rows' constants over the entries below the
//                      threshold, which is right unless the entry that decides sits in a column that another row
//                      makes an outlier, writes the codes, and leaves the list of the columns in which its own rows
//                      reach the threshold.  With the columns known (KNOWN: the stand-alone calls) the constants are
//                      final and the gathered columns Xo are written too.
// join_records_kernel  joins many lists (more than 512, or 256 where they may be long) to a bitmap in memory first.
// settle_rows_kernel   joins the lists to the outlier set, or takes it from that bitmap, writes idx, count, status and Xo, clears the codes of
//                      entries below the threshold in outlier columns, and makes the rows anew whose constant came
//                      from one of those (or all rows, where more columns qualify than the buffer takes: the columns
//                      past its end are ordinary ones).
#include <type_traits>

#include "common.h"

namespace llmint8 {

typedef unsigned int u4 __attribute__((ext_vector_type(4)));

// A record: the outlier columns that one workgroup found.  Word 0 counts them, words 1 .. hold the first cap + 1 of them in
// ascending order: the set is cut after cap columns, none of its first cap columns is missing from the first cap of the
// lists that have it, and one more says that there are more.  A multiple of 32 bytes each.
__host__ __device__ inline int record_words(int cap) { return (2 + cap + 15) & ~15; }

namespace {

// Sixteen features of a row as eight words of two: whole-word operations and the packed 16-bit instructions.  (From vectors
// of sixteen-bit elements the compiler takes words apart and puts them together again: 24 instructions for the
// eight of mags().)
struct w8 { unsigned w[8]; };

__device__ __forceinline__ w8 words(us8 a, us8 b)
{
    const u4 x = __builtin_bit_cast(u4, a), y = __builtin_bit_cast(u4, b);
    return {{x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]}};
}
__device__ __forceinline__ w8 mags(const w8& v)
{
    w8 a;
#pragma unroll
    for (int q = 0; q < 8; q++) a.w[q] = v.w[q] & 0x7fff7fffu;
    return a;
}
// the largest of 16 magnitudes
__device__ __forceinline__ unsigned top16(const w8& a)
{
    const unsigned m = pk_max_u16(pk_max_u16(pk_max_u16(a.w[0], a.w[1]), pk_max_u16(a.w[2], a.w[3])),
                                  pk_max_u16(pk_max_u16(a.w[4], a.w[5]), pk_max_u16(a.w[6], a.w[7])));
    const unsigned lo = m & 0xffffu, hi = m >> 16;
    return lo > hi ? lo : hi;
}

// The columns whose bits are set in bitmap[0 .. nw), as a record: by one wave.
__device__ __forceinline__ void write_record(const unsigned* bitmap, int nw, int lane, int cap, unsigned short* rec)
{
    const int q = (nw + 63) >> 6, b0 = lane * q, b1 = min(nw, b0 + q);
    int mine = 0;
    for (int b = b0; b < b1; b++) mine += __popc(bitmap[b]);
    int incl = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int t = __shfl_up(incl, d);
        if (lane >= d) incl += t;
    }
    if (lane == 63) rec[0] = (unsigned short)min(incl, 0xffff);
    int pos = incl - mine;
    if (mine)
        for (int b = b0; b < b1 && pos <= cap; b++)
            for (unsigned x = bitmap[b]; x && pos <= cap; x &= x - 1) rec[1 + pos++] = (unsigned short)(b * 32 + __ffs(x) - 1);
}

// The bits of those of 16 magnitudes that reach thr = t1 + 1, t2 = t1 | t1 << 16: per pair a saturating subtraction that leaves
// 0 below the threshold, a minimum with 1, and the two bits into place.
__device__ __forceinline__ unsigned reach16(const w8& a, unsigned t2)
{
    unsigned f = 0;
#pragma unroll
    for (int q = 0; q < 8; q++) {
        unsigned x;
        asm("v_pk_sub_u16 %0, %1, %2 clamp" : "=v"(x) : "v"(a.w[q]), "v"(t2));
        asm("v_pk_min_u16 %0, %1, %2" : "=v"(x) : "v"(x), "v"(0x10001u));
        f |= ((x | x >> 15) & 3u) << (2 * q);
    }
    return f;
}

// a word of two features with ones where their bits (2q, 2q + 1) are set
__device__ __forceinline__ unsigned spread(unsigned bits, int q)
{
    return __builtin_amdgcn_perm((unsigned)__builtin_amdgcn_sbfe((int)bits, 2 * q + 1, 1), (unsigned)__builtin_amdgcn_sbfe((int)bits, 2 * q, 1), 0x05040100u);
}
__device__ __forceinline__ void clear16(w8& v, unsigned off)
{
#pragma unroll
    for (int q = 0; q < 8; q++) v.w[q] &= ~spread(off, q);
}

// 16 codes of a row, from its 16 features: absmax
__device__ __forceinline__ u4 codes16(const w8& v, float f)
{
    u4 r;
#pragma unroll
    for (int e = 0; e < 4; e++)
        r[e] = pack_low_bytes(code_of_half(v.w[2 * e], f, false), code_of_half(v.w[2 * e], f, true), code_of_half(v.w[2 * e + 1], f, false),
                              code_of_half(v.w[2 * e + 1], f, true));
    return r;
}

// zeropoint; features whose bit in `off` is set have no code (0).  sum: of the codes
__device__ __forceinline__ u4 zp_codes16(const w8& v, double f, int z, unsigned off, int& sum)
{
    u4 r;
#pragma unroll
    for (int q = 0; q < 4; q++) {
        unsigned c[4];
#pragma unroll
        for (int e = 0; e < 4; e++) c[e] = zp_u_bits((unsigned short)(v.w[2 * q + (e >> 1)] >> (16 * (e & 1))), f) - (unsigned)z;
        r[q] = pack_low_bytes(c[0], c[1], c[2], c[3]);
    }
    if (off) {
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const unsigned o4 = (off >> (4 * q)) & 0xfu;
            r[q] &= ~(((o4 & 1u) | (o4 & 2u) << 7 | (o4 & 4u) << 14 | (o4 & 8u) << 21) * 0xffu);
        }
    }
#pragma unroll
    for (int q = 0; q < 4; q++) sum = __builtin_amdgcn_sdot4((int)r[q], 0x01010101, sum, false);
    return r;
}

// Which of the features c .. c+15 do not exist in a row of h
__device__ __forceinline__ unsigned past_row(int c, int h)
{
    return c + 16 <= h ? 0u : (c < h ? (0xffffu << (h - c)) & 0xffffu : 0xffffu);
}

// The extremes of 16 values into hi and lo, two of each in a word
__device__ __forceinline__ void range16(const w8& v, unsigned& hi, unsigned& lo)
{
#pragma unroll
    for (int q = 0; q < 8; q++) {
        hi = pk_max_f16(hi, v.w[q]);
        lo = pk_min_f16(lo, v.w[q]);
    }
}
// the same without the features whose bit in `off` is set: they take part as the lowest and the highest finite value
__device__ __forceinline__ void range16_without(const w8& v, unsigned off, unsigned& hi, unsigned& lo)
{
#pragma unroll
    for (int q = 0; q < 8; q++) {
        const unsigned m = spread(off, q);
        hi = pk_max_f16(hi, (v.w[q] & ~m) | (0xfbfffbffu & m));
        lo = pk_min_f16(lo, (v.w[q] & ~m) | (0x7bff7bffu & m));
    }
}
__device__ __forceinline__ void keys_of(unsigned hi, unsigned lo, unsigned& kmin, unsigned& kmax)
{
    const unsigned k0 = f16_key(lo & 0xffffu), k1 = f16_key(lo >> 16), k2 = f16_key(hi & 0xffffu), k3 = f16_key(hi >> 16);
    kmin = k1 < k0 ? k1 : k0;
    kmax = k3 > k2 ? k3 : k2;
}

// what runs seldom is to lie outside the way of what runs always
__device__ __forceinline__ bool rare(bool x) { return __builtin_expect(x, 0); }

__device__ __forceinline__ void add_bit(unsigned* bitmap, unsigned j)
{
    // (mostly there already; an atomic load, because a volatile one comes out as a flat access that waits for all of memory)
    const unsigned there = __hip_atomic_load(&bitmap[j >> 5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (!((there >> (j & 31)) & 1u)) atomicOr(&bitmap[j >> 5], 1u << (j & 31));
}

// first feature of a lane's group n; past the last group: the last one again
template <int N, int STEP>
__device__ __forceinline__ int first_feature(int g0, int n, int G)
{
    return (n < N - 1 ? g0 + n * STEP : min(g0 + n * STEP, G - 1)) * 16;
}

// The constants and codes of R rows that a workgroup holds in registers: row r in the lanes l of every wave with l % R = r,
// N groups of 16 features per lane in v (group g0 + n STEP of the row; past its last group, that one again), without the
// columns whose bits are set in bitmap.  FIRST: the columns are those that the workgroup's own rows mark, top[] holds the groups' largest
// magnitudes, and zeropoint records carry how many threads hold the row's extremes, for settle_rows_kernel.  valid: the lane's row
// exists (constant and codes zero if not); store: its codes are written, to dst; cx, zc: its constant's place.
template <int N, int LR, int NT, bool ZP, bool FIRST, bool RAGGED>
__device__ __forceinline__ void constants_and_codes(w8 (&v)[N], const unsigned (&top)[N], const unsigned* bitmap, int h, int G, int g0,
                                                    bool valid, bool store, int8_t* dst, unsigned short* cx, int4* zc)
{
    constexpr int R = 1 << LR, STEP = NT >> LR, NW = NT / 64;
    __shared__ unsigned red[ZP ? 2 : 1][NW][R];
    __shared__ int s_sum[ZP ? NW : 1][R], s_like[ZP && FIRST ? NW : 1][R];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r = lane & (R - 1);
    // ---- constants
    unsigned skip[ZP ? (N + 1) / 2 : 1];  // zeropoint: features without a code, 16 bits per group
    unsigned mx = 0, kmin = 0xffffu, kmax = 0;
    unsigned hi = 0xfbfffbffu, lo = 0x7bff7bffu;
    if constexpr (ZP) {
#pragma unroll
        for (int n = 0; n < (N + 1) / 2; n++) skip[n] = 0;
    }
#pragma unroll
    for (int n = 0; n < N; n++) {
        const int c = first_feature<N, STEP>(g0, n, G);
        unsigned off = !RAGGED || c < h ? (bitmap[c >> 5] >> (c & 31)) & 0xffffu : 0u;
        if constexpr (ZP) {
            if (RAGGED) off |= past_row(c, h);
            // (the last group once more: its own thread alone counts towards how many have an extreme)
            if (FIRST && n == N - 1 && g0 + n * STEP >= G) off = 0xffffu;
            if (__any(off != 0)) {
                range16_without(v[n], off, hi, lo);
                skip[n / 2] |= off << (16 * (n & 1));
            } else {
                range16(v[n], hi, lo);
            }
        } else {
            unsigned m = FIRST ? top[n] : 0u;
            const bool some = __any(off != 0);
            if (some) clear16(v[n], off);
            if (!FIRST || some) m = top16(mags(v[n]));
            mx = m > mx ? m : mx;
        }
    }
    if constexpr (ZP) keys_of(hi, lo, kmin, kmax);
    const unsigned mykeys = kmin | kmax << 16;
#pragma unroll
    for (int d = 32; d >= R; d >>= 1) {
        if constexpr (ZP) {
            const unsigned a = (unsigned)__shfl_xor((int)kmin, d), b = (unsigned)__shfl_xor((int)kmax, d);
            kmin = a < kmin ? a : kmin;
            kmax = b > kmax ? b : kmax;
        } else {
            const unsigned t = (unsigned)__shfl_xor((int)mx, d);
            mx = t > mx ? t : mx;
        }
    }
    if (lane < R) {
        if constexpr (ZP) {
            red[0][w][r] = kmin;
            red[1][w][r] = kmax;
        } else {
            red[0][w][r] = mx;
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NW; q++) {
        if constexpr (ZP) {
            kmin = red[0][q][r] < kmin ? red[0][q][r] : kmin;
            kmax = red[1][q][r] > kmax ? red[1][q][r] : kmax;
        } else {
            mx = red[0][q][r] > mx ? red[0][q][r] : mx;
        }
    }
    // ---- codes
    int sum = 0;
    int4 rec = make_int4(0, 0, 0, 0);
    double D = 0.0;
    if constexpr (ZP) {
        if (valid && kmin <= kmax) rec = make_const(kmin, kmax);
        D = zp_factor(zp_range((unsigned)rec.x));
    }
    const float f = !ZP && valid ? code_factor(f16_bits_to_float((unsigned short)mx)) : 0.0f;
#pragma unroll
    for (int n = 0; n < N; n++) {
        const int grp = g0 + n * STEP;
        if (store && (n < N - 1 || grp < G)) {
            if constexpr (ZP)
                *(u4*)(dst + (size_t)grp * 512) = zp_codes16(v[n], D, rec.y, (skip[n / 2] >> (16 * (n & 1))) & 0xffffu, sum);
            else
                *(u4*)(dst + (size_t)grp * 512) = codes16(v[n], f);
        }
    }
    if constexpr (ZP) {
#pragma unroll
        for (int d = 32; d >= R; d >>= 1) sum += __shfl_xor(sum, d);
        if (lane < R) s_sum[w][r] = sum;
        if constexpr (FIRST) {  // how many threads have the smallest and the largest, for settle_rows_kernel
            const unsigned long long mine = (R == 8 ? 0x0101010101010101ull : R == 4 ? 0x1111111111111111ull : R == 2 ? 0x5555555555555555ull : ~0ull) << r;
            const int n0 = __popcll(__ballot((mykeys & 0xffffu) == kmin) & mine), n1 = __popcll(__ballot(mykeys >> 16 == kmax) & mine);
            if (lane < R) s_like[w][r] = n0 | n1 << 16;
        }
        __syncthreads();
        if (tid < R && valid) {
            sum = 0;
#pragma unroll
            for (int q = 0; q < NW; q++) sum += s_sum[q][r];
            rec.z = sum;
            if constexpr (FIRST) {
#pragma unroll
                for (int q = 0; q < NW; q++) rec.w += s_like[q][r];
            }
            *zc = rec;
        }
    } else {
        if (tid < R && valid) *cx = (unsigned short)mx;
    }
}

}  // namespace

// ---------------------------------------------------------------------------
// R = 2^LR rows per workgroup of NT threads, N groups of 16 features per thread.  Lane l of a wave holds row l % R: a
// wave's 16-byte stores are R * 16 bytes side by side in the tiled layout, its loads 64 / R * 32 bytes of each row.
//
// Bound by memory where X is large and by its own arithmetic close behind (about 100 instructions for 16 features, a third of
// a large call's time), by one workgroup's chain of loads, two barriers and stores where it is not.  Us, against the floor of
// 2.8 us of launch and drain and 6.9 TB/s, and then both kernels against the four that were there before (colmax_rowmax,
// outlier_lists, row_const, quantize_rows): 4096 x 5120 13.5 (floor 11.9), with settle_rows 18.9 / 33; 2048 x 4096 8.3
// (6.4), 12.5 / 20; 1013 x 4099 7.7 (4.6), 12.8 / 19; 2048 x 49152 70 (46), 80 / 103 (with join_records); zeropoint 2048 x 5120 11.8 (7.4),
// 17.1 / 27.
// The columns that a workgroup's own rows make outliers are left out at once, between the two barriers: where outlier columns
// are outliers in most tokens, eight rows know nearly all of them and settle_rows_kernel has next to nothing to take back.
// ---------------------------------------------------------------------------
struct RowArgs {
    const unsigned short* X;
    int s, h, KT, cap, opad;
    unsigned thr;          // !KNOWN
    const int32_t *idx, *count;  // KNOWN
    unsigned short* rec;   // !KNOWN: a record per workgroup
    unsigned* joined;      // !KNOWN: words of a bitmap of h to clear, or NULL
    int8_t* Xq;
    unsigned short* cx;    // absmax
    int4* zc;              // zeropoint
    unsigned short* Xo;    // KNOWN
};

// waves per SIMD that the registers are to leave room for
constexpr int row_waves(int n) { return n <= 3 ? 8 : n <= 4 ? 7 : n <= 5 ? 6 : n <= 7 ? 5 : 4; }

// RAGGED: h is not a multiple of 128 or X not 16-byte aligned.
template <int N, int LR, int NT, bool ZP, bool KNOWN, bool RAGGED>
__global__ void __launch_bounds__(NT, row_waves(N)) row_codes_kernel(const RowArgs g)
{
    constexpr int R = 1 << LR, STEP = NT >> LR, NW = NT / 64;
    extern __shared__ unsigned bitmap[];  // ceil(h / 32) words
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r = lane & (R - 1);
    const int s = g.s, h = g.h, G = g.KT * 2;
    // Row groups that share 128-byte lines of the codes go to one XCD, one after the other.
    const int nb = gridDim.x, xcd = blockIdx.x & 7;
    const int rg = xcd * (nb >> 3) + min(xcd, nb & 7) + (blockIdx.x >> 3);
    const int i = rg * R + r;
    const bool valid = i < s;  // (a row past the last one: the last one again, its constant and codes zero in the end)
    const unsigned short* row = g.X + (size_t)(valid ? i : s - 1) * h;
    const int g0 = w * (64 >> LR) + (lane >> LR);  // this lane's first group
    int8_t* dst = g.Xq + ((size_t)((rg * R) >> 5) * g.KT) * TILE_BYTES + (((rg * R) & 31) + r) * 16;
    if (rg * R >= s) {  // no such rows (the end of the last row tile): codes 0, no columns
        for (int grp = g0; grp < G; grp += STEP) *(u4*)(dst + (size_t)grp * 512) = (u4)(0u);
        if (!KNOWN && tid == 0) g.rec[(size_t)rg * record_words(g.cap)] = 0;
        return;
    }
    w8 v[N];
    us8 x[N][2];
#pragma unroll
    for (int n = 0; n < N; n++) {
        const int c = first_feature<N, STEP>(g0, n, G);
        x[n][0] = RAGGED ? chunk_load(row, c, h) : *(const us8*)(row + c);
        x[n][1] = RAGGED ? chunk_load(row, c + 8, h) : *(const us8*)(row + c + 8);
    }
    const int nw = (h + 31) >> 5;
    for (int q = tid; q < nw; q += NT) bitmap[q] = 0;
    if (!KNOWN && g.joined && rg == 0)
        for (int q = tid; q < nw; q += NT) g.joined[q] = 0;
    int cnt = 0;
    if constexpr (KNOWN) {
        cnt = *g.count;
        cnt = cnt < 0 ? 0 : (cnt > g.cap ? g.cap : cnt);
    }
    __syncthreads();
    if constexpr (KNOWN) {
        for (int t = tid; t < cnt; t += NT) {
            const unsigned j = (unsigned)g.idx[t];
            if (j < (unsigned)h) atomicOr(&bitmap[j >> 5], 1u << (j & 31));
        }
        for (int q = tid; q < R * g.opad; q += NT) {
            const int rr = q / g.opad, t = q - rr * g.opad, ii = rg * R + rr;
            unsigned short x = 0;
            if (t < cnt && ii < s) {
                const unsigned j = (unsigned)g.idx[t];
                if (j < (unsigned)h) x = g.X[(size_t)ii * h + j];
            }
            if (ii < s) g.Xo[(size_t)ii * g.opad + t] = x;
        }
    }
    // ---- the columns that reach the threshold
    unsigned top[N];  // largest magnitude of each group
    const unsigned thr2 = (g.thr ? g.thr - 1 : 0) * 0x10001u, all = g.thr ? 0u : 0xffffu;
#pragma unroll
    for (int n = 0; n < N; n++) {
        const int c = first_feature<N, STEP>(g0, n, G);
        if (RAGGED && c + 16 > h) {
            x[n][0] = chunk_fix(x[n][0], c, h);
            x[n][1] = chunk_fix(x[n][1], c + 8, h);
        }
        v[n] = words(x[n][0], x[n][1]);
        if (KNOWN) continue;
        const w8 a = mags(v[n]);
        top[n] = top16(a);
        if (top[n] >= g.thr) {
            unsigned f = reach16(a, thr2) | all;
            if (RAGGED) f &= ~past_row(c, h);
            if (!RAGGED || f) atomicOr(&bitmap[c >> 5], f << (c & 31));
        }
        // (opaque: what was worked out from them is not kept for later)
#pragma unroll
        for (int q = 0; q < 8; q++) asm volatile("" : "+v"(v[n].w[q]));
    }
    __syncthreads();
    constants_and_codes<N, LR, NT, ZP, !KNOWN, RAGGED>(v, top, bitmap, h, G, g0, valid, true, dst, g.cx + i, g.zc + i);
    if (!KNOWN && w == NW - 1) write_record(bitmap, nw, lane, g.cap, g.rec + (size_t)rg * record_words(g.cap));
}

// The columns of nrec <= U NT records into the bitmap (cleared here), U records in flight per thread; complete after the barrier
// at the end.
template <int NT, int U>
__device__ __forceinline__ void gather_records(const unsigned short* __restrict__ rec, int nrec, int cap, int nw, unsigned* bitmap)
{
    __shared__ unsigned s_long[U * NT];  // records of more than 31 columns: their numbers, their columns << 16
    __shared__ int s_longs, s_most;
    const int tid = threadIdx.x, pitch = record_words(cap);
    // Most records name the same columns.  Sixteen of them go into the bitmap first, two columns of the first 31 and up to
    // sixteen of the others to a thread; of the rest only those that know more add anything.  (Every record's columns added to
    // the bitmap by its thread, 64 at a time to one word of LDS: 34 us for 2 048 records of 20 columns.)
    us8 a[U], b[U], c[U], d[U];
    auto request = [&](us8* x, int at) {
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int r = tid + NT * u < nrec ? tid + NT * u : nrec - 1;
            x[u] = *(const us8*)(rec + (size_t)r * pitch + min(at, pitch - 8));
        }
    };
    const int e0 = tid & 15;
    const unsigned short* seed = rec + (size_t)((long long)((tid >> 4) & 15) * nrec >> 4) * pitch;
    const int sn = min((int)seed[0], cap + 1);
    const unsigned sj = seed[e0], sk = seed[min(16 + e0, pitch - 1)];
    us8 t0 = (us8)(0), t1 = (us8)(0);
    if (cap > 32) {
        t0 = *(const us8*)(seed + min(32 + 8 * e0, pitch - 8));
        t1 = *(const us8*)(seed + min(160 + 8 * e0, pitch - 8));
    }
    request(a, 0);
    request(b, 8);
    if (U == 1) {  // (few records: columns 16 to 31 along with the others, no round trip of their own)
        request(c, 16);
        request(d, 24);
    }
    for (int q = tid; q < nw; q += NT) bitmap[q] = 0;
    if (tid == 0) s_longs = s_most = 0;
    __syncthreads();
    if (tid < 256) {
        if (e0 > 0 && e0 <= sn) add_bit(bitmap, sj);
        if (16 + e0 <= sn) add_bit(bitmap, sk);
        if (rare(cap > 32 && __any(sn > 31))) {
#pragma unroll
            for (int k = 0; k < 8; k++)
                if (31 + 8 * e0 + k < sn) atomicOr(&bitmap[t0[k] >> 5], 1u << (t0[k] & 31));
        }
        if (rare(cap > 32 && __any(sn > 159))) {
#pragma unroll
            for (int k = 0; k < 8; k++)
                if (159 + 8 * e0 + k < sn) atomicOr(&bitmap[t1[k] >> 5], 1u << (t1[k] & 31));
        }
    }
    __syncthreads();
    // the n columns from word k of a piece on, looked up together; those that are not there are added
    auto look = [&](const us8& piece, int n, int k0) {
        unsigned lack = 0;
#pragma unroll
        for (int k = k0; k < 8; k++) {
            const bool in = k - k0 < n;
            const unsigned j = in ? piece[k] : 0u;
            const unsigned there = bitmap[j >> 5] >> (j & 31);
            lack |= (in ? ~there & 1u : 0u) << k;
        }
        if (rare(__any(lack != 0))) {
#pragma unroll
            for (int k = k0; k < 8; k++)
                if ((lack >> k) & 1u) atomicOr(&bitmap[piece[k] >> 5], 1u << (piece[k] & 31));
        }
    };
    int n[U], most = 0;
#pragma unroll
    for (int u = 0; u < U; u++) {
        n[u] = tid + NT * u < nrec ? min((int)a[u][0], cap + 1) : 0;
        most = n[u] > most ? n[u] : most;
        if (rare(n[u] > 31)) {
            s_long[atomicAdd(&s_longs, 1)] = (unsigned)(tid + NT * u) | (unsigned)n[u] << 16;
            atomicMax(&s_most, n[u]);
        }
    }
    auto look_all = [&](const us8* piece, int e, int k0) {
#pragma unroll
        for (int u = 0; u < U; u++) look(piece[u], n[u] - e, k0);
    };
    look_all(a, 0, 1);
    if (__any(most > 7)) look_all(b, 7, 0);
    if (__any(most > 15)) {
        if (U > 1) {
            request(c, 16);
            request(d, 24);
        }
        look_all(c, 15, 0);
        if (__any(most > 23)) look_all(d, 23, 0);
    }
    __syncthreads();
    // The columns from the 32nd on, in chunks of eight, of which every thread has four in flight.  (A thread for each record, one chunk
    // after the other: calls of 200 columns and 64 output columns 42.7 us instead of 27.8 at 96 x 5120, 90 / 42.6 at 1024 x 8192, 137 / 47.5
    // at 4096 x 5120; a wave for each record, eight at a time: 29.6, 43.2, 48.2, and 46 against 42.7 at 2048 x 4096.)
    const int longs = s_longs, C = (s_most - 31 + 7) >> 3;
    if (!rare(longs > 0)) return;  // uniform
    constexpr int Q = 4;
    const int items = longs * C;  // (record, chunk)
    const unsigned inv = ((1u << 20) + C - 1) / C;  // item / C: exact below 512 * 32
    for (int i0 = tid; i0 < items; i0 += Q * NT) {
        us8 x[Q];
        int left[Q];  // columns of the chunk
#pragma unroll
        for (int q = 0; q < Q; q++) {
            const int i = i0 + q * NT < items ? i0 + q * NT : items - 1;
            const int l = (int)(((unsigned)i * inv) >> 20), c = i - l * C;
            const unsigned r = s_long[l];
            left[q] = i0 + q * NT < items ? (int)(r >> 16) - 31 - 8 * c : 0;
            x[q] = *(const us8*)(rec + (size_t)(r & 0xffffu) * pitch + 32 + (left[q] > 0 ? 8 * c : 0));
        }
#pragma unroll
        for (int q = 0; q < Q; q++)
            if (__any(left[q] > 0)) look(x[q], left[q], 0);
    }
    __syncthreads();
}

// More records than a workgroup joins in little time: 32 of them to a workgroup here, what these find added to one bitmap, which
// row_codes_kernel has cleared.
constexpr int JOIN_SLICE = 32;
__global__ void __launch_bounds__(256) join_records_kernel(const unsigned short* __restrict__ rec, int nrec, int cap, int nw,
                                                           unsigned* __restrict__ joined)
{
    extern __shared__ unsigned bitmap[];
    const int first = blockIdx.x * JOIN_SLICE;
    gather_records<256, 1>(rec + (size_t)first * record_words(cap), min(JOIN_SLICE, nrec - first), cap, nw, bitmap);
    for (int q = threadIdx.x; q < nw; q += 256)
        if (bitmap[q]) atomicOr(&joined[q], bitmap[q]);
}

// Which calls take that kernel: those of many records, and of fewer where they may be long.  Us per call with 512 output columns, so /
// joined by every workgroup for itself: 256 records (512 x 4096), 7 columns 18.2 / 16.8, 40 columns 21.7 / 21.8, 200 columns 29.9 / 35.5;
// 512 records of a buffer of 32 (1024 x 8192), 7 columns 29.6 / 28.3, 31 columns 31.3 / 31.0; of a buffer of 256, 7 columns 29.7 / 28.7, 40
// columns 34.7 / 38.8, 200 columns 45.7 / 60.7.
static bool join_first(int nrec, int cap) { return nrec > (cap > 32 ? 256 : 512); }

// ---------------------------------------------------------------------------
// The outlier set, by all NT threads of a workgroup: s_idx[0 .. min(total, cap)) ascending, from up to 512 records or the joined
// bitmap.  bitmap: ceil(h / 32) words of LDS, left with the bits of all qualifying columns.  Returns their number.
// ---------------------------------------------------------------------------
template <int NT>
__device__ __forceinline__ int outlier_set(const unsigned short* __restrict__ rec, int nrec, const unsigned* __restrict__ joined, int cap,
                                           int nw, unsigned* bitmap, int* s_idx)
{
    __shared__ int s_wsum[NT / 64];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (rare(joined != nullptr)) {
        for (int q = tid; q < nw; q += NT) bitmap[q] = joined[q];
        __syncthreads();
    } else if (NT >= 512 || nrec <= NT) {
        gather_records<NT, 1>(rec, nrec, cap, nw, bitmap);
    } else {
        gather_records<NT, NT >= 512 ? 1 : 2>(rec, nrec, cap, nw, bitmap);
    }
    const int q = (nw + NT - 1) / NT, b0 = tid * q, b1 = min(nw, b0 + q);
    int mine = 0;
    for (int x = b0; x < b1; x++) mine += __popc(bitmap[x]);
    int incl = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int t = __shfl_up(incl, d);
        if (lane >= d) incl += t;
    }
    if (lane == 63) s_wsum[w] = incl;
    __syncthreads();
    int woff = 0, total = 0;
#pragma unroll
    for (int k = 0; k < NT / 64; k++) {
        if (k < w) woff += s_wsum[k];
        total += s_wsum[k];
    }
    int pos = woff + incl - mine;
    if (mine)
        for (int x = b0; x < b1 && pos < cap; x++)
            for (unsigned m = bitmap[x]; m && pos < cap; m &= m - 1) s_idx[pos++] = x * 32 + __ffs(m) - 1;
    __syncthreads();
    return total;
}

// ---------------------------------------------------------------------------
// A workgroup settles 2^lsr rows (one or more times those that row_codes_kernel gave a workgroup), NT >> lsr
// threads to a row; the workgroups past the rows take a column job.  A chain of round trips: records, columns of X and codes,
// stores; 4.4 us for 256 records of 7 columns, 5.2 of 20, 15 of 200 (2.8 of them launch and drain).
// Rows to be made anew are held in registers as there, R at a time and all of a workgroup's lanes on them.  Where that is every
// row, calls with 64 output columns, us (one row after the other / the kernels of prepass.hip, zeropoint.hip): 96 x 5120 15.8
// (27.8 / 16.5), 1024 x 8192 31.1 (44.5 / 35.1), 4096 x 5120 37.7 (52.2 / 48.0), 4096 x 12288 81.3 (105.4 / 84.0), 2048 x 49152 206
// (296 / 170), zeropoint 512 x 4096 19.2 (32.0 / 22.6), 2048 x 5120 33.7 (47.8 / 34.5), 1024 x 28672 80.8 (110.5 / 71.6).
// ---------------------------------------------------------------------------
constexpr int MAX_SR = 8;
struct SettleArgs {
    const unsigned short* X;
    int s, h, KT, cap, opad, nrec;
    int lsr, nb;  // rows of a workgroup (log2), workgroups of rows
    const unsigned short* rec;
    const unsigned* joined;  // or NULL
    int32_t *idx, *count, *status;
    int8_t* Xq;
    unsigned short* cx;
    int4* zc;
    unsigned short* Xo;
    ColumnJob cj;
};

template <int N, int LR, int NT, bool ZP>
__global__ void __launch_bounds__(NT, 4) settle_rows_kernel(const SettleArgs a)
{
    constexpr int R = 1 << LR, STEP = NT >> LR;
    extern __shared__ unsigned bitmap[];
    __shared__ int s_idx[JOB_MAX_CAP];
    __shared__ unsigned s_need;
    __shared__ int s_gone[ZP ? 3 : 1][MAX_SR];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int s = a.s, h = a.h, KT = a.KT, opad = a.opad, nw = (h + 31) >> 5;
    // (all arguments requested at once: behind the first branch they would be another round trip)
    asm volatile("" ::"s"(a.X), "s"(a.rec), "s"(a.joined), "s"(a.nrec), "s"(a.cap), "s"(a.opad), "s"(a.KT), "s"(a.idx), "s"(a.count), "s"(a.Xq),
                 "s"(ZP ? (const void*)a.zc : (const void*)a.cx), "s"(a.Xo));
    const int tpr = NT >> a.lsr, tr = tid >> (__builtin_ctz(NT) - a.lsr), t1 = tid & (tpr - 1);  // this thread's row of the workgroup, its first outlier column
    const bool job = (int)blockIdx.x >= a.nb;
    // (the rows on the XCD whose L2 may still have their codes)
    const int xcd = blockIdx.x & 7, b = job ? 0 : xcd * (a.nb >> 3) + min(xcd, a.nb & 7) + (blockIdx.x >> 3);
    const int i0 = b << a.lsr, i = i0 + tr;
    if (i0 >= s) return;  // the end of the last row tile
    const bool mine = i < s;
    unsigned m1 = 0;
    int4 z = make_int4(0, 0, 0, 0);
    if constexpr (ZP)
        z = a.zc[mine ? i : 0];
    else
        m1 = a.cx[mine ? i : 0];
    if (tid == 0) s_need = 0;
    if (ZP && tid < 3 * MAX_SR) s_gone[tid / MAX_SR][tid % MAX_SR] = 0;
    const int total = outlier_set<NT>(a.rec, a.nrec, a.joined, a.cap, nw, bitmap, s_idx);
    const int cnt = total < a.cap ? total : a.cap;
    if (rare(job)) {
        if (tid >= 256) return;
        const int jb = (int)blockIdx.x - a.nb, parts = a.cj.pitch >> 8, j = (jb % parts) * 256 + tid;
        if constexpr (ZP)
            zp_col_factors(a.cj.Wq, (const int4*)a.cj.wconst, h, a.cj.o, KT, s_idx, cnt, a.cj.pitch, (double*)a.cj.out, j);
        else if (j < a.cj.o)
            rebuild_rows(a.cj.Wq, (const unsigned short*)a.cj.wconst, h, a.cj.o, KT, s_idx, cnt, jb / parts * JOB_SLOTS,
                         min(jb / parts * JOB_SLOTS + JOB_SLOTS, opad), (unsigned short*)a.cj.out, j);
        return;
    }
    if (b == 0) {
        for (int t = tid; t < cnt; t += NT) a.idx[t] = s_idx[t];
        if (tid == 0) {
            *a.count = cnt;
            if (a.status) *a.status = total > a.cap ? 1 : 0;
        }
    }
    // An entry below the threshold in an outlier column went into its row's constants and has a code if no row of its
    // workgroup reached the threshold there.  Where it is an extreme of the row (its code is then 127 in magnitude) and
    // the row may have no other like it, the row is made anew; else its code goes.
    // (Zeropoint: a constant row has no codes to say so, and with no ordinary column left its record is zero.)
    const bool all = total > a.cap || (ZP && cnt == h);
    const unsigned short* row = a.X + (size_t)(mine ? i : 0) * h;
    int8_t* q = a.Xq + (size_t)(mine ? i >> 5 : 0) * KT * TILE_BYTES;
    auto take_back = [&](auto in_flight) {
        constexpr int K = in_flight;
        for (int base = 0; base < opad; base += K * tpr) {
            unsigned short x[K];
            int code[K];
            int8_t* at[K];
#pragma unroll
            for (int u = 0; u < K; u++) {
                const int t = base + u * tpr + t1;
                if (base + u * tpr >= cnt) continue;  // uniform
                const int j = t < cnt ? s_idx[t] : 0;
                at[u] = q + (size_t)(j >> 5) * TILE_BYTES + tile_byte(i & 31, j & 31);
                x[u] = row[j];
                code[u] = *at[u];
            }
#pragma unroll
            for (int u = 0; u < K; u++) {
                const int t = base + u * tpr + t1;
                if (base + u * tpr >= opad) continue;
                const bool in = t < cnt;
                if (mine && t < opad) a.Xo[(size_t)i * opad + t] = in ? x[u] : (unsigned short)0;
                if (rare(mine && in && code[u] != 0)) {
                    if constexpr (ZP) {  // the sum of the codes that go, entries that are the smallest, the largest
                        atomicAdd(&s_gone[0][tr], code[u]);
                        if (code[u] == -127) atomicAdd(&s_gone[1][tr], 1);
                        if (code[u] == 127) atomicAdd(&s_gone[2][tr], 1);
                    } else {
                        if ((unsigned)(x[u] & 0x7fff) == m1) atomicOr(&s_need, 1u << tr);
                    }
                    *at[u] = 0;
                }
            }
        }
    };
    if (opad <= tpr)
        take_back(std::integral_constant<int, 1>());
    else
        take_back(std::integral_constant<int, 4>());
    __syncthreads();
    if constexpr (ZP) {
        if (t1 == 0 && mine) {
            const int nlo = s_gone[1][tr], nhi = s_gone[2][tr];
            if ((nlo > 0 && nlo >= (z.w & 0xffff)) || (nhi > 0 && nhi >= (int)((unsigned)z.w >> 16))) {
                atomicOr(&s_need, 1u << tr);
            } else if (!all) {
                z.z -= s_gone[0][tr];
                z.w = 0;
                a.zc[i] = z;
            }
        }
        __syncthreads();
    }
    const unsigned again = all ? (1u << (1 << a.lsr)) - 1 : s_need;
    if (!rare(again != 0)) return;
    // ---- rows to be made anew
    if (total > a.cap) {  // the columns that the buffer takes, in place of all
        for (int x = tid; x < nw; x += NT) bitmap[x] = 0;
        __syncthreads();
        for (int t = tid; t < cnt; t += NT) atomicOr(&bitmap[s_idx[t] >> 5], 1u << (s_idx[t] & 31));
    }
    const int r = lane & (R - 1), G = KT * 2;
    for (int r0 = 0; r0 < 1 << a.lsr; r0 += R) {
        if (!((again >> r0) & ((1u << R) - 1))) continue;
        __syncthreads();  // the bitmap is there; the rows before have left LDS
        const int ir = i0 + r0 + r;
        int g0 = w * (64 >> LR) + (lane >> LR);
        asm volatile("" : "+v"(g0));  // (opaque: what follows from it is worked out here, not kept from one turn to the next)
        const bool act = ((again >> (r0 + r)) & 1u) && ir < s;
        us8 x[N][2];
        if (act) {
            const unsigned short* row2 = a.X + (size_t)ir * h;
#pragma unroll
            for (int n = 0; n < N; n++) {
                const int c = first_feature<N, STEP>(g0, n, G);
                x[n][0] = chunk_load(row2, c, h);
                x[n][1] = chunk_load(row2, c + 8, h);
            }
        }
        w8 v[N];
        unsigned none[N];
#pragma unroll
        for (int n = 0; n < N; n++) {
            const int c = first_feature<N, STEP>(g0, n, G);
            if (c + 16 > h) {
                x[n][0] = chunk_fix(x[n][0], c, h);
                x[n][1] = chunk_fix(x[n][1], c + 8, h);
            }
            v[n] = words(x[n][0], x[n][1]);
        }
        constants_and_codes<N, LR, NT, ZP, false, true>(v, none, bitmap, h, G, g0, act, act,
                                                        a.Xq + (size_t)(ir >> 5) * KT * TILE_BYTES + (ir & 31) * 16, a.cx + ir, a.zc + ir);
    }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
struct RowShape { int lr, n, nt; };
// Rows per workgroup (log2), groups per thread and threads.  Eight rows where that gives the chip at least one workgroup per
// compute unit, two or one below, so that more of them are in flight; as many more as fill 256 threads where rows are short; and
// fewer where the registers do not hold them (n <= 8).  One row: more threads sooner, its latency is what counts.
static RowShape row_shape(int s, int h)
{
    const int G = k_tiles(h) * 2;
    int lr = s >= 2048 ? 3 : s >= 512 ? 1 : 0;
    while (lr < 3 && (G << lr) < 256) lr++;
    while (lr > 1 && (G << lr) > 512 * 5) lr--;
    const int items = G << lr;
    const int nt = items <= (lr == 1 ? 1536 : lr ? 1024 : 512) ? 256 : items <= 512 * (lr ? 5 : 8) ? 512 : 1024;
    return {lr, (items + nt - 1) / nt, nt};
}

// The same for settle_rows_kernel.  In place of eight or four rows in 512 threads half as many in 256, the registers per lane the same: a
// thread more than a row's 32 outlier columns only waits.  Calls with 7 columns, us, so / in 512 threads: 2048 x 4096 x 4096 45.1 /
// 45.6, 4096 x 5120 x 64 27.1 / 27.4.  Not for longer buffers (2048 x 4096 x 64, 200 columns 44.5 / 41.9), nor in place of 1 024 threads, which hold
// rows of many features (2048 x 49152 x 64 with every row made anew 237 / 207, with 7 columns no difference).
static RowShape settle_shape(int s, int h, int cap)
{
    RowShape q = row_shape(s, h);
    if (cap <= 32 && q.nt == 512 && q.lr > 1) { q.nt = 256; q.lr--; }
    return q;
}

// the joined bitmap's place in front of the records
static size_t joined_bytes(int h, int nrec, int cap) { return join_first(nrec, cap) ? (size_t)((h + 255) / 256) * 32 : 0; }

// Which calls come here, us per call, here / with the kernels of prepass.hip and zeropoint.hip (which keep the rest):
//   up to 128 tokens, 16-bit weights: 16 x 4096 x 2048 15.0 / 17.7, 32 x 4100 x 4100 16.1 / 19.3, 16 x 12288 x 49152 99.1 / 101.1, 33 x 4096
//     x 4096 15.3 / 16.0, 96 x 5120 x 15360 26.3 / 28.9, 2 x 20480 x 2048 22.8 / 23.7, 40 x 20480 x 512 25.8 / 26.4; with more features
//     one compute unit has too much of a row: 2 x 37120 x 2048 32.2 / 31.3, 100 x 24576 x 1024 31.0 / 30.3, 128 x 49152 x 2048 53.3 / 49.4
//   the same without 16-bit weights, where the rebuilt rows of W wait for the records: 16 x 4096 x 4096 14.7 / 17.3, 32 x 4096 x 4096
//     18.6 / 19.1, 96 x 2048 x 4096 15.6 / 16.2, 128 x 4096 x 4096 17.7 / 17.6, but 32 x 12288 x 2048 22.3 / 21.8, 60 x 8192 x 28672 49.9 / 48.7,
//     and from 33 to 64 tokens 33 x 1024 x 4096 13.7 / 13.3, 48 x 4096 x 4096 16.2 / 15.5, 64 x 4096 x 16384 25.7 / 25.0, with 200 columns
//     64 x 4096 x 4096 35.0 / 30.1
//   zeropoint, up to 128 tokens: 2 x 1024 x 2048 14.2 / 17.1, 32 x 4096 x 2048 15.5 / 21.8, 64 x 4096 x 4096 16.2 / 19.8, 2 x 12288 x 2048
//     20.1 / 22.2, 16 x 37120 x 2048 36.5 / 38.7, 40 x 49152 x 512 52.0 / 54.7, 48 x 12288 x 4096 with 20 columns 26.3 / 26.0 the least;
//     but 2 x 37120 x 2048 34.9 / 33.2, 12 x 20480 x 2048 with 20 columns 28.9 / 28.2, 3 x 14591 x 1240 with 16 24.3 / 23.5
//   above: 256 x 4096 x 4096 19.8 / 24.8, 200 x 49152 x 512 53.7 / 53.7, 2047 x 5120 x 1024 34.8 / 40.3, 4000 x 1000 x 1000 21.8 /
//     32.1, zeropoint 4096 x 1024 x 1024 26.5 / 37.5
//   the columns known: 20 x 4096 26.9 / 31.7 (three calls), 4096 x 5120 47.3 / 53.3; not where a second row of many features falls
//     to some compute units (300 x 49152 64.9 / 63.7; 30 x 49152 50.7 / 53.1, 700 x 49152 99.8 / 100.2)
// Up to 2 048 records: 16 384 tokens up to 5 120 features, 8 192 up to 10 240, 4 096 above (row_shape).  Longer X was not measured here since
// join_records_kernel took the join off settle_rows_kernel's workgroups.
bool row_codes_takes(int s, int h, int cap, RowCall call, size_t room)
{
    if (h < 8 || h > 65536 || cap > JOB_MAX_CAP) return false;
    if (call == RowCall::known) return !(h > 32768 && s > 256 && s < 512);
    if (call == RowCall::zeropoint ? s < 16 && h > 12288 : s <= 128 && h > (call == RowCall::rebuilt ? 4096 : 20480)) return false;
    if (call == RowCall::rebuilt && s > 32 && s <= 64) return false;
    const int nrec = (row_tiles(s) * 32) >> row_shape(s, h).lr;
    return nrec <= 2048 && (size_t)nrec * record_words(cap) * 2 + joined_bytes(h, nrec, cap) <= room;
}

// f(threads, log2 of the rows of a workgroup, groups per thread) of q, as constants
template <class F>
static hipError_t with_shape(const RowShape& q, F f)
{
    switch (q.nt + q.lr * 16 + q.n) {
#define ROWS(NT, LR, N)                                                                                                             \
    case NT + LR * 16 + N:                                                                                                          \
        f(std::integral_constant<int, NT>(), std::integral_constant<int, LR>(), std::integral_constant<int, N>());                  \
        break
        ROWS(256, 3, 1); ROWS(256, 3, 2); ROWS(256, 3, 3); ROWS(256, 3, 4);
        ROWS(256, 2, 1); ROWS(256, 2, 2); ROWS(256, 2, 3); ROWS(256, 2, 4); ROWS(256, 2, 5);
        ROWS(256, 1, 1); ROWS(256, 1, 2); ROWS(256, 1, 3); ROWS(256, 1, 4); ROWS(256, 1, 5); ROWS(256, 1, 6);
        ROWS(256, 0, 1); ROWS(256, 0, 2);
        ROWS(512, 3, 3); ROWS(512, 3, 4); ROWS(512, 3, 5);
        ROWS(512, 2, 3); ROWS(512, 2, 4); ROWS(512, 2, 5);
        ROWS(512, 1, 4); ROWS(512, 1, 5);
        ROWS(512, 0, 2); ROWS(512, 0, 3); ROWS(512, 0, 4); ROWS(512, 0, 5); ROWS(512, 0, 6); ROWS(512, 0, 7); ROWS(512, 0, 8);
        ROWS(1024, 1, 3); ROWS(1024, 1, 4); ROWS(1024, 1, 5); ROWS(1024, 1, 6); ROWS(1024, 1, 7); ROWS(1024, 1, 8);
#undef ROWS
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <bool ZP, bool KNOWN>
static hipError_t launch_row_codes(const RowArgs& g, hipStream_t st)
{
    const RowShape q = row_shape(g.s, g.h);
    const int nb = (row_tiles(g.s) * 32) >> q.lr;
    const size_t shm = (size_t)((g.h + 31) / 32) * 4;
    const bool ragged = g.h % 128 != 0 || ((uintptr_t)g.X & 15) != 0;
    return with_shape(q, [&](auto nt, auto lr, auto n) {
        if (ragged)
            row_codes_kernel<n(), lr(), nt(), ZP, KNOWN, true><<<nb, nt(), shm, st>>>(g);
        else
            row_codes_kernel<n(), lr(), nt(), ZP, KNOWN, false><<<nb, nt(), shm, st>>>(g);
    });
}

template <bool ZP>
static hipError_t launch_settle(const SettleArgs& a, int jobs, hipStream_t st)
{
    return with_shape(settle_shape(a.s, a.h, a.cap), [&](auto nt, auto lr, auto n) {
        settle_rows_kernel<n(), lr(), nt(), ZP><<<a.nb + jobs, nt(), (size_t)((a.h + 31) / 32) * 4, st>>>(a);
    });
}

hipError_t launch_prepass_rows(const void* X, int s, int h, unsigned thr, void* records, int32_t* idx, int cap,
                               int32_t* count, int32_t* status, int8_t* Xq, unsigned short* cx, int4* zc,
                               unsigned short* Xo, const ColumnJob* cj, hipStream_t st)
{
    const int lr = row_shape(s, h).lr, nrec = (row_tiles(s) * 32) >> lr, nw = (h + 31) / 32;
    unsigned* joined = join_first(nrec, cap) ? (unsigned*)records : nullptr;
    const RowArgs g = {(const unsigned short*)X, s, h, k_tiles(h), cap, opad_of(cap), thr, nullptr, nullptr,
                       (unsigned short*)((char*)records + joined_bytes(h, nrec, cap)), joined, Xq, cx, zc, nullptr};
    hipError_t e = zc ? launch_row_codes<true, false>(g, st) : launch_row_codes<false, false>(g, st);
    if (e != hipSuccess) return e;
    if (joined) {
        join_records_kernel<<<(nrec + JOIN_SLICE - 1) / JOIN_SLICE, 256, nw * 4, st>>>(g.rec, nrec, cap, nw, joined);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    int lsr = lr;  // more rows to a workgroup while that leaves one for every compute unit: each joins the records for itself
    while ((1 << lsr) < MAX_SR && s >= 256 << (lsr + 1)) lsr++;
    const ColumnJob job = cj ? *cj : ColumnJob{nullptr, nullptr, nullptr, 0, 0};
    const int parts = zc ? 1 : (g.opad + JOB_SLOTS - 1) / JOB_SLOTS;
    const SettleArgs a = {g.X, s, h, g.KT, cap, g.opad, nrec, lsr, (row_tiles(s) * 32) >> lsr, g.rec, joined, idx, count, status, Xq, cx, zc, Xo, job};
    return zc ? launch_settle<true>(a, job.pitch / 256 * parts, st) : launch_settle<false>(a, job.pitch / 256 * parts, st);
}

hipError_t launch_quantize_rows_known(const void* X, int s, int h, const int32_t* idx, const int32_t* count, int cap,
                                      int8_t* Xq, unsigned short* cx, int4* zc, unsigned short* Xo, hipStream_t st)
{
    const RowArgs g = {(const unsigned short*)X, s, h, k_tiles(h), cap, opad_of(cap), 0, idx, count, nullptr, nullptr, Xq, cx, zc, Xo};
    return zc ? launch_row_codes<true, true>(g, st) : launch_row_codes<false, true>(g, st);
}

}  // namespace llmint8
