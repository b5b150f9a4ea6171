// fp32 products on the bf16 matrix pipe (included by the GraphSAGE and GAT translation units inside
// their anonymous namespaces, after gemm_common.h); the method is published: Henry, Tang, Heinecke, "Leveraging
// the bfloat16 artificial intelligence datatype for higher-precision computations", ARITH 2019.
//
// The fp32 MFMA reaches a sixteenth of the bf16 rate, and the products of a layer were bound by it: a
// 24k x 200 x 256 product took 32 us for 15 us of fp32 matrix time and 7 us of memory traffic.  A float
// is the exact sum of three bfloat16 values,
//     x = x1 + x2 + x3,   x1 = bf16(x), x2 = bf16(x - x1), x3 = x - x1 - x2,
// (round to nearest: 8 + 8 + 8 significand bits, every difference is exact), and a product of bfloat16
// values is exact in float.  Of the nine partial products the six larger ones are summed,
//     x1 y1  +  (x1 y2 + x2 y1 + x2 y2 + x1 y3 + x3 y1),
// the three dropped ones reach 2^-24 |x y| together (x = y = 1 + 2^-8 - 2^-17).  The leading products and
// the five small ones have an accumulator each, so that the large sum is rounded once per 16 k (an fp32 MFMA
// chain rounds it once per 2).  Against 64-bit sums of normally distributed operands, 2-norm in units of 2^-24, here
// and the fp32 MFMA tiles: 8 k 0.49 / 0.91, 64 k 0.80 / 1.42, 256 k 1.07 / 4.8, 512 k 1.28 / 3.5.
// bfloat16 ends at 2^-133 and float at 2^-149, so an operand is split times 2^16: the last bit of every float
// then is a bfloat16 (the matrix unit keeps subnormals), and the sum is brought back by 2^-32.  Unscaled,
// operands below 2^-110 lost their last part, then the second: 440 units of 2^-24 in the results at 1e-36.
// Of one or two products the dropped terms are a larger error than the saved roundings of an fp32 chain (at worst
// 1.45 units of 2^-24 against 1, and 2.3 against 1.85; of three 1.9 against 2.2): those go through the fp32 MFMA.
// Values the split cannot carry (infinities, NaN, operands of 2^112 and results of 2^96 and more) make the
// scaled result non-finite: a wave that finds one in its tile forms the tile again with fp32 MFMAs straight
// from global memory.
#pragma once

#include "split_rules.h"

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

constexpr int SNT = 256;                // threads of a workgroup: four waves
constexpr int SPLIT_MIN_K = 3;          // shorter contractions are formed with fp32 MFMAs
constexpr float SPLIT_SCALE = 0x1p16f, SPLIT_UNSCALE = 0x1p-32f;        // of an operand, of a product of two

__device__ __forceinline__ uint32_t cvt2bf(float a, float b) {      // round to nearest even, a in the low half
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){a, b}, bf16x2_t));
}
// two values -> one word (two bfloat16) of each of the three parts
__device__ __forceinline__ void split2(float a, float b, uint32_t &p1, uint32_t &p2, uint32_t &p3) {
    p1 = cvt2bf(a, b);
    a -= __uint_as_float(p1 << 16); b -= __uint_as_float(p1 & 0xFFFF0000u);
    p2 = cvt2bf(a, b);
    a -= __uint_as_float(p2 << 16); b -= __uint_as_float(p2 & 0xFFFF0000u);
    p3 = cvt2bf(a, b);
}
__device__ __forceinline__ void split8(const float (&v)[8], uint4 (&p)[3]) {
    split2(v[0], v[1], p[0].x, p[1].x, p[2].x);
    split2(v[2], v[3], p[0].y, p[1].y, p[2].y);
    split2(v[4], v[5], p[0].z, p[1].z, p[2].z);
    split2(v[6], v[7], p[0].w, p[1].w, p[2].w);
}
__device__ __forceinline__ floatx16 mfma_bf(const uint4 &a, const uint4 &b, const floatx16 &c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}
__device__ __forceinline__ floatx16 zero16() {
    floatx16 z;
#pragma unroll
    for (int r = 0; r < 16; ++r) z[r] = 0.f;
    return z;
}
__device__ __forceinline__ bool finite16(const floatx16 &v) {
    bool ok = true;
#pragma unroll
    for (int r = 0; r < 16; ++r) ok = ok && fabsf(v[r]) < INFINITY;
    return ok;
}

// ---- operand laid out once per call: the weights --------------------------------------------------
// Matrix B (k x n) as the fragments a wave feeds the MFMA: block (nb, ks) covers 32 columns x 16 k in
// three planes of 64 lanes x 16 bytes (of the scaled values); lane l holds column 32 nb + l % 32 and the eight k of granule
// 2 (ks % 2) + l / 32 of k-tile ks / 2.  Granule g of a tile of 32 k is k = 4 g .. 4 g + 3 and
// 16 + 4 g .. 16 + 4 g + 3: the four threads that fetch a row's granules then read 64 consecutive bytes
// with one instruction.  Past the matrix: zeros.
__host__ __device__ inline int split_halves(int K) { return 2 * ((K + 31) / 32); }      // 16-k blocks, in pairs
__host__ __device__ inline int64_t split_frag_words(int K, int N) {     // 16-byte words
    return (int64_t)((N + 31) / 32) * split_halves(K) * 192;
}
__device__ __forceinline__ int granule_k(int g, int j) { return 4 * g + j + (j < 4 ? 0 : 12); }
template <class Get>
__device__ __forceinline__ void split_frag_fill(uint4 *frag, int K, int N, int64_t x, int64_t stride, const Get &get) {
    const int KS = split_halves(K);
    const int64_t items = (int64_t)((N + 31) / 32) * KS * 64;
    for (; x < items; x += stride) {
        const int lane = (int)(x & 63);
        const int blk = (int)(x >> 6), nb = blk / KS, ks = blk - nb * KS;
        const int n = 32 * nb + (lane & 31), k0 = 32 * (ks >> 1), g = 2 * (ks & 1) + (lane >> 5);
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = get(min(k0 + granule_k(g, j), K - 1), min(n, N - 1));
        // (no condition around a load: the scaling would follow it there, and a wait in front of that, one load after the
        // other: 11 -> 24 us for the weights of a 128 x 256 x 47 model)
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = (n < N && k0 + granule_k(g, j) < K) ? v[j] * SPLIT_SCALE : 0.f;
        uint4 p[3];
        split8(v, p);
#pragma unroll
        for (int q = 0; q < 3; ++q) frag[(int64_t)blk * 192 + q * 64 + lane] = p[q];
    }
}

// A: rows x K floats at row stride ld.  VA = 4: rows are 16-byte aligned and K is a multiple of 4.
struct SplitA { const float *p; int64_t ld; int rows; int K; };
// B: fragments of K x N, and the matrix itself: element (k, n) at ref[k * rk + n * rn]
struct SplitB { const uint4 *frag; const float *ref; int64_t rk, rn; int N; };

// The products of k_begin .. k_end - 1 with fp32 MFMAs, sums of 16 k added up (a single chain of 64 k rounded more
// often than the fp32 tiles whose waves each took a part of the contraction: 2.4 units of 2^-24 against 1.4).
template <class GetA, class GetB>
__device__ __forceinline__ floatx16 exact_sum(int k_begin, int k_end, int half, const GetA &get_a, const GetB &get_b) {
    floatx16 sum = zero16();
#pragma unroll 1
    for (int k0 = k_begin; k0 < k_end; k0 += 16) {
        floatx16 part = zero16();
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int k = k0 + 8 * half + q;
            part = __builtin_amdgcn_mfma_f32_32x32x2f32(get_a(k), get_b(k), part, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) sum[r] += part[r];
    }
    return sum;
}
// one 32 x 32 block with fp32 MFMAs from global memory (non-finite results and short contractions only)
__device__ __forceinline__ floatx16 split_exact_block(const SplitA &a, const SplitB &b, int m, int n, int half) {
    const float *ap = a.p + (int64_t)min(m, a.rows - 1) * a.ld;
    const float *bp = b.ref + (int64_t)min(n, b.N - 1) * b.rn;
    const int K = a.K;
    return exact_sum(0, K, half, [&](int k) { return k < K ? ap[k] : 0.f; }, [&](int k) { return k < K ? bp[k * b.rk] : 0.f; });
}

// Epilogues: out (row 0 of the output, row stride ld) and what becomes of an element; side() is an input of
// value() that depends on the column, the row or both (SIDE).  advance(): the same some output columns on.
enum SplitSide { SIDE_NONE, SIDE_COL, SIDE_ROW, SIDE_ELEM };
struct SplitEpiBias {       // v + vec[n], rectified if relu
    static constexpr SplitSide SIDE = SIDE_COL;
    float *out; int ld; const float *vec; int relu;
    __device__ __forceinline__ void advance(int cols) { out += cols; vec += cols; }
    __device__ __forceinline__ float side(int, int n) const { return vec[n]; }
    __device__ __forceinline__ float value(float v, float x, int) const { v += x; return (relu && v < 0.f) ? 0.f : v; }
};
// the same, rectified, and a bit per element that says whether it is above zero (row stride ldb words of 32 columns): the
// backward pass asks for nothing else of the activations.  Tiled forms only.
struct SplitEpiRelu : SplitEpiBias { uint32_t *bits; int ldb; };
template <class EF> constexpr bool split_keeps_bits = false;
template <> constexpr bool split_keeps_bits<SplitEpiRelu> = true;
// (the instruction has no builtin; as inline assembly the compiler would not keep it from the comparison whose mask it reads)
extern "C" __device__ unsigned write_lane(unsigned value, unsigned lane, unsigned old) __asm("llvm.amdgcn.writelane.i32");
// Which rows' words the ballots of a 32 x 32 block of accumulators hold: register r, low half row 8 (r / 4) + r % 4, high half
// four rows on; lane k gets the word of row k.
__device__ __forceinline__ void keep_ballot(unsigned &word, const int r, bool above) {
    const uint64_t b = __ballot(above);
    word = write_lane((unsigned)b, (r >> 2) * 8 + (r & 3), word);
    word = write_lane((unsigned)(b >> 32), (r >> 2) * 8 + 4 + (r & 3), word);
}
struct SplitEpiScale {      // input gradients: v * vec[m] in the columns from `first` on
    static constexpr SplitSide SIDE = SIDE_ROW;
    float *out; int ld; const float *vec; int first;
    __device__ __forceinline__ void advance(int cols) { out += cols; }
    __device__ __forceinline__ float side(int m, int) const { return vec[m]; }
    __device__ __forceinline__ float value(float v, float x, int n) const { return n >= first ? v * x : v; }
};

// ------------------------------------------------------------------------------------------
// C[rows x N] = A * B, persistent workgroups over tiles of 64 rows x 128 columns: four waves of 64 x 32.
// A is split on its way into LDS (a thread takes 8 consecutive k of a row: 44 vector instructions); B's
// fragments come from the L2 straight into registers, half a k-tile of 32 ahead.  Two LDS stages, one
// barrier per k-tile, two k-tiles of A in flight in registers, and a tile's first ones are asked for before
// the tile in front is stored, so that neither the memory latency nor the drain of the stores stands
// between two tiles.  The stores are bounds-checked buffer stores: with a branch around them the number of
// operations in flight is unknown at compile time, and every wait for a load waits for all stores.
// LDS: [plane][row][four 16-byte granules of 8 k], granule g of a row at g ^ ((row >> 2) & 3): sixteen
// consecutive rows of one granule column fall into sixteen different bank groups.
// ------------------------------------------------------------------------------------------
// Tiles of 64 x 64, waves of 32 x 32: for outputs of at most 64 columns, and where wide tiles leave compute units idle
// (see split_rules.h).
template <int MI_, int WN_>
struct SplitTile {
    static constexpr int MI = MI_, WN = WN_, BM = 64, BN = 32 * WN_, OCC = 3;
    static_assert(MI_ * (SNT / 64) == 2 * WN_ && BM * 4 == SNT, "64 rows: a piece (8 k of a row) per thread");
};
using SplitWide = SplitTile<2, 4>;
using SplitNarrow = SplitTile<1, 2>;

constexpr int SPLIT_LDS = 2 * 3 * 64 * 4;        // 16-byte words that a workgroup of any form needs
template <class T, int VA, class EF>
__device__ __forceinline__ void split_rows_product(const SplitA &a, const SplitB &b, const EF &epi, uint4 *lds) {
    constexpr int MI = T::MI, BM = T::BM, BN = T::BN;
    static_assert(2 * 3 * BM * 4 <= SPLIT_LDS, "LDS");
    uint4 (*sA)[3][BM * 4] = reinterpret_cast<uint4 (*)[3][BM * 4]>(lds);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31, wc = wave % T::WN, wr = wave / T::WN * 32 * MI;
    const int K = a.K, KT = (K + 31) / 32, KS = 2 * KT, NB32 = (b.N + 31) / 32;
    const int tiles_m = (a.rows + BM - 1) / BM, tiles_n = (b.N + BN - 1) / BN;
    const int total = ((tiles_m + 7) & ~7) * tiles_n;
    const int prow = tid >> 2, pg = tid & 3, at = prow * 4 + (pg ^ ((prow >> 2) & 3));
    const int sw = (l32 >> 2) & 3;

    struct RegA { float v[8]; };
    struct RegB { uint4 q[3]; };
    struct At { const float *a; const uint4 *b; int m0, n0; };       // a tile, as this thread sees it
    auto tile_at = [&](int gid, At &x) __attribute__((always_inline)) {
        const bool some = next_tile<T>(gid, tiles_m, tiles_n, x.m0, x.n0);
        x.a = a.p + (int64_t)min(x.m0 + prow, a.rows - 1) * a.ld;
        x.b = b.frag + (int64_t)min(x.n0 / 32 + wc, NB32 - 1) * KS * 192 + lane;
        return some;
    };
    // (addresses past K are clamped: no condition around a load, and none on the value, which meets zeros of B; one
    // that is not finite makes its row's results NaN, and they are those of a row with such a value anyway)
    auto load_a = [&](RegA &r, const At &x, int t) __attribute__((always_inline)) {
        const int k0 = 32 * t + 4 * pg;
        if (VA == 4) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const float4 f = *reinterpret_cast<const float4 *>(x.a + min(k0 + 16 * j, K - 4));
                r.v[4 * j] = f.x; r.v[4 * j + 1] = f.y; r.v[4 * j + 2] = f.z; r.v[4 * j + 3] = f.w;
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) r.v[j] = x.a[min(32 * t + granule_k(pg, j), K - 1)];
        }
    };
    auto land_a = [&](RegA &r, int st) __attribute__((always_inline)) {
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = r.v[j] * SPLIT_SCALE;
        uint4 p[3];
        split8(v, p);
#pragma unroll
        for (int q = 0; q < 3; ++q) sA[st][q][at] = p[q];
    };
    auto load_b = [&](RegB &r, const At &x, int ks) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 3; ++q) r.q[q] = x.b[min(ks, KS - 1) * 192 + q * 64];
    };
    floatx16 hi[MI], lo[MI];
    auto multiply = [&](const RegB &r, int s, int st) __attribute__((always_inline)) {
        uint4 f[MI][3];
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int i = 0; i < MI; ++i) f[i][q] = sA[st][q][(wr + 32 * i + l32) * 4 + ((2 * s + half) ^ sw)];
#pragma unroll
        for (int i = 0; i < MI; ++i) hi[i] = mfma_bf(f[i][0], r.q[0], hi[i]);
#pragma unroll
        for (int i = 0; i < MI; ++i) lo[i] = mfma_bf(f[i][0], r.q[2], lo[i]);
#pragma unroll
        for (int i = 0; i < MI; ++i) lo[i] = mfma_bf(f[i][0], r.q[1], lo[i]);
#pragma unroll
        for (int i = 0; i < MI; ++i) lo[i] = mfma_bf(f[i][1], r.q[0], lo[i]);
#pragma unroll
        for (int i = 0; i < MI; ++i) lo[i] = mfma_bf(f[i][1], r.q[1], lo[i]);
#pragma unroll
        for (int i = 0; i < MI; ++i) lo[i] = mfma_bf(f[i][2], r.q[0], lo[i]);
    };
    RegA ra0, ra1;
    RegB rb0, rb1;
    At cur, nxt;
    int gid = blockIdx.x;
    for (; gid < total; gid += gridDim.x)
        if (tile_at(gid, cur)) break;
    if (gid >= total) return;
    load_b(rb0, cur, 0);
    load_a(ra1, cur, 0);
    load_a(ra0, cur, 1);
    for (;;) {
#pragma unroll
        for (int i = 0; i < MI; ++i) hi[i] = lo[i] = zero16();
        land_a(ra1, 0);
        __syncthreads();
        // k-tile t: its A is in LDS stage st, its first B half in rb0, the next tile's A in `ra`.  A wave without
        // columns stages and waits only; the branch is around the whole loop, not in it, where it would keep the
        // loads from running ahead (16.8 against 14.6 us for 3.5k x 512 x 256).
        auto k_loop = [&](auto live_c) __attribute__((always_inline)) {
            constexpr bool LIVE = decltype(live_c)::value;
            auto step = [&](RegA &ra, RegA &ra_next, int t, int st) __attribute__((always_inline)) {
                if (LIVE) { load_b(rb1, cur, 2 * t + 1); multiply(rb0, 0, st); load_b(rb0, cur, 2 * t + 2); }
                load_a(ra_next, cur, t + 2);
                if (LIVE) multiply(rb1, 1, st);
                land_a(ra, st ^ 1);
                __syncthreads();
            };
            int t = 0;
            for (; t + 2 <= KT - 1; t += 2) {
                step(ra0, ra1, t, 0);
                step(ra1, ra0, t + 1, 1);
            }
            if (t < KT - 1) step(ra0, ra1, t++, 0);
            if (LIVE) {
                load_b(rb1, cur, 2 * t + 1);
                multiply(rb0, 0, t & 1);
                if (32 * t + 8 < K) multiply(rb1, 1, t & 1);            // (granules 2 and 3 start at k = 8)
            }
            __syncthreads();
        };
        if (cur.n0 + 32 * wc < b.N) k_loop(std::true_type{});
        else k_loop(std::false_type{});
        // side inputs of the epilogue, then the next tile's first loads, then the stores: a wait for the
        // former does not wait for the latter
        const int n = cur.n0 + 32 * wc + l32;
        auto row_of = [&](int i, int r) { return cur.m0 + wr + 32 * i + (r >> 2) * 8 + half * 4 + (r & 3); };
        float side[EF::SIDE >= SIDE_ROW ? 16 * MI : 1];
        if (EF::SIDE >= SIDE_ROW) {
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    side[EF::SIDE >= SIDE_ROW ? 16 * i + r : 0] = epi.side(min(row_of(i, r), a.rows - 1), min(n, b.N - 1));
        } else {
            side[0] = EF::SIDE == SIDE_COL ? epi.side(0, min(n, b.N - 1)) : 0.f;
        }
        bool more = false;
        for (gid += gridDim.x; gid < total; gid += gridDim.x)
            if ((more = tile_at(gid, nxt))) break;
        if (!more) nxt = cur;
        load_b(rb0, nxt, 0);
        load_a(ra1, nxt, 0);
        load_a(ra0, nxt, 1);
        bool ok = true;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
#pragma unroll
            for (int r = 0; r < 16; ++r) hi[i][r] = (hi[i][r] + lo[i][r]) * SPLIT_UNSCALE;
            ok = ok && finite16(hi[i]);
        }
        const bool again = K < SPLIT_MIN_K || __ballot(!ok) != 0ull;
        // accumulator layout of the 32 x 32 block: register r of lane l holds row (r / 4) * 8 + (l / 32) * 4 + (r % 4), column l % 32
        const int rows = min(BM, a.rows - cur.m0);
        auto rsrc = __builtin_amdgcn_make_buffer_rsrc(epi.out + (int64_t)cur.m0 * epi.ld, 0, ((rows - 1) * epi.ld + b.N) * 4, 0x00020000);
        // (rows and columns past the edge get an offset past the buffer's end and are dropped)
        const int base = (4 * half * epi.ld + n) * 4;
        const int cols = again ? 0 : b.N;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            unsigned word = 0u;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = wr + 32 * i + (r >> 2) * 8 + (r & 3);
                const float v = epi.value(hi[i][r], side[EF::SIDE >= SIDE_ROW ? 16 * i + r : 0], n);
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rsrc, n < cols && row + 4 * half < rows ? base + row * epi.ld * 4 : 0x7FFFFFFC, 0, 0);
                if constexpr (split_keeps_bits<EF>) keep_ballot(word, r, v > 0.f);
            }
            if constexpr (split_keeps_bits<EF>) {
                const int row = wr + 32 * i + lane;
                auto brsrc = __builtin_amdgcn_make_buffer_rsrc(epi.bits + (int64_t)cur.m0 * epi.ldb, 0, rows * epi.ldb * 4, 0x00020000);
                __builtin_amdgcn_raw_buffer_store_b32(word, brsrc, lane < 32 && row < rows && cur.n0 + 32 * wc < cols
                                                                       ? (row * epi.ldb + (cur.n0 >> 5) + wc) * 4 : 0x7FFFFFFC, 0, 0);
            }
        }
        // formed again only here, where the sums and side inputs above need no registers any more (the lane's position
        // made opaque, or what follows from it is worked out in front of the loop over the tiles and kept there)
        if (again) {
            int l = lane;
            asm volatile("" : "+v"(l));
            const int col = cur.n0 + 32 * wc + (l & 31);
#pragma unroll 1
            for (int i = 0; i < MI; ++i) {
                const floatx16 e = split_exact_block(a, b, cur.m0 + wr + 32 * i + (l & 31), col, l >> 5);
                unsigned word = 0u;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int m = cur.m0 + wr + 32 * i + (r >> 2) * 8 + (l >> 5) * 4 + (r & 3);
                    float v = 0.f;
                    if (m < a.rows && col < b.N) {
                        const float x = EF::SIDE == SIDE_NONE ? 0.f : epi.side(m, col);
                        epi.out[(int64_t)m * epi.ld + col] = v = epi.value(e[r], x, col);
                    }
                    if constexpr (split_keeps_bits<EF>) keep_ballot(word, r, v > 0.f);
                }
                if constexpr (split_keeps_bits<EF>) {
                    const int m = cur.m0 + wr + 32 * i + l;
                    if (l < 32 && m < a.rows && cur.n0 + 32 * wc < b.N) epi.bits[(int64_t)m * epi.ldb + (cur.n0 >> 5) + wc] = word;
                }
            }
        }
        if (!more) return;
        cur = nxt;
    }
}

// The same for few rows: a workgroup takes 32 rows x 32 columns, its four waves every fourth k-tile each.  With about
// one workgroup per compute unit the k loop above is a chain of staging, barrier and multiplication per k-tile; here
// every wave fetches and splits its A fragments itself (the split is repeated for every 32 columns, on compute units
// that would idle), four steps of 16 k ahead and without a barrier, and the four partial sums meet in LDS, added in a
// fixed order.  (64 rows per workgroup: 9.0 to 9.5 us for 1024 x 512 x 256 and x 47.)
struct SplitFew { static constexpr int BM = 32, BN = 32; };

template <int VA, class EF>
__device__ __forceinline__ void split_few_rows_product(const SplitA &a, const SplitB &b, const EF &epi, uint4 *lds) {
    constexpr int BM = SplitFew::BM, WAVES = SNT / 64, AHEAD = 4;
    static_assert(WAVES * 16 * 64 * sizeof(float) <= SPLIT_LDS * sizeof(uint4), "LDS");
    float (*s_acc)[16][64] = reinterpret_cast<float (*)[16][64]>(lds);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int K = a.K, KT = (K + 31) / 32, KS = 2 * KT;
    const int tiles_m = (a.rows + BM - 1) / BM, tiles_n = (b.N + 31) / 32;
    const int total = ((tiles_m + 7) & ~7) * tiles_n;
    const int steps = 2 * ((KT - wave + WAVES - 1) / WAVES);        // steps of 16 k of this wave (0 for a wave past the last k-tile)
    for (int gid = blockIdx.x; gid < total; gid += gridDim.x) {
        int m0, n0;
        if (!next_tile<SplitFew>(gid, tiles_m, tiles_n, m0, n0)) continue;
        const uint4 *bp = b.frag + (int64_t)(n0 / 32) * KS * 192 + lane;
        const float *ap = a.p + (int64_t)min(m0 + l32, a.rows - 1) * a.ld;
        struct Reg { float v[8]; uint4 q[3]; };
        // step u: half u % 2 of k-tile wave + WAVES (u / 2)  (past the end: clamped addresses, not used)
        auto load = [&](Reg &r, int u) __attribute__((always_inline)) {
            const int t = min(wave + WAVES * (u >> 1), KT - 1), g = 2 * (u & 1) + half, k0 = 32 * t + 4 * g;
#pragma unroll
            for (int q = 0; q < 3; ++q) r.q[q] = bp[(2 * t + (u & 1)) * 192 + q * 64];
            if (VA == 4) {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const float4 f = *reinterpret_cast<const float4 *>(ap + min(k0 + 16 * j, K - 4));
                    r.v[4 * j] = f.x; r.v[4 * j + 1] = f.y; r.v[4 * j + 2] = f.z; r.v[4 * j + 3] = f.w;
                }
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) r.v[j] = ap[min(32 * t + granule_k(g, j), K - 1)];
            }
        };
        floatx16 hi = zero16(), lo = zero16();
        auto multiply = [&](const Reg &r) __attribute__((always_inline)) {
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = r.v[j] * SPLIT_SCALE;
            uint4 f[3];
            split8(v, f);
            hi = mfma_bf(f[0], r.q[0], hi);
            lo = mfma_bf(f[0], r.q[2], lo);
            lo = mfma_bf(f[0], r.q[1], lo);
            lo = mfma_bf(f[1], r.q[0], lo);
            lo = mfma_bf(f[1], r.q[1], lo);
            lo = mfma_bf(f[2], r.q[0], lo);
        };
        Reg r[AHEAD];
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) load(r[u], u);
        // side inputs of the epilogue: this wave finishes rows 8 wave + 4 half + 0..3
        const int n = n0 + l32, m = m0 + 8 * wave + 4 * half;
        float side[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) side[x] = EF::SIDE == SIDE_NONE ? 0.f : epi.side(min(m + x, a.rows - 1), min(n, b.N - 1));
        for (int u = 0; u < steps; u += AHEAD) {
#pragma unroll
            for (int j = 0; j < AHEAD; ++j) {
                if (u + j < steps) multiply(r[j]);
                load(r[j], u + j + AHEAD);
            }
        }
#pragma unroll
        for (int x = 0; x < 16; ++x) s_acc[wave][x][lane] = hi[x] + lo[x];
        __syncthreads();
        float v[4];
        bool ok = true;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const int reg = 4 * wave + x;
            v[x] = ((s_acc[0][reg][lane] + s_acc[1][reg][lane]) + (s_acc[2][reg][lane] + s_acc[3][reg][lane])) * SPLIT_UNSCALE;
            ok = ok && fabsf(v[x]) < INFINITY;
        }
        if (K < SPLIT_MIN_K || __ballot(!ok) != 0ull) {
            int l = lane;
            asm volatile("" : "+v"(l));         // (as above)
            const floatx16 e = split_exact_block(a, b, m0 + (l & 31), n0 + (l & 31), l >> 5);
#pragma unroll
            for (int x = 0; x < 16; ++x)
                if (x >> 2 == wave) v[x & 3] = e[x];
        }
#pragma unroll
        for (int x = 0; x < 4; ++x)
            if (m + x < a.rows && n < b.N) epi.out[(int64_t)(m + x) * epi.ld + n] = epi.value(v[x], side[x], n);
        __syncthreads();            // the next tile's sums go to the same LDS
    }
}

// one product per blockIdx.y (head): A, B and the output start that many steps further on
struct SplitSteps { int64_t a = 0, frag = 0, ref = 0; int out = 0; };
// FORMS: those the kernel holds and chooses from on the device, where the rows are known.
template <int FORMS, int VA, class EF>
__global__ __launch_bounds__(SNT) __attribute__((amdgpu_waves_per_eu(VA == 4 ? 3 : 2, VA == 4 ? 3 : 2)))
void k_rows_gemm_split(SplitA a, SplitB b, EF epi, SplitSteps step, const GsLevelMeta *__restrict__ meta_rows, int S, int n_cu) {
    __shared__ __attribute__((aligned(16))) uint4 lds[SPLIT_LDS];
    const int head = blockIdx.y;
    a.rows = meta_rows->front_off[S];
    a.p += head * step.a; b.frag += head * step.frag; b.ref += head * step.ref; epi.advance(head * step.out);
    const int form = split_form(FORMS, a.rows, b.N, a.K, gridDim.y, VA == 4, n_cu);
    if ((FORMS & FORM_FEW) && form == FORM_FEW) split_few_rows_product<VA>(a, b, epi, lds);
    else if ((FORMS & FORM_NARROW) && form == FORM_NARROW) split_rows_product<SplitNarrow, VA>(a, b, epi, lds);
    else if (FORMS & FORM_WIDE) split_rows_product<SplitWide, VA>(a, b, epi, lds);
}
template <class EF>
void launch_rows_split(gsplit_ctx *ctx, hipStream_t st, int64_t ub, bool va, const SplitA &a, const SplitB &b, const EF &epi,
                       const GsLevelMeta *meta_rows, int heads = 1, const SplitSteps &step = SplitSteps{}) {
    const int forms = split_forms(ub, b.N, a.K, heads, va, ctx->n_cu);
    // workgroups: enough for every form the kernel may take
    int64_t grid = 8;
    if (forms & FORM_FEW) grid = std::max(grid, std::min<int64_t>(gs_ceil_div(gs_ceil_div(ub, 32), 8) * 8 * gs_ceil_div(b.N, 32), 512));
    if (forms & FORM_NARROW) grid = std::max<int64_t>(grid, row_block_grid<SplitNarrow>(ctx, ub * heads, b.N) / heads);
    if (forms & FORM_WIDE) grid = std::max<int64_t>(grid, row_block_grid<SplitWide>(ctx, ub * heads, b.N) / heads);
    const dim3 blocks((unsigned)(grid + 7) / 8 * 8, heads);
#define GS_SPLIT(FORMS)                                                                                                  \
    do {                                                                                                                 \
        if (va) hipLaunchKernelGGL((k_rows_gemm_split<FORMS, 4, EF>), blocks, dim3(SNT), 0, st, a, b, epi, step, meta_rows, ctx->S, ctx->n_cu); \
        else hipLaunchKernelGGL((k_rows_gemm_split<FORMS, 1, EF>), blocks, dim3(SNT), 0, st, a, b, epi, step, meta_rows, ctx->S, ctx->n_cu);    \
    } while (0)
    if constexpr (split_keeps_bits<EF>) {       // (the few-rows form is none of its forms, rows come in pieces)
#define GS_SPLIT_BITS(FORMS) hipLaunchKernelGGL((k_rows_gemm_split<FORMS, 4, EF>), blocks, dim3(SNT), 0, st, a, b, epi, step, meta_rows, ctx->S, ctx->n_cu)
        if (forms == FORM_WIDE) GS_SPLIT_BITS(FORM_WIDE);
        else if (forms == FORM_NARROW) GS_SPLIT_BITS(FORM_NARROW);
        else GS_SPLIT_BITS(FORM_NARROW | FORM_WIDE);
#undef GS_SPLIT_BITS
    } else switch (forms) {
        case FORM_WIDE: GS_SPLIT(FORM_WIDE); break;
        case FORM_NARROW: GS_SPLIT(FORM_NARROW); break;
        case FORM_FEW | FORM_NARROW: GS_SPLIT(FORM_FEW | FORM_NARROW); break;
        case FORM_NARROW | FORM_WIDE: GS_SPLIT(FORM_NARROW | FORM_WIDE); break;
        default: GS_SPLIT(FORM_FEW | FORM_NARROW | FORM_WIDE); break;
    }
#undef GS_SPLIT
}

// ------------------------------------------------------------------------------------------
// Weight gradients: G[M x N] = X^T dZ over a chunk of rows (split_grad_chunks; split-K: a slab of partials per chunk, summed in
// a fixed order by a later kernel), a B x B block per workgroup, four waves of B/2 x B/2 (a team).  Both operands are
// k-major; a k-tile is 32 rows: waves 0, 1 fetch X, waves 2, 3 dZ, a thread an 8 (rows) x B/32 (columns)
// patch (32 lanes cover a block's piece of a row).  Splitting two rows of a column at a time is what the
// bf16 conversion packs into one word anyway, so the transposition to "8 consecutive k of one column" costs
// nothing; 128-bit LDS stores follow.  One LDS stage a team (48 KB for B = 128); the next patch travels in registers meanwhile.
// (B = 128, 290k x 256 x 256: steps of 16 rows in two stages 258 us, patches two steps ahead 241, this 220.)
// B = 128: two teams, one workgroup per compute unit, take every other 32 rows of the chunk, one splits while the other
// multiplies, and trade halves of their sums in LDS at the end.  As two workgroups with a chunk each they took as long (56k x
// 256 x 256 47.3 us, then 47.8, 9.6k x 512 x 256 23.2 / 22.9, 22k x 200 x 256 25.5 / 25.0, 274k x 256 x 256 186.5 / 190: before the
// order of the reads in `multiply`) but left twice the slabs, which the sum over them pays for: 19.1 -> 14.1 us for the gradients
// of 128-256-256-172, 16.8 -> 12.4 for 128-256-256-64, 10.9 -> 9.1 for 100-256-256-47.  What bounds the large ones is the matrix
// rate (274k rows at 1.12 PFLOP/s, six products per product), the small ones 8 to 10 us of launch, first rows and the trade.
// LDS: [plane][k granule of 8][B columns], column c at c ^ ((c >> 3) & 3): eight lanes of a store (columns
// B / 32 apart) fall into eight different groups of four banks, and so do those of a fragment read.
// The column sums of dZ (the bias gradient, row M of a slab) are taken by the dZ threads of the first tile
// row from the values they load, and added over the k granules in a fixed order.
// ------------------------------------------------------------------------------------------
struct SplitGrad {
    const float *x; int64_t ldx; int M;         // X: rows x M of each head, heads M columns apart
    const float *dz; int64_t ldz; int N;        // dZ: rows x N of each head, heads N columns apart
    float *part;                                // slabs [chunk][head][(M + 1) x N]
    int heads, nchunk;
};

// Teams of four waves that form a block together, each from every other 32 rows of the chunk.
constexpr int split_grad_teams(int B) { return B == 128 ? 2 : 1; }

// VX, VZ = 4: rows of the operand can be read in 16-byte pieces
template <int B, int VX, int VZ>
__device__ __forceinline__ void split_grad_tile(const SplitGrad &g, float *__restrict__ slab, const float *__restrict__ X,
                                                const float *__restrict__ dZ, int m0, int n0, int k_begin, int k_end, bool want_cs) {
    constexpr int CPT = B / 32, MI = B / 64;        // columns of a thread's patch; 32 x 32 blocks of a wave in each direction
    constexpr int TEAMS = split_grad_teams(B);
    typedef float patch_row __attribute__((ext_vector_type(CPT)));
    typedef float piece4 __attribute__((ext_vector_type(4)));
    __shared__ __attribute__((aligned(16))) uint4 s_parts[TEAMS * 24 * B];
    const int M = g.M, N = g.N;
    const int team = TEAMS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / SNT);
    const int tid = threadIdx.x % SNT, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint4 (*sX)[4 * B] = reinterpret_cast<uint4 (*)[4 * B]>(s_parts + team * 24 * B), (*sZ)[4 * B] = sX + 3;
    const int half = lane >> 5, l32 = lane & 31;
    auto word = [](int c, int kg) { return kg * B + (c ^ ((c >> 3) & 3)); };
    const bool is_z = wave >= 2;
    const int kg = (wave & 1) * 2 + half;                       // loader: columns CPT l32 .., rows 8 kg .. + 7
    const float *src = is_z ? dZ : X;
    const int64_t ld = is_z ? g.ldz : g.ldx;
    const int cols = is_z ? N : M, c_first = (is_z ? n0 : m0) + CPT * l32;
    const bool vec = is_z ? VZ == 4 : VX == 4;
    int cc[CPT];                                                // (columns past the edge re-read the last ones; never stored)
#pragma unroll
    for (int j = 0; j < CPT; ++j) cc[j] = min(c_first + j, cols - 1);
    if (vec) cc[0] = min(c_first, cols - CPT);

    floatx16 hi[MI][MI], lo[MI][MI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < MI; ++j) hi[i][j] = lo[i][j] = zero16();
    patch_row cs, in[8];
#pragma unroll
    for (int c = 0; c < CPT; ++c) cs[c] = 0.f;
    auto load = [&](int k0) __attribute__((always_inline)) {
        // (one branch around all rows: around each of them, where only one operand comes in pieces, it put a wait behind every row,
        // which two waves on a SIMD do not cover: 274k x 256 x 130 565 us, 211 so, 22k x 1024 x 130 140 / 65)
        auto row = [&](int i) __attribute__((always_inline)) { return src + (int64_t)min(k0 + 8 * kg + i, k_end - 1) * ld; };
        if ((VX == 4 && VZ == 4) || vec) {
#pragma unroll
            for (int i = 0; i < 8; ++i) in[i] = *reinterpret_cast<const patch_row *>(row(i) + cc[0]);
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int c = 0; c < CPT; ++c) in[i][c] = row(i)[cc[c]];
        }
    };
    auto land = [&](int k0) __attribute__((always_inline)) {
        if (k0 + 32 > k_end) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (k0 + 8 * kg + i >= k_end) {
#pragma unroll
                    for (int c = 0; c < CPT; ++c) in[i][c] = 0.f;
                }
        }
        if (want_cs) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int c = 0; c < CPT; ++c) cs[c] += in[i][c];
        }
        uint4 (*t)[4 * B] = is_z ? sZ : sX;
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            float v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = in[i][c] * SPLIT_SCALE;
            uint4 p[3];
            split8(v, p);
#pragma unroll
            for (int q = 0; q < 3; ++q) t[q][word(CPT * l32 + c, kg)] = p[q];
        }
    };
    const int wm0 = (wave >> 1) * (B / 2), wn0 = (wave & 1) * (B / 2);
    // (a wave whose block lies outside the matrix only stages)
    const bool live = m0 + wm0 < M && n0 + wn0 < N;
    int ra[MI], rb[MI];
#pragma unroll
    for (int i = 0; i < MI; ++i) { ra[i] = word(wm0 + 32 * i + l32, half); rb[i] = word(wn0 + 32 * i + l32, half); }
    // The two halves of the tile one after the other.  With two waves on a SIMD nobody covers for one that waits for the LDS,
    // and the scheduler puts every read right in front of its product; so a fragment of the second half is asked for when one of
    // the first has been used, and the rows of the next tile behind the first products (56k x 256 x 256 49 -> 46 us, 22k x 200 x
    // 256 25.1 -> 23.5, 29k x 512 x 256 50.5 -> 47.6).  Four waves on a SIMD, B = 64, do without: an order of reads costs them
    // 0.5 us of 144 in a training step of 777 targets.  Rows read float by float are asked for in front of the products (behind
    // the first ones 274k x 254 x 256 249 -> 244 us, 274k x 254 x 130 281 -> 276).
    auto multiply = [&](int kv, int k_next) __attribute__((always_inline)) {
        constexpr bool LATE = TEAMS > 1 && VX == 4 && VZ == 4;
        if constexpr (!LATE) load(k_next);
        if (!live || kv <= 0) {
            if constexpr (LATE) load(k_next);
            return;
        }
        uint4 fa[2][3][MI], fb[2][3][MI];
        auto get_a = [&](int s, int q) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < MI; ++i) fa[s][q][i] = sX[q][ra[i] + 2 * s * B];
        };
        auto get_b = [&](int s, int q) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < MI; ++i) fb[s][q][i] = sZ[q][rb[i] + 2 * s * B];
        };
        auto product = [&](floatx16 (&acc)[MI][MI], int s, int pa, int pb) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < MI; ++j) acc[i][j] = mfma_bf(fa[s][pa][i], fb[s][pb][j], acc[i][j]);
        };
        if constexpr (TEAMS == 1) {
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                if (s == 1 && kv <= 16) break;
#pragma unroll
                for (int q = 0; q < 3; ++q) { get_a(s, q); get_b(s, q); }
                product(hi, s, 0, 0);
                product(lo, s, 2, 0);
                product(lo, s, 0, 2);
                product(lo, s, 1, 1);
                product(lo, s, 1, 0);
                product(lo, s, 0, 1);
            }
            return;
        }
        auto in_order = [] { __builtin_amdgcn_sched_barrier(0); };
        get_a(0, 0); get_b(0, 0); in_order();
        get_a(0, 2); get_b(0, 2); in_order();
        get_a(0, 1); get_b(0, 1); in_order();
        product(hi, 0, 0, 0); in_order();
        if constexpr (LATE) load(k_next);
        product(lo, 0, 2, 0); in_order();
        get_a(1, 0); in_order();
        product(lo, 0, 0, 2); in_order();
        get_b(1, 0); in_order();
        product(lo, 0, 1, 1);
        product(lo, 0, 1, 0); in_order();
        get_a(1, 2); get_b(1, 2); in_order();
        product(lo, 0, 0, 1); in_order();
        get_a(1, 1); get_b(1, 1); in_order();
        product(hi, 1, 0, 0);
        product(lo, 1, 2, 0);
        product(lo, 1, 0, 2);
        product(lo, 1, 1, 1);
        product(lo, 1, 1, 0);
        product(lo, 1, 0, 1);
    };
    constexpr int STEP = 32 * TEAMS;
    load(k_begin + 32 * team);
    if (team) __syncthreads();               // half a step behind: one team multiplies while the other stages
    for (int k0 = k_begin; k0 < k_end; k0 += STEP) {
        const int k = k0 + 32 * team;
        land(k);
        __syncthreads();
        multiply(k_end - k, k + STEP);       // (next rows past the end: the last one again, never landed)
        if (!team || k0 + STEP < k_end) __syncthreads();
    }
    if (TEAMS > 1) __syncthreads();          // (the second team has multiplied its last step)
    float *red = reinterpret_cast<float *>(s_parts + (TEAMS > 1 ? 32 * B : 0));
    if (want_cs && is_z) {
#pragma unroll
        for (int c = 0; c < CPT; ++c) red[(team * 4 + kg) * B + CPT * l32 + c] = cs[c];
    }
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < MI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) hi[i][j][r] = (hi[i][j][r] + lo[i][j][r]) * SPLIT_UNSCALE;
    // two teams: each hands the other half of its sums, and finishes and stores the rows of 32 x 32 blocks of its number
    constexpr int MINE = MI / TEAMS;         // rows of blocks that a wave stores
    piece4 *trade = reinterpret_cast<piece4 *>(s_parts) + wave * (8 * MI * 64 / 2) + lane;
    if constexpr (TEAMS == 2) {
        static_assert(MI == 2, "a row of blocks for each team");
#pragma unroll
        for (int j = 0; j < MI; ++j)
#pragma unroll
            for (int r = 0; r < 16; r += 4) {
                piece4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = team ? hi[0][j][r + e] : hi[1][j][r + e];
                trade[(team * 4 * 8 + j * 4 + r / 4) * 64] = v;
            }
    }
    if (TEAMS > 1 || want_cs) __syncthreads();
    if (want_cs && team == 0 && tid < B && n0 + tid < N) {
        float sum = 0.f;
#pragma unroll
        for (int t = 0; t < TEAMS; ++t) sum += red[4 * t * B + tid] + red[(4 * t + 1) * B + tid] + red[(4 * t + 2) * B + tid] + red[(4 * t + 3) * B + tid];
        slab[(int64_t)M * N + n0 + tid] = sum;
    }
    if (!live) return;
    if constexpr (TEAMS == 2) {
#pragma unroll
        for (int j = 0; j < MI; ++j)
#pragma unroll
            for (int r = 0; r < 16; r += 4) {
                const piece4 v = trade[((1 - team) * 4 * 8 + j * 4 + r / 4) * 64];
#pragma unroll
                for (int e = 0; e < 4; ++e) hi[0][j][r + e] = team ? v[e] + hi[1][j][r + e] : hi[0][j][r + e] + v[e];
            }
    }
    const int row0 = m0 + wm0 + 32 * MINE * team;
    bool ok = true;
#pragma unroll
    for (int i = 0; i < MINE; ++i)
#pragma unroll
        for (int j = 0; j < MI; ++j) ok = ok && finite16(hi[i][j]);
    if (k_end - k_begin < SPLIT_MIN_K || __ballot(!ok) != 0ull) {
#pragma unroll 1
        for (int b = 0; b < MINE * MI; ++b) {
            const float *xp = X + min(row0 + 32 * (b / MI) + l32, M - 1), *zp = dZ + min(n0 + wn0 + 32 * (b % MI) + l32, N - 1);
            const floatx16 e = exact_sum(k_begin, k_end, half, [&](int k) { return k < k_end ? xp[k * g.ldx] : 0.f; },
                                         [&](int k) { return k < k_end ? zp[k * g.ldz] : 0.f; });
#pragma unroll
            for (int x = 0; x < MINE * MI; ++x)
                if (x == b) hi[x / MI][x % MI] = e;
        }
    }
#pragma unroll
    for (int i = 0; i < MINE; ++i)
#pragma unroll
        for (int j = 0; j < MI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = row0 + 32 * i + (r >> 2) * 8 + half * 4 + (r & 3), n = n0 + wn0 + 32 * j + l32;
                if (m < M && n < N) slab[(int64_t)m * N + n] = hi[i][j][r];
            }
}

// The output tiles of one chunk read the same rows of X and dZ; the workgroup id is decoded so that they land on the same
// XCD (workgroups are dealt round-robin to the 8 XCDs) and share its L2: every eighth chunk is an XCD's.  Where the chunks do not
// come in eights, an XCD takes an eighth of the blocks, chunk after chunk, and shares one with its neighbour (taken for
// all: 1000 x 512 x 256 14.1 -> 14.6 us a backward pass).
template <int B, int VX, int VZ>
__device__ __forceinline__ void split_grad_block_product(const SplitGrad &g, int block, int n1) {
    const int kchunk = grad_w_chunk_rows(n1, g.nchunk, SGW_ROWS_MIN);
    const int tiles_m = (g.M + B - 1) / B, tiles = tiles_m * ((g.N + B - 1) / B);
    const int xcd = block & 7, per = tiles * g.heads;
    int j = block >> 3, chunk = 0;
    if (B != 128 || (g.nchunk & 7) == 0) chunk = j / per * 8 + xcd;
    else {
        const int each = ((n1 + kchunk - 1) / kchunk * per + 7) >> 3;
        if (j >= each) return;
        j += xcd * each;
        chunk = j / per;
    }
    const int tile = j % tiles, head = (j / tiles) % g.heads, k_begin = chunk * kchunk;
    if (k_begin >= n1) return;      // (the loop over a chunk's rows is built for one that has some: 50k x 512 x 256 73 us without)
    const int k_end = min(n1, k_begin + kchunk), tm = tile % tiles_m;
    split_grad_tile<B, VX, VZ>(g, g.part + ((int64_t)chunk * g.heads + head) * (g.M + 1) * g.N, g.x + head * g.M, g.dz + head * g.N,
                               tm * B, (tile / tiles_m) * B, k_begin, k_end, tm == 0);
}
template <int B, int VX, int VZ>
__global__ __launch_bounds__(SNT * split_grad_teams(B)) __attribute__((amdgpu_waves_per_eu(B == 128 ? 2 : 4, B == 128 ? 2 : 4)))
void k_grad_w_split(SplitGrad g, const GsLevelMeta *__restrict__ meta_up, int S) {
    split_grad_block_product<B, VX, VZ>(g, blockIdx.x, meta_up->front_off[S]);
}
// workgroups of a launch, a multiple of 8
inline int split_grad_blocks(const SplitGrad &g, int B) {
    return (int)(gs_ceil_div(g.nchunk * g.heads * gs_ceil_div(g.M, B) * gs_ceil_div(g.N, B), 8) * 8);
}

inline void launch_grad_w_split(hipStream_t st, int64_t ub_rows, bool vx, bool vz, const SplitGrad &g, const GsLevelMeta *mu, int S) {
    const int B = split_grad_block(ub_rows, g.M, g.N);
    const dim3 grid((unsigned)split_grad_blocks(g, B));
#define GS_GRAD(VX, VZ)                                                                                       \
    do {                                                                                                      \
        if (B == 128) hipLaunchKernelGGL((k_grad_w_split<128, VX, VZ>), grid, dim3(SNT * split_grad_teams(128)), 0, st, g, mu, S); \
        else hipLaunchKernelGGL((k_grad_w_split<64, VX, VZ>), grid, dim3(SNT), 0, st, g, mu, S);       \
    } while (0)
    if (vx && vz) GS_GRAD(4, 4);
    else if (vx) GS_GRAD(4, 1);
    else if (vz) GS_GRAD(1, 4);
    else GS_GRAD(1, 1);
#undef GS_GRAD
}
