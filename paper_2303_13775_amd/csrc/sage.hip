// GraphSAGE-mean forward and backward over the split mini-batch (paper Algorithm 2 `sp_forward`
// and the backward description after it).  The rows of all S logical splits are processed in one
// launch per step: on one GPU the training shuffle of layer l is the composition of the shuffle
// index with edges[l] (self_row / edge_row, built during sampling), so "shuffle then aggregate"
// is a gather through one index and the reverse shuffle of the backward pass is a scatter-add
// through the same index.
//
// Dense products run on the matrix cores; those of fp32 storage as six bfloat16 products (gemm_split.h).
#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "gsplit_internal.h"
#include "resident.h"

namespace {

#include "gemm_common.h"
#include "gemm_split.h"

// [W_self; W_neigh] stacked into one 2 D x Npad matrix (Npad = N rounded up to 4, padding zeroed):
// every product then reads the weights as one plain matrix in 16-byte pieces whatever N is.  All
// layers are laid out by the workgroups behind the bottom layer's input assembly's own (they are needed no
// earlier than the product that follows; a launch of its own took 5.6 us of a bf16 pass).
struct WeightStack {
    const float *ws[GS_MAXL]; const float *wn[GS_MAXL]; float *stacked[GS_MAXL]; int D[GS_MAXL]; int N[GS_MAXL];
    uint4 *frag_fwd[GS_MAXL]; uint4 *frag_gin[GS_MAXL];
    // part b of KINDS x n x layers: 0 the stacked matrix, 1 and 2 the fragments of the split products: B = the stacked matrix
    // (forward), its transpose (input gradient).  Workgroups of their own for each: one after the other in the same ones,
    // they made the input assembly of 33 rows 9.0 us instead of 5.8.
    static constexpr int KINDS = 3;
    __device__ __forceinline__ void run(int b, int n) const {
        const int l = b / (KINDS * n), what = b / n % KINDS;
        const int d = D[l], cols = N[l], np = (cols + 3) & ~3;
        const float *s = ws[l], *t = wn[l];
        auto at = [&](int k, int c) { return *(k < d ? s + (int64_t)k * cols + c : t + (int64_t)(k - d) * cols + c); };
        const int64_t x0 = (b % n) * (int64_t)blockDim.x + threadIdx.x, stride = (int64_t)n * blockDim.x;
        if (what == 1) {
            split_frag_fill(frag_fwd[l], 2 * d, cols, x0, stride, at);
        } else if (what == 2) {
            if (frag_gin[l]) split_frag_fill(frag_gin[l], cols, 2 * d, x0, stride, [&](int k, int c) { return at(c, k); });
        } else {
            const int64_t words = (int64_t)2 * d * np;
            for (int64_t x = x0; x < words; x += stride) {
                const int k = (int)(x / np), c = (int)(x % np);
                stacked[l][x] = c < cols ? at(k, c) : 0.f;
            }
        }
    }
};
// bf16: float [D x N] pairs -> bf16 stacked [2D x Npad] (rows j, for dZ * W^T) and transposed [N x 2D] (rows n, for
// X * W).  Npad = N rounded up to 8, padding columns are zero.
struct WeightPrep {
    const float *ws[GS_MAXL]; const float *wn[GS_MAXL];
    uint16_t *stacked[GS_MAXL]; uint16_t *transposed[GS_MAXL];
    int D[GS_MAXL]; int N[GS_MAXL];
    static constexpr int KINDS = 1;
    __device__ __forceinline__ void run(int b, int n_blocks) const {
        const int l = b / n_blocks;
        const int d = D[l], cols = N[l], np = (cols + 7) & ~7;
        const int64_t total = (int64_t)2 * d * np;
        for (int64_t x = (b % n_blocks) * (int64_t)blockDim.x + threadIdx.x; x < total; x += (int64_t)n_blocks * blockDim.x) {
            const int j = (int)(x / np), n = (int)(x - (int64_t)j * np);
            uint16_t h = 0;
            if (n < cols) {
                h = f2bf(j < d ? ws[l][(int64_t)j * cols + n] : wn[l][(int64_t)(j - d) * cols + n]);
                transposed[l][(int64_t)n * 2 * d + j] = h;
            }
            stacked[l][x] = h;
        }
    }
};

// VEC consecutive floats of a row: features, activations (held in float or in bf16), gradients
template <int VEC> struct FloatVec { float v[VEC]; };

template <int VEC, bool HALF>
__device__ __forceinline__ FloatVec<VEC> load_vec(const void *__restrict__ p, int64_t idx) {
    FloatVec<VEC> r;
    if constexpr (HALF) {
        static_assert(VEC == 4, "bf16 rows come in pieces of four");
        const uint2 raw = reinterpret_cast<const uint2 *>(p)[idx];
        r.v[0] = bf2f(raw.x & 0xFFFFu); r.v[1] = bf2f(raw.x >> 16); r.v[2] = bf2f(raw.y & 0xFFFFu); r.v[3] = bf2f(raw.y >> 16);
    } else if constexpr (VEC == 4) {
        const float4 x = reinterpret_cast<const float4 *>(p)[idx];
        r.v[0] = x.x; r.v[1] = x.y; r.v[2] = x.z; r.v[3] = x.w;
    } else if constexpr (VEC == 2) {
        const float2 x = reinterpret_cast<const float2 *>(p)[idx];
        r.v[0] = x.x; r.v[1] = x.y;
    } else {
        r.v[0] = reinterpret_cast<const float *>(p)[idx];
    }
    return r;
}

template <int VEC>
__device__ __forceinline__ void add_vec(FloatVec<VEC> &a, const FloatVec<VEC> &b) {
#pragma unroll
    for (int i = 0; i < VEC; ++i) a.v[i] += b.v[i];
}

template <int VEC>
__device__ __forceinline__ void store_vec(float *__restrict__ p, int64_t idx, const FloatVec<VEC> &x) {
    if constexpr (VEC == 4) reinterpret_cast<float4 *>(p)[idx] = make_float4(x.v[0], x.v[1], x.v[2], x.v[3]);
    else if constexpr (VEC == 2) reinterpret_cast<float2 *>(p)[idx] = make_float2(x.v[0], x.v[1]);
    else p[idx] = x.v[0];
}

// ------------------------------------------------------------------------------------------
// Layer input assembly: for destination row i
//   X[i, 0:D]  = H[self_row[i], :]                         (its own lower-layer row)
//   X[i, D:2D] = (1/cnt_i) * sum_e H[edge_row[e], :]        (mean over its sampled sources)
// i.e. the training shuffle and the mean aggregation in one gather through the composed shuffle
// index.  One lane group per destination row, a piece of it per lane (16 bytes where the rows allow, else 8 or 4),
// edges in slot order (deterministic), 4, 8 or 16 row loads in flight by the fanout (see assemble_step).  X feeds the
// forward product and, transposed, the weight-gradient product.
// Bound by the reads of the source rows: 266k rows of 20 edges x 512 bytes take 410 us, 6.6 TB/s with the rows
// written.  (bf16 rows in pieces of 8 bytes, two in flight: 567k rows of 10 edges x 256 bytes 305 us, this 247;
// 129k x 512 bytes 142 / 122.  Slices of 128-byte lines, one per XCD, so that an L2 sees an eighth of the rows'
// bytes: fp32 410 -> 445, bf16 the same.)
// ------------------------------------------------------------------------------------------
// A piece of a row: what a lane loads of it, the sums over the sources, what it stores.
template <int VEC>
struct PieceF {
    using Weights = WeightStack;
    using Raw = FloatVec<VEC>;
    static constexpr int VALUES = VEC;
    FloatVec<VEC> sum{};
    __device__ __forceinline__ static Raw load(const void *p, int64_t idx) { return load_vec<VEC, false>(p, idx); }
    __device__ __forceinline__ static void store(void *p, int64_t idx, const Raw &r) { store_vec(reinterpret_cast<float *>(p), idx, r); }
    __device__ __forceinline__ void add(const Raw &r) { add_vec(sum, r); }
    __device__ __forceinline__ Raw over(float cnt) const {
        Raw r;
#pragma unroll
        for (int i = 0; i < VEC; ++i) r.v[i] = sum.v[i] / cnt;
        return r;
    }
};
// bf16 rows, the mean accumulated in float: WORDS pairs of values
template <int WORDS>
struct PieceH {
    using Weights = WeightPrep;
    struct alignas(4 * WORDS) Raw { uint32_t w[WORDS]; };
    static constexpr int VALUES = 2 * WORDS;
    float sum[2 * WORDS] = {};
    __device__ __forceinline__ static Raw load(const void *p, int64_t idx) { return reinterpret_cast<const Raw *>(p)[idx]; }
    __device__ __forceinline__ static void store(void *p, int64_t idx, const Raw &r) { reinterpret_cast<Raw *>(p)[idx] = r; }
    __device__ __forceinline__ void add(const Raw &r) {
#pragma unroll
        for (int i = 0; i < WORDS; ++i) { sum[2 * i] += bf2f(r.w[i] & 0xFFFFu); sum[2 * i + 1] += bf2f(r.w[i] >> 16); }
    }
    __device__ __forceinline__ Raw over(float cnt) const {
        Raw r;
#pragma unroll
        for (int i = 0; i < WORDS; ++i) r.w[i] = (uint32_t)f2bf(sum[2 * i] / cnt) | ((uint32_t)f2bf(sum[2 * i + 1] / cnt) << 16);
        return r;
    }
};

// STEP: edges in flight, see assemble_step
template <int LPR, int STEP, class Piece>
__global__ __launch_bounds__(256) void k_assemble_input(const void *__restrict__ H, int D,
                                                            const int32_t *__restrict__ blk_indptr,
                                                            const int32_t *__restrict__ edge_row,
                                                            const int32_t *__restrict__ self_row,
                                                            const GsLevelMeta *__restrict__ meta_up,
                                                            int S, int fan, void *__restrict__ X,
                                                            float *__restrict__ inv_cnt, int n_main,
                                                            typename Piece::Weights weights, int n_stack) {
    if ((int)blockIdx.x >= n_main) {        // the workgroups behind the kernel's own lay out the weights
        weights.run((int)blockIdx.x - n_main, n_stack);
        return;
    }
    const int n1 = meta_up->front_off[S];
    const int nvec = D / Piece::VALUES;
    const int c0 = threadIdx.x % LPR;
    const int groups = (n_main * blockDim.x) / LPR;
    const int n_c = (nvec + LPR - 1) / LPR;      // column rounds, the same for every lane of a group
    using Raw = typename Piece::Raw;
    static_assert(LPR % STEP == 0, "rounds of STEP edges");
    // A row is a chain of dependent accesses (offsets -> source rows of its edges -> their values), and
    // the kernel's time is the length of that chain, not its bytes.  So the lanes of a group fetch the
    // source rows of up to LPR edges with one load (lane u takes edge u, the others get it by shuffle)
    // and keep the values of STEP edges in flight; the sum still runs in edge order.  Edges a row
    // does not have are read from its own row (a valid address) and not added.
    for (int row = (blockIdx.x * blockDim.x + threadIdx.x) / LPR; row < n1; row += groups) {
        const int e0 = blk_indptr[row];
        const int m = blk_indptr[row + 1] - e0;
        const int64_t self = self_row[row];
        const float cnt = (float)m;
        if (c0 == 0) inv_cnt[row] = m > 0 ? 1.f / cnt : 0.f;
        for (int ci = 0; ci < n_c; ++ci) {
            const int c = c0 + ci * LPR;
            const bool cv = c < nvec;
            const int cc = cv ? c : 0;
            const Raw own = Piece::load(H, self * nvec + cc);
            Piece acc;
            for (int chunk = 0; chunk < fan; chunk += LPR) {
                const int mine = chunk + c0 < m ? edge_row[e0 + chunk + c0] : -1;
#pragma unroll
                for (int half = 0; half < LPR; half += STEP) {
                    // wave-uniform: does any row of this wave reach this far?
                    if (__ballot(chunk + half < m) == 0ull) break;
                    Raw v[STEP];
                    unsigned have = 0u;
#pragma unroll
                    for (int u = 0; u < STEP; ++u) {
                        const int r = __shfl(mine, half + u, LPR);
                        have |= (r >= 0 ? 1u : 0u) << u;
                        v[u] = Piece::load(H, (r >= 0 ? (int64_t)r : self) * nvec + cc);
                    }
#pragma unroll
                    for (int u = 0; u < STEP; ++u) {
                        if ((have >> u) & 1u) acc.add(v[u]);
                    }
                }
            }
            const Raw mean = acc.over(m > 0 ? cnt : 1.f);
            if (cv) {
                Piece::store(X, (int64_t)row * 2 * nvec + c, own);
                Piece::store(X, (int64_t)row * 2 * nvec + nvec + c, mean);
            }
        }
    }
}

// ---- operand accessors and epilogues ---------------------------------------------------------
__device__ const uint16_t g_one_then_zero_h[4] __attribute__((aligned(8))) = {0x3F80, 0, 0, 0};   // bf16 1, 0, 0, 0

// input gradients per destination row: [dH_self | dMean / cnt]; the reverse shuffle (pull through
// the scatter side of the shuffle index) follows in k_pull_input_grad
struct EpiGradIn {
    float *out; const float *inv_cnt; int D; int n1;
    __device__ __forceinline__ float col(int) const { return 0.f; }
    __device__ __forceinline__ float row(int i) const { return i < n1 ? inv_cnt[i] : 0.f; }
    __device__ __forceinline__ void store(int i, int j, float v, float w, float) const {
        if (i >= n1 || j >= 2 * D) return;
        out[(int64_t)i * 2 * D + j] = j < D ? v : v * w;
    }
};

// tile of the bf16 kernels
constexpr int GBM = 64, GBN = 128, GWM = 2, GWN = 4;

// Sum the per-chunk partials in a fixed order into the caller's gradient buffers, all layers in one
// launch (blockIdx.y = layer).
struct GradReduce {
    const float *part[GS_MAXL]; float *gws[GS_MAXL]; float *gwn[GS_MAXL]; float *gb[GS_MAXL];
    int D[GS_MAXL]; int N[GS_MAXL]; int nchunk[GS_MAXL]; int rows_min[GS_MAXL];
    int fixed_chunks[GS_MAXL];      // > 0: the layer's slabs were written by that many workgroups, all of them
    // a level of at least stream_rows rows (> 0) had its slabs written by the streaming bf16 kernel,
    // whose chunks follow (stream_nchunk, stream_rows_min)
    int stream_rows[GS_MAXL]; int stream_nchunk[GS_MAXL]; int stream_rows_min[GS_MAXL];
};
__global__ __launch_bounds__(256) void k_reduce_grads(GradReduce g, const GsLevelMeta *__restrict__ meta, int S) {
    const int l = blockIdx.y;
    const int n1 = meta[l + 1].front_off[S];
    const bool streamed = g.stream_rows[l] > 0 && n1 >= g.stream_rows[l];
    const int kchunk = streamed ? grad_w_chunk_rows(n1, g.stream_nchunk[l], g.stream_rows_min[l])
                                : grad_w_chunk_rows(n1, g.nchunk[l], g.rows_min[l]);
    const int chunks = g.fixed_chunks[l] > 0 ? g.fixed_chunks[l] : (n1 + kchunk - 1) / kchunk;
    const int D = g.D[l], N = g.N[l];
    const int64_t words = (int64_t)(2 * D + 1) * N, wn = (int64_t)D * N;
    sum_slabs(g.part[l], words, words, chunks, [&](int64_t x, float v) {
        if (x < wn) g.gws[l][x] = v;
        else if (x < 2 * wn) g.gwn[l][x - wn] = v;
        else g.gb[l][x - 2 * wn] = v;
    });
}

// Reverse shuffle of the backward pass as a pull: row u of local_cat[l] sums the gradient rows of
// every destination it fed (its own self term and one mean term per sampled edge), listed by the
// scatter side of the shuffle index.  The ReLU of the layer below is applied on the way out, so
// the result is that layer's dZ.  No atomics; rows that fed nothing get zeros.
//
// The entries of a row sit in its segment in the order an atomic cursor handed them out, which
// differs from run to run; a float sum in that order would too.  So the sum runs in ascending order
// of the entry codes (2 * destination [+ 1]), whatever the segment's order: one wave per row, one
// entry per lane, sorted across the wave with a bitonic network of shuffles (21 exchange steps, no
// memory traffic); then LPR lanes cover a gradient row 4 floats each, the 64 / LPR lane groups of
// the wave take every (64 / LPR)-th entry of the sorted list, and their partial sums are added in
// a fixed tree.  A row with up to 256 entries keeps four per lane (the same network over registers and
// lanes).  Gradients are bit-reproducible.
// A row with more than 256 entries (a hub: tens of thousands of destinations can sample the same
// vertex) is left to the workgroups behind the launch's own (blockIdx.x >= n_main), which walk the
// list of such rows that the sampler made: codes sorted in LDS (bitonic, up to PULL_LONG_CAP at a
// time: a longer row in windows of ascending values), the four waves sum a quarter of the sorted
// window each, partial sums added in wave order, windows in ascending order.
constexpr int PULL_LONG_CAP = 2048;
constexpr int PULL_LONG_BLOCKS = 1024;
// destinations (by their bound) up to which the weight gradients go with the pull: larger levels fill the chip with either
constexpr int64_t PULL_GRAD_ROWS = 16384;

// Bitonic sort across a wave, ascending, of the first p2 lanes' values (p2 a power of two; the lanes
// behind hold INT_MAX padding and stay where they are): log2(p2) * (log2(p2) + 1) / 2 exchange steps, so
// the common rows with two or three entries cost one or three shuffles, not the 21 of a full wave.
__device__ __forceinline__ int wave_sort_ascending(int v, int p2) {
    const int lane = threadIdx.x & 63;
    for (int k = 2; k <= p2; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            const int o = __shfl_xor(v, j);
            v = (((lane & j) == 0) == ((lane & k) == 0)) ? min(v, o) : max(v, o);
        }
    }
    return v;
}

// The same for 256 values, four per lane: element r * 64 + lane lives in v[r].  Exchanges at a distance
// of 64 or 128 elements are between registers of one lane, the others between lanes.
__device__ __forceinline__ void wave_sort4_ascending(int (&v)[4]) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int k = 2; k <= 256; k <<= 1) {
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1) {
            if (j >= 64) {
                const int jr = j >> 6;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if ((r & jr) == 0) {
                        const bool asc = ((r * 64 + lane) & k) == 0;
                        const int a = v[r], b = v[r | jr];
                        if ((a > b) == asc) { v[r] = b; v[r | jr] = a; }
                    }
                }
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int o = __shfl_xor(v[r], j);
                    const bool asc = ((r * 64 + lane) & k) == 0;
                    v[r] = (((lane & j) == 0) == asc) ? min(v[r], o) : max(v[r], o);
                }
            }
        }
    }
}

// What gates a piece of a gradient row, the ReLU's derivative: the activations themselves, held in float or bf16, or a bit
// for each (rows of (D + 31) / 32 words, pieces of four; see keeps_relu_bits).  The pull of a large level is bound by the bytes it
// moves, and float activations are a quarter of them: 274k rows of 256 173 -> 147 us.
enum GateBy { GATE_FLOAT = 0, GATE_HALF = 1, GATE_BITS = 2 };
template <int VEC, GateBy GATE>
struct Gate {
    FloatVec<VEC> h{};
    __device__ __forceinline__ void load(const void *p, int64_t row, int nvec, int c) { h = load_vec<VEC, GATE == GATE_HALF>(p, row * nvec + c); }
    __device__ __forceinline__ bool open(int i) const { return h.v[i] > 0.f; }
};
template <int VEC>
struct Gate<VEC, GATE_BITS> {
    static_assert(VEC == 4, "rows in pieces of four");
    unsigned b = 0u;
    __device__ __forceinline__ void load(const void *p, int64_t row, int nvec, int c) {
        asm volatile("" : "+v"(c));         // (opaque: what follows from it is worked out here, not kept in registers across the rows)
        b = (unsigned)reinterpret_cast<const uint8_t *>(p)[row * ((nvec + 7) / 8 * 4) + (c >> 1)] >> ((c & 1) * 4);
    }
    __device__ __forceinline__ bool open(int i) const { return (b >> i) & 1u; }
};

template <int VEC, bool OUT_H, GateBy GATE>
__device__ __forceinline__ void store_masked(void *__restrict__ gout, int64_t idx, FloatVec<VEC> acc, const Gate<VEC, GATE> &gate) {
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc.v[i] = gate.open(i) ? acc.v[i] : 0.f;
    // bf16 storage: dZ is kept as the bf16 value that both backward products consume
    if constexpr (OUT_H)
        reinterpret_cast<uint2 *>(gout)[idx] = make_uint2((uint32_t)f2bf(acc.v[0]) | ((uint32_t)f2bf(acc.v[1]) << 16),
                                                          (uint32_t)f2bf(acc.v[2]) | ((uint32_t)f2bf(acc.v[3]) << 16));
    else store_vec(reinterpret_cast<float *>(gout), idx, acc);
}

// gradient row of an entry, piece c
template <int VEC>
__device__ __forceinline__ int64_t entry_piece(int code, int nvec, int c) { return (int64_t)(code >> 1) * 2 * nvec + (code & 1) * nvec + c; }

// Gradient rows a lane group has in flight, and waves per SIMD the registers are cut for (they decide how many rows
// are on their way together): bf16 activations four and eight (567k rows of 256 of 129k destinations 352 -> 326 us; eight
// in flight spill at eight waves, 389, and six waves hold fewer rows, 358), float eight and six (266k of 28k 174 -> 170 us,
// four in flight 220 us, eight waves 186).
constexpr int pull_flight(bool half) { return half ? 4 : 8; }
constexpr int pull_waves(bool half) { return half ? 8 : 6; }

struct PullArgs {
    const float *gin; int D;
    const int32_t *rev_ptr, *rev_cnt, *rev_list, *rev_long;
    const void *hact; const GsLevelMeta *meta_lo; int S;
    void *gout; int n_main;         // workgroups of the rows a wave takes; those behind take the long rows
};

// SCALAR: a row's segment (it is the whole wave's) moves to scalar registers when it has come.  Worth it for float rows in pieces
// of four that take all lanes: 32k rows of 256 gated by bits 41.7 us in vector registers, 38.5 so, 57k rows gated by activations
// 38.3 / 36.3, 51k rows of 512 65.4 / 64.0, 274k rows of 256 143.5 / 147.  Where lane groups share a row's entries it is not: 274k
// rows of 128 104 / 113, of 64 92 / 99, of 32 88 / 94; nor in pieces of two, of 130 237 / 247, or beside weight gradients, 29k
// rows of 256 22.7 / 24.0.
template <int LPR, int VEC, GateBy GATE, bool OUT_H, bool SCALAR>
__device__ __forceinline__ void pull_rows(const float *__restrict__ gin, int D, const int32_t *__restrict__ rev_ptr,
                                          const int32_t *__restrict__ rev_cnt, const int32_t *__restrict__ rev_list,
                                          const int32_t *__restrict__ rev_long, const void *__restrict__ hact,
                                          const GsLevelMeta *__restrict__ meta_lo, int S, void *__restrict__ gout, int n_main,
                                          int block, int n_blocks) {
    using Vec = FloatVec<VEC>;
    const int nvec = D / VEC;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (block >= n_main) {
        // ---- long rows: one workgroup per row
        __shared__ int s_code[PULL_LONG_CAP];
        __shared__ Vec s_part[4][64];
        __shared__ int s_cnt;
        const int n_long = meta_lo->n_long;
        for (int i = block - n_main; i < n_long; i += n_blocks - n_main) {
            const int u = rev_long[i];
            const int n = rev_cnt[u], e0 = rev_ptr[u];
            for (int cb = 0; cb < nvec; cb += 64) {
                const int c = cb + lane;
                const bool cv = c < nvec;
                Vec total{};
                // A row of at most PULL_LONG_CAP entries is one window.  A longer one is taken in windows of
                // values (lo, T]: the codes of a row are distinct, so the largest T with at most
                // PULL_LONG_CAP codes inside (found by bisection over the values, one counting pass over
                // the row per step) yields the next PULL_LONG_CAP codes in ascending order whatever
                // order the row was filled in.
                int lo = -1;
                for (int taken = 0; taken < n;) {
                    int T = 0x7FFFFFFE;
                    if (n > PULL_LONG_CAP) {
                        int a = lo + 1, b = 0x7FFFFFFE;
                        while (a < b) {
                            const int mid = a + ((b - a + 1) >> 1);
                            __syncthreads();
                            if (threadIdx.x == 0) s_cnt = 0;
                            __syncthreads();
                            int cnt = 0;
                            for (int t = threadIdx.x; t < n; t += 256) {
                                const int code = rev_list[e0 + t];
                                cnt += (code > lo && code <= mid) ? 1 : 0;
                            }
                            for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o);
                            if (lane == 0 && cnt) atomicAdd(&s_cnt, cnt);
                            __syncthreads();
                            if (s_cnt <= PULL_LONG_CAP) a = mid; else b = mid - 1;
                        }
                        T = a;
                    }
                    __syncthreads();
                    if (threadIdx.x == 0) s_cnt = 0;
                    __syncthreads();
                    if (n > PULL_LONG_CAP) {
                        for (int t = threadIdx.x; t < n; t += 256) {
                            const int code = rev_list[e0 + t];
                            if (code > lo && code <= T) {
                                const int at = atomicAdd(&s_cnt, 1);
                                if (at < PULL_LONG_CAP) s_code[at] = code;
                            }
                        }
                    } else {
                        for (int t = threadIdx.x; t < n; t += 256) s_code[t] = rev_list[e0 + t];
                        if (threadIdx.x == 0) s_cnt = n;
                    }
                    __syncthreads();
                    const int m = min(s_cnt, PULL_LONG_CAP);
                    int p2 = 64;
                    while (p2 < m) p2 <<= 1;
                    for (int t = m + threadIdx.x; t < p2; t += 256) s_code[t] = 0x7FFFFFFF;
                    __syncthreads();
                    lo = T;
                    taken += max(m, 1);         // (a window is never empty; the loop ends whatever the row holds)
                    for (int k = 2; k <= p2; k <<= 1) {
                        for (int j = k >> 1; j > 0; j >>= 1) {
                            for (int t = threadIdx.x; t < (p2 >> 1); t += 256) {
                                const int ia = ((t & ~(j - 1)) << 1) | (t & (j - 1)), ib = ia | j;
                                const int x = s_code[ia], y = s_code[ib];
                                const bool asc = (ia & k) == 0;
                                if ((x > y) == asc) { s_code[ia] = y; s_code[ib] = x; }
                            }
                            __syncthreads();
                        }
                    }
                    // the four waves sum a quarter of the sorted codes each, eight gradient rows in flight
                    const int q = (m + 3) >> 2;
                    const int jb = wave * q, je = min(m, jb + q);
                    Vec acc{};
                    for (int j = jb; j < je; j += 8) {
                        Vec v[8];
#pragma unroll
                        for (int x = 0; x < 8; ++x) {
                            v[x] = Vec{};
                            if (cv) v[x] = load_vec<VEC, false>(gin, entry_piece<VEC>(s_code[min(j + x, je - 1)], nvec, c));
                        }
#pragma unroll
                        for (int x = 0; x < 8; ++x)
                            if (j + x < je) add_vec(acc, v[x]);
                    }
                    s_part[wave][lane] = acc;
                    __syncthreads();
                    if (wave == 0) {
                        Vec t = s_part[0][lane];
                        add_vec(t, s_part[1][lane]); add_vec(t, s_part[2][lane]); add_vec(t, s_part[3][lane]);
                        add_vec(total, t);
                    }
                }
                if (wave == 0 && cv) {
                    Gate<VEC, GATE> gate;
                    gate.load(hact, u, nvec, c);
                    store_masked<VEC, OUT_H>(gout, (int64_t)u * nvec + c, total, gate);
                }
            }
        }
        return;
    }
    constexpr int G = 64 / LPR;                 // lane groups of a wave: entries summed side by side
    constexpr int MANY = pull_flight(OUT_H);
    const int sub = lane / LPR, c0 = lane % LPR;
    const int n_c = (nvec + LPR - 1) / LPR;      // column rounds, the same for every lane
    // A row is a chain of three dependent accesses (segment -> codes -> gradient rows), and with one
    // row per wave at a time the kernel runs at the rate of that chain, not of the memory.  So a wave
    // looks two rows ahead: while it sums row u it already holds the codes of its next row and the
    // segment of the one after, and only the gradient rows themselves are waited for.
    const int n_lo = meta_lo->front_off[S];
    const int waves = (n_main * (int)blockDim.x) >> 6;
    const int u_first = (int)((block * blockDim.x + threadIdx.x) >> 6);
    auto uniform = [](int v) __attribute__((always_inline)) { return SCALAR ? __builtin_amdgcn_readfirstlane(v) : v; };
    int n_a = 0, e_a = 0, n_b = 0, e_b = 0, code_a = 0x7FFFFFFF;
    if (u_first < n_lo) { n_a = rev_cnt[u_first]; e_a = rev_ptr[u_first]; }
    if (u_first + waves < n_lo) { n_b = rev_cnt[u_first + waves]; e_b = rev_ptr[u_first + waves]; }
    n_a = uniform(n_a); e_a = uniform(e_a);
    if (lane < min(n_a, 64)) code_a = rev_list[e_a + lane];
    for (int u = u_first; u < n_lo; u += waves) {
        int n_c2 = 0, e_c2 = 0, code_b = 0x7FFFFFFF;
        if (u + 2 * waves < n_lo) { n_c2 = rev_cnt[u + 2 * waves]; e_c2 = rev_ptr[u + 2 * waves]; }
        const int n_next = uniform(n_b), e_next = uniform(e_b);
        if (u + waves < n_lo && lane < min(n_next, 64)) code_b = rev_list[e_next + lane];
        const int n = n_a, e0 = e_a, us = uniform(u);
        int v4[4];
        v4[0] = code_a;
        n_a = n_next; e_a = e_next; n_b = n_c2; e_b = e_c2; code_a = code_b;
        if (n > GS_REV_LONG) continue;          // a workgroup behind the launch's own takes it
        // the row's codes in registers, sorted: entry j of the sorted list is v[j / 64] of lane j % 64
        const int n_reg = (n + 63) >> 6;          // registers in use (uniform)
        if (n <= 64) {
            if (n > 1) {
                int p2 = 2;
                while (p2 < n) p2 <<= 1;
                v4[0] = wave_sort_ascending(v4[0], p2);
            }
        } else {
#pragma unroll
            for (int r = 1; r < 4; ++r) v4[r] = r * 64 + lane < n ? rev_list[e0 + r * 64 + lane] : 0x7FFFFFFF;
            wave_sort4_ascending(v4);
        }
        for (int ci = 0; ci < n_c; ++ci) {
            const int c = c0 + ci * LPR;
            const bool cv = c < nvec;
            // the activation that gates the result does not depend on the sum: fetched first, it
            // travels while the gradient rows are fetched
            Gate<VEC, GATE> gate;
            if (cv) gate.load(hact, us, nvec, c);
            Vec acc{};
            // FLIGHT entries per lane group side by side
            auto add_entries = [&](auto flight, int code, int j0, int m) __attribute__((always_inline)) {
                constexpr int FLIGHT = decltype(flight)::value;
                Vec v[FLIGHT];
                bool have[FLIGHT];
#pragma unroll
                for (int x = 0; x < FLIGHT; ++x) {
                    const int j = j0 + x * G + sub;
                    const int k = __shfl(code, j < 64 ? j : 63);
                    have[x] = j < m && cv;
                    v[x] = Vec{};
                    if (have[x]) v[x] = load_vec<VEC, false>(gin, entry_piece<VEC>(k, nvec, c));
                }
#pragma unroll
                for (int x = 0; x < FLIGHT; ++x)
                    if (have[x]) add_vec(acc, v[x]);
            };
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (r >= n_reg) break;
                const int m = min(64, n - r * 64);
                int j0 = 0;
                for (; m - j0 > 4 * G; j0 += MANY * G) add_entries(std::integral_constant<int, MANY>{}, v4[r], j0, m);
                if (j0 < m) add_entries(std::integral_constant<int, 4>{}, v4[r], j0, m);
            }
            // the lane groups' partial sums, added in a fixed tree
#pragma unroll
            for (int o = LPR; o < 64; o <<= 1)
#pragma unroll
                for (int i = 0; i < VEC; ++i) acc.v[i] += __shfl_xor(acc.v[i], o);
            if (sub == 0 && cv) store_masked<VEC, OUT_H>(gout, (int64_t)us * nvec + c, acc, gate);
        }
    }
}

// (Its arguments one by one and not as PullArgs: the eight waves of the bf16 rows leave 64 registers, and with the structure
// four of them spilled: 359 us for the 567k rows above, 336 so; float 179 and 175.)
template <int LPR, int VEC, bool HACT_H, bool OUT_H>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(pull_waves(OUT_H), 8))) void k_pull_input_grad(
    const float *__restrict__ gin, int D, const int32_t *__restrict__ rev_ptr, const int32_t *__restrict__ rev_cnt,
    const int32_t *__restrict__ rev_list, const int32_t *__restrict__ rev_long, const void *__restrict__ hact,
    const GsLevelMeta *__restrict__ meta_lo, int S, void *__restrict__ gout, int n_main) {
    pull_rows<LPR, VEC, HACT_H ? GATE_HALF : GATE_FLOAT, OUT_H, !HACT_H && VEC == 4 && LPR == 64>(gin, D, rev_ptr, rev_cnt, rev_list, rev_long, hact, meta_lo, S, gout, n_main,
                                                                blockIdx.x, gridDim.x);
}
// the same of float rows, gated by bits
template <int LPR>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(pull_waves(false), 8))) void k_pull_gated(
    const float *__restrict__ gin, int D, const int32_t *__restrict__ rev_ptr, const int32_t *__restrict__ rev_cnt,
    const int32_t *__restrict__ rev_list, const int32_t *__restrict__ rev_long, const void *__restrict__ bits,
    const GsLevelMeta *__restrict__ meta_lo, int S, void *__restrict__ gout, int n_main) {
    pull_rows<LPR, 4, GATE_BITS, false, LPR == 64>(gin, D, rev_ptr, rev_cnt, rev_list, rev_long, bits, meta_lo, S, gout, n_main, blockIdx.x, gridDim.x);
}

// The weight gradients of the layer whose input gradients are pulled, in the same launch: they wait for nothing the pull
// does, and of a small layer neither fills the chip (a chain of dependent accesses, a chain of k-tiles): 4595 rows of 130
// 20.8 -> 14.9 us, 21.6k rows of 256 29.3 -> 25.5.  (Half or a quarter of the chunks, and two workgroups of the pull per
// compute unit beside them, measured within a microsecond.)
template <int LPR, int VEC, int VZ>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4)))
void k_pull_and_grad_w(PullArgs p, SplitGrad g, const GsLevelMeta *__restrict__ meta_up, int n_grad) {
    if ((int)blockIdx.x < n_grad) split_grad_block_product<64, VEC == 1 ? 1 : 4, VZ>(g, blockIdx.x, meta_up->front_off[p.S]);
    else pull_rows<LPR, VEC, GATE_FLOAT, false, false>(p.gin, p.D, p.rev_ptr, p.rev_cnt, p.rev_list, p.rev_long, p.hact, p.meta_lo, p.S, p.gout,
                                           p.n_main, (int)blockIdx.x - n_grad, (int)gridDim.x - n_grad);
}

// Mean softmax cross-entropy of the target rows and its gradient w.r.t. the logits: one wave per
// target; the label of row r is labels[local_cat[L][r]].
__global__ __launch_bounds__(256) void k_softmax_xent(const float *__restrict__ logits, int C,
                                                      const int64_t *__restrict__ labels,
                                                      const int32_t *__restrict__ front_top,
                                                      const GsLevelMeta *__restrict__ meta_top, int S,
                                                      float *__restrict__ grad, float *__restrict__ row_loss) {
    const int n = meta_top->front_off[S];
    const int lane = threadIdx.x & 63;
    const int waves = (gridDim.x * blockDim.x) >> 6;
    for (int r = (blockIdx.x * blockDim.x + threadIdx.x) >> 6; r < n; r += waves) {
        const float *z = logits + (int64_t)r * C;
        float mx = -3.4e38f;
        for (int c = lane; c < C; c += 64) mx = fmaxf(mx, z[c]);
        for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
        float sum = 0.f;
        for (int c = lane; c < C; c += 64) sum += __expf(z[c] - mx);
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
        const int y = (int)labels[front_top[r]];
        const float inv = 1.f / sum, invn = 1.f / (float)n;
        for (int c = lane; c < C; c += 64) {
            const float p = __expf(z[c] - mx) * inv;
            grad[(int64_t)r * C + c] = (p - (c == y ? 1.f : 0.f)) * invn;
        }
        if (row_loss && lane == 0) row_loss[r] = (y >= 0 && y < C) ? (logf(sum) + mx - z[y]) : 0.f;
    }
}

// ------------------------------------------------------------------------------------------
// The top layer of a training step in one launch.  Its products are tiny (n_targets x 2 D x classes:
// 49 MFLOP each for 1024 targets, 512 inputs, 47 classes) and as separate launches the chain
//   input assembly -> forward product -> loss -> weight-gradient product -> input-gradient product
// is five kernel boundaries around a few microseconds of work.  Here a workgroup takes TOP_R
// destination rows at a time through all of it: the assembled rows [H_self | mean] and dZ stay in LDS, the
// weights come from the L2 as the fragments the matrix cores take (asked for before the rows they meet are there), and the
// weight-gradient partial of the workgroup goes to its own slab (summed in a fixed order by
// k_reduce_grads: deterministic, no atomics).  The kernel's time is its chain of dependent steps (offsets, source rows,
// three products with a barrier between them; clocks in the kernel, 1024 targets of 5 sources x 256 x 47 in fp32: weights and
// offsets 1.7 us, rows 4.7, forward product 1.7, loss 1.7, input gradient 3.5, weight gradient 3.8).  With plain FMAs, eight
// rows a workgroup, it took 26 us, now 20 (and half the slabs to sum); in bf16 the five launches 30 us, this 17.5.  fp32 rows
// and dZ are split as in gemm_split.h, with the same fall-back to plain fp32 sums for what the parts cannot carry.
// bf16 rows and dZ go as they are, and logits, loss and input gradients are formed in the order of the separate launches: dZ is
// rounded to bf16, and one that rounds the other way because a sum ran in another order moves the gradients below by
// up to 3e-4 (contraction dealt to eight waves, 143 targets of four layers; it took 16.5 us).
// ------------------------------------------------------------------------------------------
constexpr int TOP_R = 16;          // destination rows of a workgroup per round: the rows of a 16 x 16 MFMA, the k of a 32 x 32 one
constexpr int TOP_W = 8;           // waves of a workgroup
constexpr int TOP_T = 64 * TOP_W;
// More targets than 128 workgroups take in one round: launches of their own.  The batch at hand decides, not the room of its
// context.  (A captured step may be replayed on a batch of more targets: the workgroups then take further rounds.)
constexpr int TOP_MAX_ROWS = 2048;
constexpr int TOP_NMAX = 64;       // classes the kernel takes
constexpr int TOP_DMAX = 384;      // input width it takes
constexpr int TOP_KT = 2 * TOP_DMAX / 32 / TOP_W;      // k-tiles of a wave in the forward product, at most
constexpr int TOP_DZ = TOP_NMAX + 4;                   // row stride of dZ in LDS

// workgroups (= slabs): TOP_R rows each, at most 128 of them
inline int top_slabs(int64_t targets) { return (int)std::min<int64_t>(TOP_MAX_ROWS / TOP_R, std::max<int64_t>(32, gs_ceil_div(targets, TOP_R))); }

struct TopArgs {
    const void *H; int D; int N;
    const int32_t *blk_indptr; const int32_t *edge_row; const int32_t *self_row;
    const uint4 *frag_fwd; const uint4 *frag_gin;       // fp32: the stacked weights and their transpose as split fragments
    const float *W; int Npad;                           // fp32: the stacked weights [2 D x Npad]
    const uint16_t *wt; const uint16_t *ws;             // bf16: the weights [N x 2 D] and [2 D x Npad]
    const float *bias;
    const int64_t *labels; const int32_t *front_top;
    float *logits; float *row_loss;
    float *gin; float *part;
    const GsLevelMeta *meta_up; int S;
};

// row stride of the assembled rows in LDS: whole k-tiles, and four floats on, so that a fragment's rows start in
// different banks
__host__ __device__ inline int top_ldx(int D) { return (2 * D + 31) / 32 * 32 + 4; }
__host__ __device__ inline size_t top_lds_words(int D) {
    return (size_t)TOP_R * top_ldx(D) + TOP_W * TOP_R * TOP_NMAX + TOP_R * TOP_DZ + TOP_R;
}

typedef float floatx4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ floatx4_t mfma16(const uint4 &a, const uint4 &b, const floatx4_t &c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}
// an fp32 operand as its three parts (scaled), a bf16 one (its values held as floats) as one
template <bool HALF> struct TopFrag { uint4 q[HALF ? 1 : 3]; };
template <bool HALF>
__device__ __forceinline__ TopFrag<HALF> top_frag(float (&v)[8]) {
    TopFrag<HALF> f;
    if constexpr (HALF) {
        f.q[0] = make_uint4(cvt2bf(v[0], v[1]), cvt2bf(v[2], v[3]), cvt2bf(v[4], v[5]), cvt2bf(v[6], v[7]));
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] *= SPLIT_SCALE;
        split8(v, f.q);
    }
    return f;
}
// hi: the leading products; lo: the five small ones (fp32)
template <bool HALF, class Acc, class Mul>
__device__ __forceinline__ void top_multiply(const TopFrag<HALF> &a, const TopFrag<HALF> &b, Acc &hi, Acc &lo, const Mul &mul) {
    hi = mul(a.q[0], b.q[0], hi);
    if constexpr (!HALF) {
        lo = mul(a.q[0], b.q[2], lo);
        lo = mul(a.q[0], b.q[1], lo);
        lo = mul(a.q[1], b.q[0], lo);
        lo = mul(a.q[1], b.q[1], lo);
        lo = mul(a.q[2], b.q[0], lo);
    }
}

template <bool HALF>
__global__ __launch_bounds__(TOP_T) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_sage_top_fused(TopArgs a) {
    extern __shared__ __attribute__((aligned(16))) float s_mem[];
    const int D = a.D, N = a.N, D2 = 2 * D, nvec = D >> 2, ldx = top_ldx(D);
    float *s_x = s_mem;                                         // [TOP_R][ldx]
    float *s_p = s_x + (size_t)TOP_R * ldx;                     // [TOP_W][TOP_R x 64]: partial logits in accumulator order
    float *s_dz = s_p + TOP_W * TOP_R * TOP_NMAX;               // [TOP_R][TOP_DZ]
    float *s_inv = s_dz + TOP_R * TOP_DZ;
    // k-tiles and column blocks of a wave whose weights are asked for ahead (what the registers hold)
    constexpr int WF = 2, WG = 1, WFH = 16, WGH = 2;
    const int n1 = a.meta_up->front_off[a.S];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const float inv_n = n1 > 0 ? 1.f / (float)n1 : 0.f;
    float *slab = a.part + (int64_t)blockIdx.x * (D2 + 1) * N;
    const int KT = (D2 + 31) / 32, CB = (N + 15) / 16, KTN = (N + 31) / 32, CBX = (D2 + 15) / 16;
    const int KSH = D2 / 16;        // (bf16: 2 D is a multiple of 16)

    int round = 0;
    for (int r0 = blockIdx.x * TOP_R; round == 0 || r0 < n1; r0 += gridDim.x * TOP_R, ++round) {
        const int rows = max(0, min(TOP_R, n1 - r0));
        // (opaque: what follows from the lane's position, the weights themselves among it, would be worked out in front of
        // the loop over the rounds and kept in registers)
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const int l16 = ln & 15, g = ln >> 4, half = ln >> 5, l32 = ln & 31;
        // fp32: fragment of the weights for 16 columns x 32 k: lane l holds column l % 16 and the eight k that the other
        // operand's lane l holds, granule l / 16 of the k-tile.
        auto weights = [&](const uint4 *frag, int cols, int kt, int k_tiles, int cb) __attribute__((always_inline)) {
            TopFrag<false> f;
            const int kc = min(kt, k_tiles - 1);
            const uint4 *p = frag + ((int64_t)(min(16 * cb, cols - 1) >> 5) * 2 * k_tiles + 2 * kc + (g >> 1)) * 192 + (g & 1) * 32 + (cb & 1) * 16 + l16;
#pragma unroll
            for (int q = 0; q < 3; ++q) f.q[q] = p[q * 64];
            return f;
        };
        // eight k of a row in LDS, those that the weights' fragment holds
        auto row_frag = [&](const float *row, int kt) __attribute__((always_inline)) {
            const float4 u = *reinterpret_cast<const float4 *>(row + 32 * kt + 4 * g);
            const float4 w = *reinterpret_cast<const float4 *>(row + 32 * kt + 16 + 4 * g);
            float v[8] = {u.x, u.y, u.z, u.w, w.x, w.y, w.z, w.w};
            return top_frag<false>(v);
        };
        // bf16: the same for 32 columns x 16 k (lane l: column l % 32, k 8 (l / 32) .. + 7)
        auto weights_h = [&](const uint16_t *w, int ld, int k_end, int cols, int t, int cb) __attribute__((always_inline)) {
            const int k = 16 * t + 8 * half;
            const uint4 v = *reinterpret_cast<const uint4 *>(w + (int64_t)min(32 * cb + l32, cols - 1) * ld + min(k, k_end - 8));
            return k < k_end ? v : make_uint4(0u, 0u, 0u, 0u);
        };
        auto row_frag_h = [&](const float *rows16, int ld, int t) __attribute__((always_inline)) {
            const float *row = rows16 + l16 * ld + 16 * t + 8 * half;
            const float4 u = *reinterpret_cast<const float4 *>(row), w = *reinterpret_cast<const float4 *>(row + 4);
            float v[8] = {u.x, u.y, u.z, u.w, w.x, w.y, w.z, w.w};
            return top_frag<true>(v).q[0];
        };
        __syncthreads();                           // the previous round has finished with the LDS
        // (1) layer input: own lower-layer row | mean over the sampled sources, edges in slot order.  A wave takes two rows,
        // half its lanes the source rows of one each.
        int label = -1;         // (of the half's row)
        // (declared here: the forward product's first weights, which travel while the rows are assembled)
        TopFrag<false> wf[HALF ? 1 : WF][HALF ? 1 : TOP_NMAX / 16];
        uint4 wfh[HALF ? WFH : 1];
        {
            const int row = 2 * wave + half;
            int e0 = 0, e1 = 0, self = 0, id = 0;
            if (row < rows) { e0 = a.blk_indptr[r0 + row]; e1 = a.blk_indptr[r0 + row + 1]; self = a.self_row[r0 + row]; id = a.front_top[r0 + row]; }
            // the first weights of the forward product, behind the offsets (loads come back in order)
            if constexpr (!HALF) {
#pragma unroll
                for (int t = 0; t < WF; ++t)
#pragma unroll
                    for (int c = 0; c < TOP_NMAX / 16; ++c) wf[t][c] = weights(a.frag_fwd, N, wave + t * TOP_W, KT, c);
            } else if (wave < KTN) {
#pragma unroll
                for (int t = 0; t < WFH; ++t) wfh[t] = weights_h(a.wt, D2, D2, N, min(t, KSH - 1), wave);
            }
            const int m = min(64, e1 - e0);
            int src[2];
#pragma unroll
            for (int x = 0; x < 2; ++x) src[x] = 32 * x + l32 < m ? a.edge_row[e0 + 32 * x + l32] : self;
            if (row < rows) label = (int)a.labels[id];
            if (l32 == 0) s_inv[row] = m > 0 ? 1.f / (float)m : 0.f;
            const int m2[2] = {__builtin_amdgcn_readlane(m, 0), __builtin_amdgcn_readlane(m, 32)};
            const int self2[2] = {__builtin_amdgcn_readlane(self, 0), __builtin_amdgcn_readlane(self, 32)};
            // (every lane stays in the loop and in its loads: the source rows are read from the lanes that hold them)
            for (int c0 = 0; c0 < ldx / 4; c0 += 64) {
                const int c = c0 + lane, cc = min(c, nvec - 1);
                FloatVec<4> own[2]{}, sum[2]{};
                if (c0 < nvec) {
#pragma unroll
                    for (int i = 0; i < 2; ++i) own[i] = load_vec<4, HALF>(a.H, (int64_t)self2[i] * nvec + cc);
                    for (int e = 0; e < max(m2[0], m2[1]); e += 8) {
                        FloatVec<4> v[2][8];
#pragma unroll
                        for (int i = 0; i < 2; ++i)
#pragma unroll
                            for (int u = 0; u < 8; ++u) {       // (past a row's edges: its own row, not added)
                                const int r = __builtin_amdgcn_readlane(e + u < 32 ? src[0] : src[1], 32 * i + ((e + u) & 31));
                                v[i][u] = load_vec<4, HALF>(a.H, (int64_t)(e + u < m2[i] ? r : self2[i]) * nvec + cc);
                            }
#pragma unroll
                        for (int i = 0; i < 2; ++i)
#pragma unroll
                            for (int u = 0; u < 8; ++u)
                                if (e + u < m2[i]) add_vec(sum[i], v[i][u]);
                    }
                }
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    float *x = s_x + (2 * wave + i) * ldx;
                    const bool live = 2 * wave + i < rows;
                    const float cnt = m2[i] > 0 ? (float)m2[i] : 1.f;
                    if (c < nvec) {
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            const float mean = sum[i].v[k] / cnt;
                            x[4 * c + k] = live ? own[i].v[k] : 0.f;
                            x[D + 4 * c + k] = live ? (HALF ? bf2f(f2bf(mean)) : mean) : 0.f;
                        }
                    }
                    // (columns behind the row, up to a whole k-tile)
                    if (c >= (D2 >> 2) && c < ldx / 4) *reinterpret_cast<float4 *>(x + 4 * c) = make_float4(0.f, 0.f, 0.f, 0.f);
                }
            }
        }
        __syncthreads();
        // (2) logits.  bf16: a wave takes 32 classes over the whole contraction, in the order of k_sage_linear_fwd_h (the other
        // half of its accumulator's rows is formed and dropped); fp32: the k-tiles are dealt to the waves, their partial sums
        // meet in LDS and are added in wave order
        if constexpr (HALF) {
            if (wave < KTN) {
                floatx16 acc = zero16();
                for (int t0 = 0; t0 < KSH; t0 += WFH) {
#pragma unroll
                    for (int u = 0; u < WFH; ++u) {
                        if (t0 + u < KSH) acc = mfma_bf(row_frag_h(s_x, ldx, t0 + u), wfh[u], acc);
                        wfh[u] = weights_h(a.wt, D2, D2, N, min(t0 + u + WFH, KSH - 1), wave);
                    }
                }
#pragma unroll
                for (int r = 0; r < 8; ++r) s_p[((r >> 2) * 8 + half * 4 + (r & 3)) * TOP_NMAX + 32 * wave + l32] = acc[r];
            }
        } else {
            floatx4_t hi[TOP_NMAX / 16], lo[TOP_NMAX / 16];
#pragma unroll
            for (int c = 0; c < TOP_NMAX / 16; ++c) hi[c] = lo[c] = floatx4_t{0.f, 0.f, 0.f, 0.f};
            const float *row = s_x + l16 * ldx;
#pragma unroll
            for (int t = 0; t < TOP_KT; ++t) {
                const int kt = wave + t * TOP_W;
                if (kt >= KT) break;
                const TopFrag<false> x = row_frag(row, kt);
#pragma unroll
                for (int c = 0; c < TOP_NMAX / 16; ++c)
                    if (c < CB) {
                        const TopFrag<false> w = t < WF ? wf[t < WF ? t : 0][c] : weights(a.frag_fwd, N, kt, KT, c);
                        top_multiply<false>(x, w, hi[c], lo[c], mfma16);
                    }
            }
#pragma unroll
            for (int c = 0; c < TOP_NMAX / 16; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r) s_p[((wave * 4 + c) * 4 + r) * 64 + lane] = hi[c][r] + lo[c][r];
        }
        // the input gradient's first weights travel while the loss is formed
        TopFrag<false> wg[HALF ? 1 : WG][2];
        uint4 wgh[HALF ? WGH : 1][TOP_NMAX / 16];
        if constexpr (HALF) {
#pragma unroll
            for (int c = 0; c < WGH; ++c)
#pragma unroll
                for (int t = 0; t < TOP_NMAX / 16; ++t) wgh[c][t] = weights_h(a.ws, a.Npad, a.Npad, D2, t, min(wave + c * TOP_W, KT - 1));
        } else {
#pragma unroll
            for (int c = 0; c < WG; ++c)
#pragma unroll
                for (int t = 0; t < 2; ++t) wg[c][t] = weights(a.frag_gin, D2, t, KTN, min(wave + c * TOP_W, CBX - 1));
        }
        __syncthreads();
        // loss: a wave takes two rows, a lane a class (row r, column n of a block: register r % 4 of lane 16 (r / 4) + n)
        float z2[2];
        bool ok = true;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = 2 * wave + i;
            float sum = 0.f;
            if constexpr (HALF) {
                sum = lane < N ? s_p[r * TOP_NMAX + lane] : 0.f;
            } else {
#pragma unroll
                for (int w = 0; w < TOP_W; ++w) sum += s_p[((w * 4 + (lane >> 4)) * 4 + (r & 3)) * 64 + 16 * (r >> 2) + l16];
                sum *= SPLIT_UNSCALE;
            }
            z2[i] = sum;
            if (lane < N) ok = ok && fabsf(z2[i]) < INFINITY;
        }
        if (!HALF && __ballot(!ok) != 0ull) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                int l = lane;
                asm volatile("" : "+v"(l));
                const float *x = s_x + (2 * wave + i) * ldx, *w = a.W + min(l, N - 1);
                float sum = 0.f;
#pragma unroll 1
                for (int k = 0; k < D2; ++k) sum += x[k] * w[(int64_t)k * a.Npad];
                z2[i] = sum;
            }
        }
        // (both rows at once: two chains of exchanges side by side)
        float mx[2], ex[2], sum[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) mx[i] = z2[i] = lane < N ? z2[i] + a.bias[lane] : -3.4e38f;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
#pragma unroll
            for (int i = 0; i < 2; ++i) mx[i] = fmaxf(mx[i], __shfl_xor(mx[i], o));
#pragma unroll
        for (int i = 0; i < 2; ++i) sum[i] = ex[i] = lane < N ? __expf(z2[i] - mx[i]) : 0.f;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
#pragma unroll
            for (int i = 0; i < 2; ++i) sum[i] += __shfl_xor(sum[i], o);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = 2 * wave + i, row = r0 + r;
            const int y = __builtin_amdgcn_readlane(label, 32 * i);
            const bool known = y >= 0 && y < N;
            const float zy = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(z2[i]), known ? y : 0));
            float dz = 0.f;
            if (r < rows) {
                if (lane < N) {
                    a.logits[(int64_t)row * N + lane] = z2[i];
                    const float p = HALF ? ex[i] * (1.f / sum[i]) : ex[i] / sum[i];      // (bf16: as k_softmax_xent)
                    dz = (p - (lane == y ? 1.f : 0.f)) * inv_n;
                }
                if (lane == 0 && a.row_loss) a.row_loss[row] = known ? (logf(sum[i]) + mx[i] - zy) : 0.f;
            }
            // (bf16: dZ is rounded where it enters a product)
            s_dz[r * TOP_DZ + lane] = HALF ? bf2f(f2bf(dz)) : dz;
        }
        __syncthreads();
        // (3a) input gradients of the rows: [dH_self | dMean / cnt] = dZ W^T, the column blocks dealt to the waves (bf16: 32
        // columns, in the order of k_sage_grad_in_h)
        if constexpr (HALF) {
            uint4 dz[TOP_NMAX / 16];
#pragma unroll
            for (int t = 0; t < TOP_NMAX / 16; ++t) dz[t] = row_frag_h(s_dz, TOP_DZ, t);
            for (int c0 = 0; c0 * TOP_W < KT; c0 += WGH) {
                if (c0 > 0) {
#pragma unroll
                    for (int c = 0; c < WGH; ++c)
#pragma unroll
                        for (int t = 0; t < TOP_NMAX / 16; ++t)
                            wgh[c][t] = weights_h(a.ws, a.Npad, a.Npad, D2, t, min(wave + (c0 + c) * TOP_W, KT - 1));
                }
#pragma unroll
                for (int c = 0; c < WGH; ++c) {
                    const int cb = wave + (c0 + c) * TOP_W;
                    if (cb >= KT) break;
                    floatx16 acc = zero16();
#pragma unroll
                    for (int t = 0; t < TOP_NMAX / 16; ++t)
                        if (t < CB) acc = mfma_bf(dz[t], wgh[c][t], acc);
                    const int col = 32 * cb + l32;
#pragma unroll
                    for (int r = 0; r < 8; ++r) {
                        const int row = (r >> 2) * 8 + half * 4 + (r & 3);
                        if (row < rows && col < D2) a.gin[(int64_t)(r0 + row) * D2 + col] = col < D ? acc[r] : acc[r] * s_inv[row];
                    }
                }
            }
        } else {
            TopFrag<false> dz[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) dz[t] = row_frag(s_dz + l16 * TOP_DZ, t);
            // (a round's weights are asked for together; blocks past the last one are formed again and not stored)
            constexpr int AHEAD = WG > 3 ? WG : 3;
            for (int c0 = 0; c0 * TOP_W < CBX; c0 += AHEAD) {
                TopFrag<false> w[AHEAD][2];
#pragma unroll
                for (int c = 0; c < AHEAD; ++c)
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        if (c < WG && c0 == 0) w[c][t] = wg[c < WG ? c : 0][t];
                        else w[c][t] = weights(a.frag_gin, D2, t, KTN, min(wave + (c0 + c) * TOP_W, CBX - 1));
                    }
#pragma unroll
                for (int c = 0; c < AHEAD; ++c) {
                    const int cb = wave + (c0 + c) * TOP_W;
                    if (cb >= CBX) break;
                    floatx4_t hi = {0.f, 0.f, 0.f, 0.f}, lo = hi;
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        if (t < KTN) top_multiply<false>(dz[t], w[c][t], hi, lo, mfma16);
                    float v[4];
                    bool fine = true;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        v[r] = (hi[r] + lo[r]) * SPLIT_UNSCALE;
                        fine = fine && fabsf(v[r]) < INFINITY;
                    }
                    const int col = 16 * cb + l16;
                    if (N < SPLIT_MIN_K || __ballot(!fine) != 0ull) {
                        int l = lane;
                        asm volatile("" : "+v"(l));
                        const float *w = a.W + (int64_t)min(16 * cb + (l & 15), D2 - 1) * a.Npad, *d = s_dz + 4 * (l >> 4) * TOP_DZ;
#pragma unroll
                        for (int r = 0; r < 4; ++r) v[r] = 0.f;
#pragma unroll 1
                        for (int n = 0; n < N; ++n) {
#pragma unroll
                            for (int r = 0; r < 4; ++r) v[r] += d[r * TOP_DZ + n] * w[n];
                        }
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (4 * g + r < rows && col < D2) a.gin[(int64_t)(r0 + 4 * g + r) * D2 + col] = col < D ? v[r] : v[r] * s_inv[4 * g + r];
                }
            }
        }
        // (3b) this workgroup's share of X^T dZ, 32 inputs x 32 classes at a time, and of the column sums of dZ, into its slab
        // (bounds-checked buffer accesses: rows and columns past the edge get an offset past the slab's end)
        auto rsrc = __builtin_amdgcn_make_buffer_rsrc(slab, 0, (D2 + 1) * N * 4, 0x00020000);
        auto keep = [&](int at, float v) __attribute__((always_inline)) {
            if (round > 0) v += __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, at, 0, 0));
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rsrc, at, 0, 0);
        };
        {
            auto column = [&](const float *p, int ld) __attribute__((always_inline)) {
                float v[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = p[(8 * half + i) * ld];
                return top_frag<HALF>(v);
            };
            TopFrag<HALF> dz[2];
#pragma unroll
            for (int b = 0; b < 2; ++b) dz[b] = column(s_dz + 32 * b + l32, TOP_DZ);
#pragma unroll 1
            for (int mb = wave; mb < KT; mb += TOP_W) {
                const TopFrag<HALF> x = column(s_x + 32 * mb + l32, ldx);
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    if (b >= KTN) break;
                    floatx16 hi = zero16(), lo = zero16();
                    top_multiply<HALF>(x, dz[b], hi, lo, mfma_bf);
                    if (!HALF) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) hi[r] = (hi[r] + lo[r]) * SPLIT_UNSCALE;
                    }
                    const int n = 32 * b + l32;
                    if (!HALF && (rows < SPLIT_MIN_K || __ballot(!finite16(hi)) != 0ull)) {
                        int l = lane;
                        asm volatile("" : "+v"(l));
                        const float *x0 = s_x + 32 * mb + 4 * (l >> 5), *d = s_dz + 32 * b + (l & 31);
                        hi = zero16();
#pragma unroll 1
                        for (int i = 0; i < rows; ++i) {
#pragma unroll
                            for (int r = 0; r < 16; ++r) hi[r] += x0[i * ldx + (r >> 2) * 8 + (r & 3)] * d[i * TOP_DZ];
                        }
                    }
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int k = 32 * mb + (r >> 2) * 8 + half * 4 + (r & 3);
                        keep(k < D2 && n < N ? (k * N + n) * 4 : 0x7FFFFFFC, hi[r]);
                    }
                }
            }
            if (wave == TOP_W - 1 && lane < N) {        // the bias gradient
                float sum = 0.f;
#pragma unroll
                for (int r = 0; r < TOP_R; ++r) sum += s_dz[r * TOP_DZ + lane];
                keep((D2 * N + lane) * 4, sum);
            }
        }
    }
}

#include "sage_bf16.h"
#include "gemm_bf16_rows.h"

// The streaming bf16 row-block kernel takes a product when the contraction is 256 or 512, the output
// rows are whole 16-byte granules and the level is large enough (by its bound) to fill the chip.
constexpr int64_t RB_MIN_ROWS = 32768;
constexpr int RB_FWD_STAGES = 4;        // (six stages fit beside the forward product's bf16 patch and measured the same: 197 against 198 us)
bool rows_gemm_fits(int64_t ub_rows, int K, int NB, int granule) {
    return (K == 256 || K == 512) && NB % granule == 0 && ub_rows >= RB_MIN_ROWS;
}
// weight gradients of layer l through the streaming kernel: dZ held in bf16 (a level below the top
// one whose width allows 16-byte rows), whole 16-byte column groups, a level that fills the chip
bool grad_w_streams(const gsplit_sage_params *p, int l, int L, int64_t ub_rows) {
    const int D = p->dims[l], N = p->dims[l + 1];
    return p->dtype == GSPLIT_BF16 && l < L - 1 && N % 8 == 0 && N >= 128 && (2 * D) % 8 == 0 && 2 * D >= 128 &&
           ub_rows >= RB_MIN_ROWS;
}
// Do the weight gradients of layer l (float, by the bound on its rows) go with the pull of its input gradients?
bool grad_with_pull(const gsplit_sage_params *p, int l, int64_t ub) {
    return p->dtype == GSPLIT_F32 && l > 0 && ub <= PULL_GRAD_ROWS && split_grad_block(ub, 2 * p->dims[l], p->dims[l + 1]) == 64;
}
// Does the forward product into level l (1 .. L - 1) of a training step leave a bit per activation for the pull of its gradient?
// Where the pull is a launch of its own, the product one of those that fill the chip, and a row wide enough: 274k rows of 256 are
// pulled in 147 us instead of 173, behind a product of 218 instead of 212; of 128 in 104 instead of 121, of 96 96 / 103, of 72
// 94 / 94.
// (bf16: the streaming product took 126 -> 141 us for the bits of 546k x 256 and the weight gradients behind the pull 149 -> 160; the
// pull gave 341 -> 318.)  Only within gsplit_sage_step, whose backward pass is sure to come: a forward pass by itself would pay
// for nothing (skewed workload's 792 -> 798 us), and one that may be replayed or not before a backward pass of its own cannot
// be told from the host to have left them.
constexpr int RELU_BITS_MIN = 96;
bool keeps_relu_bits(const gsplit_ctx *ctx, const gsplit_sage_params *p, int l) {
    const int K = 2 * p->dims[l - 1], N = p->dims[l];
    const int64_t ub = ctx->ub_front[l];
    return p->dtype == GSPLIT_F32 && N >= RELU_BITS_MIN && N % 4 == 0 && p->dims[l - 1] % 2 == 0 && !(split_forms(ub, N, K, 1, true, ctx->n_cu) & FORM_FEW) &&
           !grad_with_pull(p, l, ctx->ub_front[l + 1]);
}
// one workgroup per compute unit, a multiple of (8 XCDs x column blocks)
unsigned rows_gemm_grid(const gsplit_ctx *ctx, int NB, int BN) {
    const int nb = (NB + BN - 1) / BN;
    return (unsigned)(std::max(1, ctx->n_cu / (8 * nb)) * 8 * nb);
}

int ensure_buffers(gsplit_ctx *ctx, const gsplit_sage_params *p) {
    GsSageBuf &sb = ctx->sage;
    const int L = ctx->L;
    bool same = sb.ready && sb.dtype == p->dtype;
    for (int l = 0; same && l <= L; ++l) same = sb.dims[l] == p->dims[l];
    if (same) return GSPLIT_OK;
    if (sb.ready) return gs_fail(ctx, GSPLIT_ESTATE, "sage: model shape changed; create a new context");
    const size_t esz = p->dtype == GSPLIT_BF16 ? 2 : 4;
    for (int l = 1; l < L; ++l) {
        int rc = gs_alloc(ctx, &sb.hidden[l], esz * ctx->ub_front[l] * p->dims[l], "hidden");
        if (rc) return rc;
        rc = gs_alloc(ctx, (void **)&sb.ghid[l], sizeof(float) * ctx->ub_front[l] * p->dims[l], "ghid");
        if (rc) return rc;
    }
    for (int l = 0; l < L; ++l) {
        int rc = gs_alloc(ctx, &sb.xin[l], esz * ctx->ub_front[l + 1] * 2 * p->dims[l], "layer input");
        if (rc) return rc;
        if (p->dtype == GSPLIT_F32) {
            const int64_t np = (p->dims[l + 1] + 3) & ~3;
            rc = gs_alloc(ctx, (void **)&sb.wstack32[l], sizeof(float) * 2 * p->dims[l] * np, "stacked weights");
            if (rc) return rc;
            rc = gs_alloc(ctx, (void **)&sb.wfrag_fwd[l], 16 * split_frag_words(2 * p->dims[l], p->dims[l + 1]), "split weights");
            if (rc) return rc;
            if (l > 0) rc = gs_alloc(ctx, (void **)&sb.wfrag_gin[l], 16 * split_frag_words(p->dims[l + 1], 2 * p->dims[l]), "split weights");
        } else {
            const int64_t np = (p->dims[l + 1] + 7) & ~7;
            rc = gs_alloc(ctx, (void **)&sb.wstack[l], 2 * (size_t)(2 * p->dims[l]) * np, "bf16 weights");
            if (rc) return rc;
            rc = gs_alloc(ctx, (void **)&sb.wtrans[l], 2 * (size_t)p->dims[l + 1] * 2 * p->dims[l], "bf16 weights^T");
        }
        if (rc) return rc;
        rc = gs_alloc(ctx, (void **)&sb.inv_cnt[l], sizeof(float) * (ctx->ub_front[l + 1] + RB_BM), "inverse counts");
        if (rc) return rc;
    }
    for (int l = 0; l < L; ++l) {
        // split-K geometry of the weight-gradient product: about as many workgroups as the chip
        // holds at once (three per compute unit); how many of the chunks are used is decided on
        // the device from the actual row count
        const int m_rows = 2 * p->dims[l] + 1;    // (bf16: plus the row of ones)
        const int tiles = (int)(gs_ceil_div(m_rows, TileMid::BM) * gs_ceil_div(p->dims[l + 1], TileMid::BN));
        int64_t chunks = gs_ceil_div(std::max<int64_t>(8, (int64_t)ctx->n_cu * 3 / tiles), 8) * 8;
        if (p->dtype == GSPLIT_F32) chunks = split_grad_chunks(ctx->ub_front[l + 1], 2 * p->dims[l], p->dims[l + 1], 1, ctx->n_cu);
        sb.nchunk[l] = (int)chunks;
        // a bf16 level below the top one that can reach gwh_min_rows() rows: when it does (decided on the
        // device), one workgroup per compute unit forms a whole 256 x 256 block over its chunk of rows
        sb.stream_rows[l] = gwh_min_rows(tiles);
        if (const char *e = std::getenv("GSPLIT_GRADW_STREAM_ROWS")) {
            const long v = std::strtol(e, nullptr, 10);
            if (v >= 64 && v <= (1l << 30)) sb.stream_rows[l] = (int)v;
        }
        sb.gw_stream[l] = grad_w_streams(p, l, L, ctx->ub_front[l + 1]) && ctx->ub_front[l + 1] >= sb.stream_rows[l];
        sb.stream_nchunk[l] = 0;
        if (sb.gw_stream[l]) {
            const int big = (int)(gs_ceil_div(2 * p->dims[l], GWH_B) * gs_ceil_div(p->dims[l + 1], GWH_B));
            sb.stream_nchunk[l] = std::max(8, ctx->n_cu / big / 8 * 8);
            chunks = std::max<int64_t>(chunks, sb.stream_nchunk[l]);
        }
        // the fused top-layer kernel writes one slab per workgroup
        int64_t slabs = chunks;
        if (l == L - 1) {
            slabs = std::max<int64_t>(slabs, top_slabs(ctx->ub_front[L]));
        }
        int rc = gs_alloc(ctx, (void **)&sb.gw_part[l],
                          sizeof(float) * slabs * (2 * p->dims[l] + 1) * p->dims[l + 1], "weight-gradient partials");
        if (rc) return rc;
    }
    {
        int rc = gs_alloc(ctx, (void **)&sb.glog, sizeof(float) * ctx->ub_front[L] * p->dims[L], "loss gradient");
        if (rc) return rc;
    }
    int64_t gtmp_words = 1;
    for (int l = 1; l < L; ++l) gtmp_words = std::max<int64_t>(gtmp_words, ctx->ub_front[l + 1] * 2 * p->dims[l]);
    {
        int rc = gs_alloc(ctx, (void **)&sb.gtmp, sizeof(float) * gtmp_words, "input gradients");
        if (rc) return rc;
    }
    // the fused top-layer kernel takes up to 85 KiB of dynamic LDS (a gfx950 workgroup may use all 160 KiB)
    GS_HIP(ctx, hipFuncSetAttribute((const void *)(p->dtype == GSPLIT_BF16 ? k_sage_top_fused<true> : k_sage_top_fused<false>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)(sizeof(float) * top_lds_words(TOP_DMAX))));
    sb.dtype = p->dtype;
    for (int l = 0; l <= L; ++l) sb.dims[l] = p->dims[l];
    sb.ready = true;
    return GSPLIT_OK;
}

// The bits of the levels that a step keeps them for, by its first call.  Without them (under capture, where nothing can be
// allocated, or where they do not fit) the pull reads the activations.
void ensure_relu_bits(gsplit_ctx *ctx, const gsplit_sage_params *p, hipStream_t st) {
    GsSageBuf &sb = ctx->sage;
    if (sb.bits_ready) return;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cap) != hipSuccess) (void)hipGetLastError();
    if (cap != hipStreamCaptureStatusNone) return;
    const std::string err = ctx->err;
    for (int l = 1; l < ctx->L; ++l)
        if (keeps_relu_bits(ctx, p, l) &&
            gs_alloc(ctx, (void **)&sb.bits[l], sizeof(uint32_t) * ctx->ub_front[l] * ((p->dims[l] + 31) / 32), "ReLU bits") != GSPLIT_OK)
            ctx->err = err;
    sb.bits_ready = true;
}

int check_params(gsplit_ctx *ctx, const gsplit_sage_params *p, const char *who) {
    if (!p || !p->dims || !p->d_w_self || !p->d_w_neigh || !p->d_bias)
        return gs_fail(ctx, GSPLIT_EINVAL, std::string(who) + ": NULL parameter block");
    if (p->dtype != GSPLIT_F32 && p->dtype != GSPLIT_BF16)
        return gs_fail(ctx, GSPLIT_EINVAL, std::string(who) + ": dtype must be GSPLIT_F32 or GSPLIT_BF16");
    if (p->dtype == GSPLIT_BF16)
        for (int l = 0; l < ctx->L; ++l)
            if (p->dims[l] % 4 != 0)
                return gs_fail(ctx, GSPLIT_EINVAL, std::string(who) + ": GSPLIT_BF16 needs input and hidden widths "
                                                                      "that are multiples of 4");
    for (int l = 0; l <= ctx->L; ++l)
        if (p->dims[l] < 1 || p->dims[l] > 4096)
            return gs_fail(ctx, GSPLIT_EINVAL, std::string(who) + ": layer width out of range");
    for (int l = 0; l < ctx->L; ++l)
        if (!p->d_w_self[l] || !p->d_w_neigh[l] || !p->d_bias[l])
            return gs_fail(ctx, GSPLIT_EINVAL, std::string(who) + ": NULL weight pointer");
    return GSPLIT_OK;
}

// Edges in flight.  An edge that a row does not have is a load all the same (of its own row): with sixteen whatever the
// fanout, 75k bf16 rows of 156 values and 5 edges took 178 us, with eight 111, three small layers of 3 to 7 edges 19.3 and
// 15.5.  From nine on the depth is worth more than the loads: ten for a fanout of 10 or 20 247 -> 260 us (567k bf16 rows of
// 128, 10 edges), 420 -> 431 (266k float rows of 128, 20 edges).
inline int assemble_step(int fan) { return fan <= 4 ? 4 : fan <= 8 ? 8 : 16; }

// weights (may be NULL; a WeightStack for float rows, a WeightPrep for bf16 rows): laid out behind the assembly's own
// workgroups, `words` of the largest layer
template <class Weights>
void launch_assemble(gsplit_ctx *ctx, int l, const void *hin, int D, hipStream_t st, const Weights *weights, int64_t words) {
    constexpr bool half = std::is_same<Weights, WeightPrep>::value;
    const GsLayerBuf &B = ctx->layer[l];
    const GsLevelMeta *mu = ctx->d_meta + (l + 1);
    const int64_t ub = ctx->ub_front[l + 1];
    GsTimeScope ts(ctx, "assemble_input", l, st);
    const int n_stack = weights ? (int)std::min<int64_t>(128, gs_ceil_div(words, 256)) : 0;
    const Weights none{};
    const Weights &w = weights ? *weights : none;
    const int extra = n_stack * Weights::KINDS * ctx->L;
    const int step = assemble_step(ctx->fan[l]);
#define GS_ASSEMBLE_S(LPR, STEP, ...)                                                                        \
    do {                                                                                                     \
        const int n_main = grid_1d(ctx, ub * LPR);                                                           \
        hipLaunchKernelGGL((k_assemble_input<LPR, STEP, __VA_ARGS__>), dim3(n_main + extra), dim3(256), 0, st, hin, D, \
                           B.blk_indptr, B.edge_row, B.self_row, mu, ctx->S, ctx->fan[l], ctx->sage.xin[l],  \
                           ctx->sage.inv_cnt[l], n_main, w, n_stack);                                        \
    } while (0)
#define GS_ASSEMBLE(LPR, ...)                                                \
    do {                                                                     \
        if (step == 4) GS_ASSEMBLE_S(LPR, 4, __VA_ARGS__);                   \
        else if (step == 8 || LPR == 8) GS_ASSEMBLE_S(LPR, 8, __VA_ARGS__);  \
        else GS_ASSEMBLE_S((LPR == 8 ? 16 : LPR), 16, __VA_ARGS__);          \
    } while (0)
#define GS_ASSEMBLE_W(...)                                                   \
    do {                                                                     \
        const int pieces = D / __VA_ARGS__::VALUES;                          \
        if (pieces <= 8) GS_ASSEMBLE(8, __VA_ARGS__);                        \
        else if (pieces <= 16) GS_ASSEMBLE(16, __VA_ARGS__);                 \
        else if (pieces <= 32) GS_ASSEMBLE(32, __VA_ARGS__);                 \
        else GS_ASSEMBLE(64, __VA_ARGS__);                                   \
    } while (0)
    // the widest pieces that the width and the alignment of the rows allow
    if constexpr (half) {
        if (D % 8 == 0) GS_ASSEMBLE_W(PieceH<4>);
        else GS_ASSEMBLE_W(PieceH<2>);
    } else {
        if (D % 4 == 0 && aligned16(hin)) GS_ASSEMBLE_W(PieceF<4>);
        else if (D % 2 == 0 && ((uintptr_t)hin & 7u) == 0) GS_ASSEMBLE_W(PieceF<2>);
        else GS_ASSEMBLE_W(PieceF<1>);
    }
#undef GS_ASSEMBLE_W
#undef GS_ASSEMBLE
#undef GS_ASSEMBLE_S
}

}  // namespace

namespace {

// forward layers 0 .. l_end - 1 (l_end = L: the whole pass, logits included); in_step: the backward pass follows in the same call
int sage_forward(gsplit_ctx *ctx, const gsplit_sage_params *p, const void *d_feat_local, float *d_logits,
                 hipStream_t st, int l_end, bool in_step) {
    const int L = ctx->L, S = ctx->S;
    GsSageBuf &sb = ctx->sage;
    if (p->dtype == GSPLIT_BF16) {
        if (!aligned16(d_feat_local)) return gs_fail(ctx, GSPLIT_EINVAL, "gsplit_sage_fwd: features must be 16-byte aligned");
        WeightPrep wp{};
        int64_t wmax = 1;
        for (int l = 0; l < L; ++l) {
            wp.ws[l] = (const float *)p->d_w_self[l]; wp.wn[l] = (const float *)p->d_w_neigh[l];
            wp.stacked[l] = sb.wstack[l]; wp.transposed[l] = sb.wtrans[l];
            wp.D[l] = p->dims[l]; wp.N[l] = p->dims[l + 1];
            wmax = std::max<int64_t>(wmax, (int64_t)2 * p->dims[l] * ((p->dims[l + 1] + 7) & ~7));
        }
        for (int l = 0; l < l_end; ++l) {
            const int D = p->dims[l], N = p->dims[l + 1];
            const uint16_t *hin = l == 0 ? (const uint16_t *)d_feat_local : (const uint16_t *)sb.hidden[l];
            const GsLevelMeta *mu = ctx->d_meta + (l + 1);
            const int64_t ub = ctx->ub_front[l + 1];
            launch_assemble(ctx, l, hin, D, st, l == 0 ? &wp : nullptr, wmax);
            MatRowsH x{(const uint16_t *)sb.xin[l], 0, 2 * D};
            MatRowsH wt{sb.wtrans[l], N, 2 * D};
            EpiFwdH epi{l == L - 1 ? (void *)d_logits : sb.hidden[l + 1], (const float *)p->d_bias[l], N, 0,
                        l < L - 1 ? 1 : 0, l == L - 1 ? 1 : 0};
            GsTimeScope ts(ctx, "linear_fwd", l, st);
            if (l < L - 1 && rows_gemm_fits(ub, 2 * D, N, 8)) {
                RbEpi re{sb.hidden[l + 1], N, (const float *)p->d_bias[l], nullptr, 0, 1};
                if (2 * D == 256)
                    hipLaunchKernelGGL((k_rows_gemm_hb<16, false, RB_FWD_STAGES>), dim3(rows_gemm_grid(ctx, N, 256)), dim3(GNT), 0, st,
                                       x.p, wt.p, N, re, mu, S);
                else
                    hipLaunchKernelGGL((k_rows_gemm_hb<32, false, RB_FWD_STAGES>), dim3(rows_gemm_grid(ctx, N, 128)), dim3(GNT), 0, st,
                                       x.p, wt.p, N, re, mu, S);
            } else {
                dim3 grid(row_block_grid<TileMid>(ctx, ub, N));
                hipLaunchKernelGGL(k_sage_linear_fwd_h, grid, dim3(GNT), 0, st, x, wt, epi, mu, S);
            }
        }
        GS_HIP(ctx, hipGetLastError());
        sb.fwd_done = l_end == L;
        sb.fwd_batch = ctx->batch_id;
        return GSPLIT_OK;
    }
    WeightStack ws{};
    int64_t stack_words = 1;
    {
        int64_t wmax = 1;
        for (int l = 0; l < L; ++l) {
            ws.ws[l] = (const float *)p->d_w_self[l]; ws.wn[l] = (const float *)p->d_w_neigh[l];
            ws.stacked[l] = sb.wstack32[l]; ws.frag_fwd[l] = sb.wfrag_fwd[l]; ws.frag_gin[l] = sb.wfrag_gin[l]; ws.D[l] = p->dims[l]; ws.N[l] = p->dims[l + 1];
            wmax = std::max<int64_t>(wmax, (int64_t)2 * p->dims[l] * ((p->dims[l + 1] + 3) & ~3));
        }
        stack_words = wmax;
    }
    for (int l = 0; l < l_end; ++l) {
        const int D = p->dims[l], N = p->dims[l + 1];
        const float *hin = l == 0 ? (const float *)d_feat_local : (const float *)sb.hidden[l];
        float *hout = l == L - 1 ? d_logits : (float *)sb.hidden[l + 1];
        const GsLevelMeta *mu = ctx->d_meta + (l + 1);
        // (the stacked weights are first needed by the bottom layer's product: its input assembly carries the stacking)
        launch_assemble(ctx, l, hin, D, st, l == 0 ? &ws : nullptr, stack_words);
        // Z = [H_self | mean] * [W_self; W_neigh] + b, ReLU except on the last layer
        const SplitA a{(const float *)sb.xin[l], 2 * D, 0, 2 * D};
        const SplitB b{sb.wfrag_fwd[l], sb.wstack32[l], (N + 3) & ~3, 1, N};
        const SplitEpiBias epi{hout, N, (const float *)p->d_bias[l], l < L - 1 ? 1 : 0};
        const bool va = D % 2 == 0;   // rows of the assembled input are 2 * D floats: 16-byte aligned
        GsTimeScope ts(ctx, "linear_fwd", l, st);
        if (in_step && l < L - 1 && sb.bits[l + 1])
            launch_rows_split(ctx, st, ctx->ub_front[l + 1], va, a, b, SplitEpiRelu{epi, sb.bits[l + 1], (N + 31) / 32}, mu);
        else launch_rows_split(ctx, st, ctx->ub_front[l + 1], va, a, b, epi, mu);
    }
    GS_HIP(ctx, hipGetLastError());
    sb.fwd_done = l_end == L;
    sb.fwd_batch = ctx->batch_id;
    return GSPLIT_OK;
}

}  // namespace

extern "C" int gsplit_sage_fwd(gsplit_ctx *ctx, const gsplit_sage_params *p, const void *d_feat_local,
                               float *d_logits, void *stream) {
    if (!ctx) return GSPLIT_EINVAL;
    int rc = check_params(ctx, p, "gsplit_sage_fwd");
    if (rc) return rc;
    if (!d_feat_local || !d_logits) return gs_fail(ctx, GSPLIT_EINVAL, "gsplit_sage_fwd: NULL buffer");
    if (ctx->batch_id == 0) return gs_fail(ctx, GSPLIT_ESTATE, "gsplit_sage_fwd: no batch");
    rc = ensure_buffers(ctx, p);
    if (rc) return rc;
    return sage_forward(ctx, p, d_feat_local, d_logits, (hipStream_t)stream, ctx->L, false);
}


namespace {

// backward pass, top layer down.  top_chunks > 0: the fused top-layer kernel has already left the top
// layer's input gradients in gtmp and its weight-gradient partials in that many slabs.  in_step: as above.
int sage_backward(gsplit_ctx *ctx, const gsplit_sage_params *p, const float *d_grad_logits, float *const *d_gw_self,
                  float *const *d_gw_neigh, float *const *d_gbias, hipStream_t st, int top_chunks, bool in_step) {
    GsSageBuf &sb = ctx->sage;
    const int L = ctx->L, S = ctx->S;
    for (int l = L - 1; l >= 0; --l) {
        const int D = p->dims[l], N = p->dims[l + 1];
        const GsLayerBuf &B = ctx->layer[l];
        const GsLevelMeta *mu = ctx->d_meta + (l + 1);
        const float *dH = l == L - 1 ? d_grad_logits : sb.ghid[l + 1];
        const int64_t ub = ctx->ub_front[l + 1];
        const bool h16 = p->dtype == GSPLIT_BF16;
        // bf16 storage: below the top level dZ is held in bf16 when its width allows 16-byte rows
        const bool dz_h = h16 && l < L - 1 && N % 8 == 0;
        MatRows dz{dH, 0, N};
        MatRowsH dzh{(const uint16_t *)dH, 0, N};
        // weight and bias gradients, summed over all splits: X^T dZ with the layer input X
        // assembled by the forward pass
        const EpiGradW ew{sb.gw_part[l], 2 * D + 1, N};
        const bool vin = D % 2 == 0;
        const bool vdz = N % 4 == 0 && aligned16(dH);
        const bool done_above = top_chunks > 0 && l == L - 1;
        const SplitGrad grad{(const float *)sb.xin[l], 2 * D, 2 * D, dH, N, N, sb.gw_part[l], 1, sb.nchunk[l]};
        const bool with_pull = !done_above && grad_with_pull(p, l, ub);
        if (!done_above && !with_pull) {
            GsTimeScope ts(ctx, "grad_w", l, st);
            if (h16) {
                MatRowsOnesH inh{(const uint16_t *)sb.xin[l], 0, 2 * D};
                const int tm = (int)gs_ceil_div(ew.rows, GBM), tn = (int)gs_ceil_div(ew.N, GBN);
                dim3 grid((unsigned)(sb.nchunk[l] * tm * tn));
                if (sb.gw_stream[l]) {
                    // two launches, one of which finds the level on its side of the bar and works
                    const int bm = (int)gs_ceil_div(2 * D, GWH_B), bn = (int)gs_ceil_div(N, GWH_B);
                    hipLaunchKernelGGL(k_grad_w_hb, dim3((unsigned)(sb.stream_nchunk[l] * bm * bn)), dim3(GWH_NT), 0, st, inh.p,
                                       2 * D, dzh.p, N, sb.gw_part[l], sb.stream_nchunk[l], GWH_ROWS_MIN, bm, bn, mu, S,
                                       sb.stream_rows[l]);
                }
                if (dz_h)
                    hipLaunchKernelGGL((k_sage_grad_w_h<PatchDzH, MatRowsH>), grid, dim3(GNT), 0, st, inh, dzh, ew,
                                       sb.nchunk[l], GRAD_W_ROWS_MIN, tm, tn, mu, S, sb.gw_stream[l] ? sb.stream_rows[l] : 0);
                else if (vdz)
                    hipLaunchKernelGGL((k_sage_grad_w_h<PatchDz<4>, MatRows>), grid, dim3(GNT), 0, st, inh, dz, ew,
                                       sb.nchunk[l], GRAD_W_ROWS_MIN, tm, tn, mu, S, 0);
                else
                    hipLaunchKernelGGL((k_sage_grad_w_h<PatchDz<1>, MatRows>), grid, dim3(GNT), 0, st, inh, dz, ew,
                                       sb.nchunk[l], GRAD_W_ROWS_MIN, tm, tn, mu, S, 0);
            } else {
                launch_grad_w_split(st, ub, vin, vdz, grad, mu, S);
            }
        }
        if (l > 0) {
            const GsLevelMeta *ml = ctx->d_meta + l;
            EpiGradIn ei{sb.gtmp, sb.inv_cnt[l], D, 0};
            if (!done_above) {
                GsTimeScope ts(ctx, "grad_in", l, st);
                if (h16) {
                    dim3 grid(row_block_grid<TileMid>(ctx, ub, 2 * D));
                    MatRowsH wsk{sb.wstack[l], 2 * D, (N + 7) & ~7};
                    if (dz_h && rows_gemm_fits(ub, N, 2 * D, 4)) {
                        RbEpi re{sb.gtmp, 2 * D, nullptr, sb.inv_cnt[l], D, 0};
                        if (N == 256)
                            hipLaunchKernelGGL((k_rows_gemm_hb<16, true, 4>), dim3(rows_gemm_grid(ctx, 2 * D, 256)), dim3(GNT), 0,
                                               st, dzh.p, wsk.p, 2 * D, re, mu, S);
                        else
                            hipLaunchKernelGGL((k_rows_gemm_hb<32, true, 4>), dim3(rows_gemm_grid(ctx, 2 * D, 128)), dim3(GNT), 0,
                                               st, dzh.p, wsk.p, 2 * D, re, mu, S);
                    } else if (dz_h) hipLaunchKernelGGL(k_sage_grad_in_hh, grid, dim3(GNT), 0, st, dzh, wsk, ei, mu, S);
                    else if (vdz) hipLaunchKernelGGL((k_sage_grad_in_h<4>), grid, dim3(GNT), 0, st, dz, wsk, ei, mu, S);
                    else hipLaunchKernelGGL((k_sage_grad_in_h<1>), grid, dim3(GNT), 0, st, dz, wsk, ei, mu, S);
                } else {
                    // [dH_self | dMean / cnt] = dZ * [W_self; W_neigh]^T per destination row
                    const SplitA sa{dH, N, 0, N};
                    const SplitB sw{sb.wfrag_gin[l], sb.wstack32[l], 1, (N + 3) & ~3, 2 * D};
                    const SplitEpiScale se{sb.gtmp, 2 * D, sb.inv_cnt[l], D};
                    launch_rows_split(ctx, st, ub, vdz, sa, sw, se, mu);
                }
            }
            GsTimeScope ts(ctx, "pull_input_grad", l, st);
            // reverse shuffle + ReLU of the layer below: dZ of layer l-1
            const void *hact = sb.hidden[l];
            const int64_t ubl = ctx->ub_front[l];
            // one wave per row of the level, and no more workgroups than stay resident at once: the waves
            // stride over the rows, and workgroups that had to queue behind the resident ones would run
            // their whole share after them on a nearly empty chip
            const bool bits = in_step && sb.bits[l];
            PullArgs pull{sb.gtmp, D, B.rev_ptr, B.rev_cnt, B.rev_list, B.rev_long, bits ? (const void *)sb.bits[l] : hact, ml, S, (void *)sb.ghid[l], 0};
#define GS_PULL_ROWS(...)                                                                                        \
    do {                                                                                                         \
        pull.n_main = (int)std::min<int64_t>(grid_1d(ctx, ubl * 64),                                             \
                                             (int64_t)ctx->n_cu * resident_blocks<__VA_ARGS__>());               \
        hipLaunchKernelGGL((__VA_ARGS__), dim3(pull.n_main + PULL_LONG_BLOCKS), dim3(256), 0, st,                \
                           pull.gin, pull.D, pull.rev_ptr, pull.rev_cnt, pull.rev_list, pull.rev_long, pull.hact,        \
                           pull.meta_lo, pull.S, pull.gout, pull.n_main);                                        \
    } while (0)
#define GS_PULL_GRAD(LPR, VEC)                                                                                   \
    do {                                                                                                         \
        const int n_grad = split_grad_blocks(grad, 64);                                                          \
        pull.n_main = (int)std::min<int64_t>(grid_1d(ctx, ubl * 64), (int64_t)ctx->n_cu * 4);                    \
        const dim3 grid(n_grad + pull.n_main + PULL_LONG_BLOCKS);                                                \
        if (vdz) hipLaunchKernelGGL((k_pull_and_grad_w<LPR, VEC, 4>), grid, dim3(256), 0, st, pull, grad, mu, n_grad); \
        else hipLaunchKernelGGL((k_pull_and_grad_w<LPR, VEC, 1>), grid, dim3(256), 0, st, pull, grad, mu, n_grad);     \
    } while (0)
#define GS_PULL_GRAD_W(VEC)                               \
    do {                                                  \
        if (D / VEC <= 16) GS_PULL_GRAD(16, VEC);         \
        else if (D / VEC <= 32) GS_PULL_GRAD(32, VEC);    \
        else GS_PULL_GRAD(64, VEC);                       \
    } while (0)
#define GS_PULL_W(VEC, HH, OH)                                                                                   \
    do {                                                                                                         \
        if (D / VEC <= 16) GS_PULL_ROWS(k_pull_input_grad<16, VEC, HH, OH>);                                     \
        else if (D / VEC <= 32) GS_PULL_ROWS(k_pull_input_grad<32, VEC, HH, OH>);                                \
        else GS_PULL_ROWS(k_pull_input_grad<64, VEC, HH, OH>);                                                   \
    } while (0)
            // (the level's dZ is held in bf16 under the same condition its consumers test (dz_h))
            if (with_pull) {
                if (D % 4 == 0) GS_PULL_GRAD_W(4);
                else if (D % 2 == 0) GS_PULL_GRAD_W(2);
                else GS_PULL_GRAD_W(1);
            } else if (bits) {
                if (D <= 128) GS_PULL_ROWS(k_pull_gated<32>);       // (at least RELU_BITS_MIN)
                else GS_PULL_ROWS(k_pull_gated<64>);
            } else if (h16 && D % 8 == 0) GS_PULL_W(4, true, true);
            else if (h16) GS_PULL_W(4, true, false);
            else if (D % 4 == 0) GS_PULL_W(4, false, false);
            else if (D % 2 == 0) GS_PULL_W(2, false, false);
            else GS_PULL_W(1, false, false);
#undef GS_PULL_GRAD_W
#undef GS_PULL_GRAD
#undef GS_PULL_W
#undef GS_PULL_ROWS
        }
    }
    {
        GradReduce gr;
        int64_t wmax = 1;
        for (int l = 0; l < L; ++l) {
            gr.part[l] = sb.gw_part[l]; gr.gws[l] = d_gw_self[l]; gr.gwn[l] = d_gw_neigh[l]; gr.gb[l] = d_gbias[l];
            gr.D[l] = p->dims[l]; gr.N[l] = p->dims[l + 1]; gr.nchunk[l] = sb.nchunk[l]; 
            gr.rows_min[l] = p->dtype == GSPLIT_F32 ? SGW_ROWS_MIN : GRAD_W_ROWS_MIN;
            gr.stream_rows[l] = sb.gw_stream[l] ? sb.stream_rows[l] : 0; gr.stream_nchunk[l] = sb.stream_nchunk[l];
            gr.stream_rows_min[l] = GWH_ROWS_MIN;
            gr.fixed_chunks[l] = l == L - 1 ? top_chunks : 0;
            wmax = std::max<int64_t>(wmax, (int64_t)(2 * p->dims[l] + 1) * p->dims[l + 1]);
        }
        GsTimeScope ts(ctx, "reduce_grads", -1, st);
        hipLaunchKernelGGL(k_reduce_grads, dim3(sum_slabs_grid(wmax), L), dim3(256),
                           0, st, gr, ctx->d_meta, S);
    }
    GS_HIP(ctx, hipGetLastError());
    return GSPLIT_OK;
}

int check_grad_outputs(gsplit_ctx *ctx, float *const *d_gw_self, float *const *d_gw_neigh, float *const *d_gbias,
                       const char *who) {
    if (!d_gw_self || !d_gw_neigh || !d_gbias) return gs_fail(ctx, GSPLIT_EINVAL, std::string(who) + ": NULL buffer");
    for (int l = 0; l < ctx->L; ++l)
        if (!d_gw_self[l] || !d_gw_neigh[l] || !d_gbias[l])
            return gs_fail(ctx, GSPLIT_EINVAL, std::string(who) + ": NULL gradient pointer");
    return GSPLIT_OK;
}

// does the top layer of this model and batch run as k_sage_top_fused?
bool top_fusable(const gsplit_ctx *ctx, const gsplit_sage_params *p, const void *top_input) {
    const int L = ctx->L;
    if (L < 2 || ctx->n_targets > TOP_MAX_ROWS) return false;
    const int D = p->dims[L - 1], N = p->dims[L];
    return N <= TOP_NMAX && D % (p->dtype == GSPLIT_BF16 ? 8 : 4) == 0 && D <= TOP_DMAX && aligned16(top_input);
}

}  // namespace

extern "C" int gsplit_sage_bwd(gsplit_ctx *ctx, const gsplit_sage_params *p, const float *d_grad_logits,
                               float *const *d_gw_self, float *const *d_gw_neigh, float *const *d_gbias,
                               void *stream) {
    if (!ctx) return GSPLIT_EINVAL;
    int rc = check_params(ctx, p, "gsplit_sage_bwd");
    if (rc) return rc;
    if (!d_grad_logits) return gs_fail(ctx, GSPLIT_EINVAL, "gsplit_sage_bwd: NULL buffer");
    rc = check_grad_outputs(ctx, d_gw_self, d_gw_neigh, d_gbias, "gsplit_sage_bwd");
    if (rc) return rc;
    GsSageBuf &sb = ctx->sage;
    if (!sb.ready || !sb.fwd_done || sb.fwd_batch != ctx->batch_id)
        return gs_fail(ctx, GSPLIT_ESTATE, "gsplit_sage_bwd: needs gsplit_sage_fwd on the current batch first");
    for (int l = 0; l <= ctx->L; ++l)
        if (sb.dims[l] != p->dims[l] || sb.dtype != p->dtype)
            return gs_fail(ctx, GSPLIT_ESTATE, "gsplit_sage_bwd: parameters differ from the forward pass");
    return sage_backward(ctx, p, d_grad_logits, d_gw_self, d_gw_neigh, d_gbias, (hipStream_t)stream, 0, false);
}

extern "C" int gsplit_sage_step(gsplit_ctx *ctx, const gsplit_sage_params *p, const void *d_feat_local,
                                const int64_t *d_labels, float *d_logits, float *d_row_loss, float *const *d_gw_self,
                                float *const *d_gw_neigh, float *const *d_gbias, void *stream) {
    if (!ctx) return GSPLIT_EINVAL;
    int rc = check_params(ctx, p, "gsplit_sage_step");
    if (rc) return rc;
    if (!d_feat_local || !d_labels || !d_logits) return gs_fail(ctx, GSPLIT_EINVAL, "gsplit_sage_step: NULL buffer");
    rc = check_grad_outputs(ctx, d_gw_self, d_gw_neigh, d_gbias, "gsplit_sage_step");
    if (rc) return rc;
    if (ctx->batch_id == 0) return gs_fail(ctx, GSPLIT_ESTATE, "gsplit_sage_step: no batch");
    rc = ensure_buffers(ctx, p);
    if (rc) return rc;
    hipStream_t st = (hipStream_t)stream;
    GsSageBuf &sb = ctx->sage;
    const int L = ctx->L, S = ctx->S;
    const int N = p->dims[L];
    ensure_relu_bits(ctx, p, st);
    if (!top_fusable(ctx, p, sb.hidden[L - 1])) {
        // the three steps one after the other, the loss gradient in the context's own buffer
        rc = sage_forward(ctx, p, d_feat_local, d_logits, st, L, true);
        if (rc) return rc;
        {
            GsTimeScope ts(ctx, "softmax_xent", -1, st);
            hipLaunchKernelGGL(k_softmax_xent, dim3(grid_1d(ctx, ctx->ub_front[L] * 64)), dim3(256), 0, st, d_logits, N,
                               d_labels, ctx->front[L], ctx->d_meta + L, S, sb.glog, d_row_loss);
        }
        rc = sage_backward(ctx, p, sb.glog, d_gw_self, d_gw_neigh, d_gbias, st, 0, true);
        sb.fwd_done = false;
        return rc;
    }
    rc = sage_forward(ctx, p, d_feat_local, d_logits, st, L - 1, true);
    if (rc) return rc;
    const int l = L - 1, D = p->dims[l];
    const GsLayerBuf &B = ctx->layer[l];
    const int chunks = top_slabs(ctx->n_targets);
    {
        const bool half = p->dtype == GSPLIT_BF16;
        TopArgs ta{sb.hidden[l], D, N, B.blk_indptr, B.edge_row, B.self_row, sb.wfrag_fwd[l], sb.wfrag_gin[l], sb.wstack32[l],
                   half ? (N + 7) & ~7 : (N + 3) & ~3, sb.wtrans[l], sb.wstack[l],
                   (const float *)p->d_bias[l], d_labels, ctx->front[L], d_logits, d_row_loss, sb.gtmp, sb.gw_part[l],
                   ctx->d_meta + L, S};
        GsTimeScope ts(ctx, "top_fused", l, st);
        const size_t lds = sizeof(float) * top_lds_words(D);
        if (half) hipLaunchKernelGGL(k_sage_top_fused<true>, dim3(chunks), dim3(TOP_T), lds, st, ta);
        else hipLaunchKernelGGL(k_sage_top_fused<false>, dim3(chunks), dim3(TOP_T), lds, st, ta);
    }
    rc = sage_backward(ctx, p, nullptr, d_gw_self, d_gw_neigh, d_gbias, st, chunks, true);
    sb.fwd_done = false;        // the step is complete: a separate backward call needs a forward call of its own
    return rc;
}

extern "C" int gsplit_softmax_xent(gsplit_ctx *ctx, const float *d_logits, int32_t n_classes,
                                   const int64_t *d_labels, float *d_grad_logits, float *d_row_loss,
                                   void *stream) {
    if (!ctx) return GSPLIT_EINVAL;
    if (!d_logits || !d_labels || !d_grad_logits || n_classes < 1)
        return gs_fail(ctx, GSPLIT_EINVAL, "gsplit_softmax_xent: bad argument");
    if (ctx->batch_id == 0) return gs_fail(ctx, GSPLIT_ESTATE, "gsplit_softmax_xent: no batch");
    hipStream_t st = (hipStream_t)stream;
    const int L = ctx->L;
    GsTimeScope ts(ctx, "softmax_xent", -1, st);
    hipLaunchKernelGGL(k_softmax_xent, dim3(grid_1d(ctx, ctx->ub_front[L] * 64)), dim3(256), 0, st, d_logits,
                       n_classes, d_labels, ctx->front[L], ctx->d_meta + L, ctx->S, d_grad_logits, d_row_loss);
    GS_HIP(ctx, hipGetLastError());
    return GSPLIT_OK;
}

