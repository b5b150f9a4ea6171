// Split-parallel sampling for all S logical splits at once (paper Algorithm 1, `sp_sample`, with
// the online splitting of section 4): neighbour sampling, mixed-frontier dedup/relabel, owner
// buckets, next local frontiers and the shuffle index.  Every kernel takes its problem size from
// device memory (GsLevelMeta), so one iteration is enqueued without any host synchronisation; which
// kernels are launched, and in which shapes, follows from the context's upper bounds and from the number of targets
// of the call.
//
// Per sampling layer (3 launches; the bottom one 4):
//   1 sample_layer       + insert (vertex, split) keys of destinations and slots into the table;
//                        + the shuffle index of the layer above (its composition with edges[l] for the
//                          forward/backward passes, and edges[l] relabelled to mixed-frontier rows)
//   2 partition: count     one multi-class pass over the slots: per split its mixed frontier, per
//   3 partition: scatter   owner its bucket (= received ids) and its new local-frontier members,
//                          and the edge numbers; + block CSR offsets, destination vertices at the
//                          head of both frontiers; + the reverse index of the layer above; + reset of a hashed table
//                          for the next layer
//   4 shuffle index of the bottom layer
// (One workgroup doing count and scatter of a small partition in a single launch was tried for the
// top layer: its chains of dependent accesses have nobody to overlap with, 85 us against 21 us
// for 5120 slots.  The targets themselves, one lookup each, do take a single workgroup when there
// are at most 1024 of them, and the top layers of a batch that has few of them go with them: k_sample_small.)
// The scatter side of the shuffle index (for every row of local_cat[l], the destination rows it
// feeds, so that the backward pass can pull) of layer l+1 rides on the two partition launches of
// layer l; only a context that keeps one for the bottom layer pays two launches of its own, after
// the layer loop.
//
// Why one partition pass serves both frontiers: the rows of a level are ordered by split, so the
// slot stream in (row, slot) order is the concatenation of the splits' slot streams, and the ids an
// owner t receives, `for s: bucket[s -> t]`, are the per-split first occurrences owned by t in
// exactly that global order.  The first occurrence of a vertex among the received ids of its owner
// is therefore its first occurrence in the whole slot stream (which is always a per-split first
// occurrence too): the smallest position among the vertex's keys in the table, which the sampler filled with
// global slot positions, tells it without a pass over the received ids.
// A dependent HBM access costs about a microsecond, and these kernels are chains of them, so every
// element remembers the table entry it landed in (no second probe sequence) and the count passes
// leave their classification behind for the scatter passes.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "gsplit_internal.h"

namespace {

constexpr int PART_BS = 256;     // threads of a partition workgroup
constexpr int PART_NK = 25;     // classes of a partition pass: 8 splits + 8 owners + 1 edge counter + 8 owners (new local)
constexpr int PART_MAX_NB = 1024;
constexpr unsigned long long EMPTY_ENTRY = ~0ull;
constexpr int CLAIM_FIRST_MAX = 1 << 18;     // destinations + slots up to which inserts claim before they read

// ------------------------------------------------------------------------------------------
// small device helpers
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

__device__ __forceinline__ uint64_t lanemask_lt() {
    return (1ull << lane_id()) - 1ull;
}

// The S + 1 split offsets of a level, loaded once per wave (all entries in flight together) into scalar
// registers.  Looking them up where they lie costs a wave S - 1 reads of the cache one after the other
// for every element, in kernels that are chains of a few dependent accesses.
struct SplitOffs {
    int o[GS_MAXS + 1];     // entries past S hold INT_MAX
    int n;                  // o[S]: rows of the level
    __device__ __forceinline__ static SplitOffs load(const int32_t *off, int S) {
        int32_t v[GS_MAXS + 1];
#pragma unroll
        for (int k = 0; k <= GS_MAXS; ++k) v[k] = off[k];
        SplitOffs r;
        r.n = 0;
#pragma unroll
        for (int k = 0; k <= GS_MAXS; ++k) {
            const int x = __builtin_amdgcn_readfirstlane(v[k]);
            r.o[k] = k <= S ? x : 0x7FFFFFFF;
            if (k == S) r.n = x;
        }
        return r;
    }
    // the split that row i belongs to
    __device__ __forceinline__ int of(int i) const {
        int s = 0;
#pragma unroll
        for (int k = 1; k < GS_MAXS; ++k) s += o[k] <= i ? 1 : 0;
        return s;
    }
    // the same, and the entry of `other` (offsets of the same splits) that belongs to it (as a sum of
    // differences: a choice between entries would put the array into memory)
    __device__ __forceinline__ int of(int i, const SplitOffs &other, int *entry) const {
        int s = 0, e = other.o[0];
#pragma unroll
        for (int k = 1; k < GS_MAXS; ++k)
            if (o[k] <= i) { s = k; e += other.o[k] - other.o[k - 1]; }
        *entry = e;
        return s;
    }
};

// Division by the fanout of a layer, for numerators below 2^31 (a layer has fewer than 2^29 slots): with
// s = ceil(log2 d) and m = ceil(2^(31 + s) / d), floor(n / d) = (n * m) >> (31 + s), because
// m * d - 2^(31 + s) < d <= 2^s.  A slot's row is wanted in every pass, and the hardware has no divide.
struct FanDiv {
    uint32_t m; int32_t sh, d;
    static FanDiv make(int d) {
        int s = 0;
        while ((1 << s) < d) ++s;
        return FanDiv{(uint32_t)(((1ull << (31 + s)) + (unsigned)d - 1) / (unsigned)d), s - 1, d};
    }
    __device__ __forceinline__ int div(int n) const {
        return d == 1 ? n : (int)(__umulhi((uint32_t)n, m) >> sh);
    }
};

__device__ __forceinline__ int table_bits(int n_inputs) {
    // capacity = 2^bits >= 2 * n_inputs, at least 1024 entries
    int want = n_inputs < 512 ? 1024 : 2 * n_inputs;
    return 32 - __clz(want - 1);
}

// Insert into a direct table: the key is its own entry index.  Keeps the smallest position that carried the key under this
// layer's stamp; *ahead is set to the smaller position the key was already there with, if it was (the position of an
// element that was itself behind nothing when it entered it).
__device__ __forceinline__ int table_insert_direct(const GsTable &t, uint32_t stamp, uint32_t key, uint32_t p, int32_t *ahead) {
    const unsigned long long mine = ((unsigned long long)stamp << 32) | p;
    const unsigned long long old = atomicMin(&t.pos[key], mine);
    if ((uint32_t)(old >> 32) == stamp && (uint32_t)old < p) *ahead = (int32_t)(uint32_t)old;
    return (int)key;
}

// The hashed table holds 64-bit entries (key << 32 | smallest position that carried it) of (vertex, split) keys,
// hashed by the vertex: the keys of a vertex start at the same line of 8 entries (64 bytes; a vertex has at most
// 8 keys) and lie there side by side, filled from the front, running over into the next line when
// one is full.  So the first occurrence of the vertex in the whole stream (the smallest position
// among its keys) is read off the line the slot's own entry is in, and there is no second table
// keyed by the vertex, with its own insert and its own access to the memory per slot.
// (Lines of 16 entries, the 128 bytes one access to the memory moves anyway, measured slower: what
// a lane asks of a line costs by the request, and half the line is half the requests.)
constexpr int LINE_ENTRIES = 8;
constexpr int LINE_LOG = 3;
__device__ __forceinline__ uint32_t table_line(uint32_t vertex, int bits) {
    return ((vertex * 0x9E3779B1u) >> (32 - (bits - LINE_LOG))) << LINE_LOG;
}

// Insert into that table: an empty entry is claimed with one compare-and-swap, a taken one of the same key lowered with a
// 64-bit atomic min, which is skipped when it cannot change anything (hub vertices would serialise on one address).
// Returns the entry index (-1 and the error flag if the table is full, which sizing excludes); *ahead as above.
// The line is read once, with plain loads: what such a read shows of a taken
// entry is true for good (an entry keeps its key, its position only falls), and an entry it shows
// empty is taken with a compare-and-swap, which answers with the truth.  The probe starts at the first
// entry that is the key's or empty, and goes on one entry after the other from there.
// claim_first: no read at all, a compare-and-swap on one entry after the other from the front of the line.  One access
// instead of two when the entry is free, which is what a small layer's path through this function consists of; only
// where few elements share a key, since every attempt on a taken entry is then an atomic on it.
__device__ __forceinline__ int table_insert_line(const GsTable &t, int bits, uint32_t vertex, uint32_t S, uint32_t split,
                                                 uint32_t p, int32_t *err, int32_t *ahead, bool claim_first) {
    const uint32_t key = vertex * S + split;
    const uint32_t mask = (1u << bits) - 1u;
    const unsigned long long mine = ((unsigned long long)key << 32) | p;
    uint32_t h = table_line(vertex, bits);
    for (uint32_t probe = 0; probe <= mask; probe += LINE_ENTRIES) {
        int j0 = 0;
        unsigned long long at0 = EMPTY_ENTRY;
        if (!claim_first) {
            const ulonglong2 *line = reinterpret_cast<const ulonglong2 *>(t.slot + h);
            ulonglong2 q[LINE_ENTRIES / 2];
#pragma unroll
            for (int i = 0; i < LINE_ENTRIES / 2; ++i) q[i] = line[i];
            j0 = LINE_ENTRIES;
#pragma unroll
            for (int j = LINE_ENTRIES - 1; j >= 0; --j) {
                const unsigned long long e = (j & 1) ? q[j >> 1].y : q[j >> 1].x;
                if (e == EMPTY_ENTRY || (uint32_t)(e >> 32) == key) { j0 = j; at0 = e; }
            }
        }
        for (int j = j0; j < LINE_ENTRIES; ++j) {
            unsigned long long cur = (claim_first || j == j0) ? at0
                                         : __hip_atomic_load(&t.slot[h + j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (cur == EMPTY_ENTRY) {
                cur = atomicCAS(&t.slot[h + j], EMPTY_ENTRY, mine);
                if (cur == EMPTY_ENTRY) return (int)(h + j);
            }
            if ((uint32_t)(cur >> 32) == key) {
                if (mine < cur) atomicMin(&t.slot[h + j], mine);
                else *ahead = (int32_t)(uint32_t)cur;
                return (int)(h + j);
            }
        }
        h = (h + LINE_ENTRIES) & mask;
    }
    *err = 1;
    return -1;
}

// smallest position among the keys of a vertex in that table (at most `start`): its lines are read
// until one shows an empty entry
__device__ __forceinline__ uint32_t table_line_first(const GsTable &t, int bits, uint32_t vertex, uint32_t S, uint32_t start) {
    const uint32_t mask = (1u << bits) - 1u;
    const uint32_t base = vertex * S;
    uint32_t h = table_line(vertex, bits), best = start;
    for (uint32_t probe = 0; probe <= mask; probe += LINE_ENTRIES) {
        const ulonglong2 *line = reinterpret_cast<const ulonglong2 *>(t.slot + h);
        ulonglong2 q[LINE_ENTRIES / 2];
#pragma unroll
        for (int i = 0; i < LINE_ENTRIES / 2; ++i) q[i] = line[i];
        bool open = false;
#pragma unroll
        for (int j = 0; j < LINE_ENTRIES; ++j) {
            const unsigned long long e = (j & 1) ? q[j >> 1].y : q[j >> 1].x;
            if (e == EMPTY_ENTRY) open = true;
            else if ((uint32_t)(e >> 32) - base < S) best = min(best, (uint32_t)e);
        }
        if (open) break;
        h = (h + LINE_ENTRIES) & mask;
    }
    return best;
}

// Stamp of the direct tables for sampling layer `layer` of the batch a context is working on: falls
// with every batch and, inside a batch, from the top layer down (8 = GSPLIT_MAX_LAYERS per batch).
__device__ __forceinline__ uint32_t table_stamp(const GsLevelMeta *meta_level0, uint32_t layer) {
    return 0xFFFFFFF0u - (meta_level0->batches * 8u + (7u - layer));
}

// ------------------------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11): counter-based generator, 10 rounds.
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint2 k) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint32_t hi0 = __umulhi(0xD2511F53u, c.x), lo0 = 0xD2511F53u * c.x;
        const uint32_t hi1 = __umulhi(0xCD9E8D57u, c.z), lo1 = 0xCD9E8D57u * c.z;
        c = make_uint4(hi1 ^ c.y ^ k.x, lo1, hi0 ^ c.w ^ k.y, lo0);
        k.x += 0x9E3779B9u;
        k.y += 0xBB67AE85u;
    }
    return c;
}

// Floyd's selection inside groups of G lanes: lane q holds t = t_q and j = d - fan + q and gets t_q, or j where t_q is
// already among the choices of the lanes before it.  One round after the other for lane s of every group: its t goes to the
// group by a lane permute (a row of 16 broadcasts its lane s) or by reads of the wave's registers, the lanes before it that
// chose it are a mask, and a field of the mask that is not zero carries into the bit of lane s.  (As an exchange through LDS and
// a shift of 64 bits a lane per round: 274k destinations x 20 261 us, now 252; 546k x 10 353 / 347; eight batches of 20k x 15
// 135.6 / 132.8; 20k x 15 25.1 / 23.9.  Reads of registers in groups of 16: 358 at 546k x 10.)
template <int G>
__device__ __forceinline__ uint32_t floyd_choice(uint32_t t, uint32_t j, int fan, bool floyd) {
    static_assert(G == 16 || G == 32 || G == 64, "lane groups");
    constexpr uint64_t each = G == 16 ? 0x0001000100010001ull : G == 32 ? 0x0000000100000001ull : 1ull;     // lane 0 of every group
    const uint64_t in = __ballot(floyd);
    uint32_t chosen = t;
    auto round = [&](uint32_t ts, int s) __attribute__((always_inline)) {
        const uint64_t hits = __ballot(chosen == ts) & in & (each * ((1ull << s) - 1ull));
        uint64_t repeat;        // lanes s of the groups that have a hit
        if (G == 64) repeat = hits != 0ull ? 1ull << s : 0ull;
        else repeat = ((hits + each * ((1ull << (G - 1)) - 1ull)) & (each << (G - 1))) >> (G - 1 - s);
        if (__builtin_amdgcn_inverse_ballot_w64(repeat)) chosen = j;
    };
    if constexpr (G == 16) {
#define GS_ROUND(S)                                                                                                        \
    if ((S) >= fan) return chosen;                                                                                         \
    round((uint32_t)__builtin_amdgcn_update_dpp(0, (int)t, 0x150 + (S), 0xF, 0xF, false), S);       /* row_newbcast:S */
        GS_ROUND(1) GS_ROUND(2) GS_ROUND(3) GS_ROUND(4) GS_ROUND(5) GS_ROUND(6) GS_ROUND(7) GS_ROUND(8)
        GS_ROUND(9) GS_ROUND(10) GS_ROUND(11) GS_ROUND(12) GS_ROUND(13) GS_ROUND(14) GS_ROUND(15)
#undef GS_ROUND
    } else {
        for (int s = 1; s < fan; ++s) {
            uint32_t ts = (uint32_t)__builtin_amdgcn_readlane((int)t, s);
            if (G == 32) {
                const uint32_t upper = (uint32_t)__builtin_amdgcn_readlane((int)t, 32 + s);
                ts = lane_id() < 32 ? ts : upper;
            }
            round(ts, s);
        }
    }
    return chosen;
}

// ------------------------------------------------------------------------------------------
// sample_layer: G lanes cooperate on one frontier vertex (G = 16, 32 or 64 >= fanout).
// degree <= fanout: copy the row in CSR order.  Otherwise Floyd's selection: lane q draws
// t_q in [0, d-fan+q] from its own Philox word; the sequential "already chosen -> take j"
// rule is resolved with fan-1 rounds of broadcast + ballot inside the lane group.
// The random word of draw q is word (q mod 4) of Philox(counter = (v, iter lo, iter hi,
// layer * 65536 + q / 4), key = (seed lo, seed hi)): a function of the global vertex id only.
// Every destination vertex (position i) and every sampled slot (position n1 + slot index) is
// also entered into the table under the key (vertex, split of the row); the entry's index is kept in
// ent_mixed (destinations first, then slots; -1 for padding slots).  A slot that found its key already
// there with a smaller position keeps that instead (-2 - position): it is not the first occurrence in its
// split, and where that is stands, after the count pass, in the entry index of the element it was behind.
// ------------------------------------------------------------------------------------------
// Arguments of one mini-batch of a launch.  Every sampling kernel serves up to GS_MAXB independent
// mini-batches (contexts over the same graph) at once, blockIdx.y = batch: the kernels of a small
// layer are chains of dependent accesses that leave the chip idle, and the chains of several batches
// overlap (sampling does not depend on the weights, so the batches of the next steps are known).
constexpr int GS_MAXB = GSPLIT_MAX_MULTI;

struct SampleArgs {
    const int32_t *front; GsLevelMeta *meta_lo; const GsLevelMeta *meta_up;
    GsTable tab;
    int32_t *ent_mixed, *nbr, *cnt; int64_t *epos;
    uint64_t iter; const uint64_t *seed_iter;
};
struct SampleArgsSet { SampleArgs b[GS_MAXB]; };

// shuffle index of every mixed-frontier row, the same lookup composed with edges[l] for the
// on-GPU forward/backward (rows of local_cat[l] per destination vertex and per edge), and edges[l]
// itself relabelled to rows of the owning split's mixed frontier
struct ShuffleArgs {
    const int32_t *row_mixed, *row_local;       // rows by position of a key's first occurrence
    const int32_t *ent_mixed, *mixed_ent, *blk_indptr;
    int32_t *blk_src, *src_row, *self_row, *edge_row, *rev_cnt;
    const GsLevelMeta *meta_lo, *meta_up;
    int32_t *pos_pair; const int32_t *mixed_pos;        // a wide layer's (null otherwise)
};
struct ShuffleArgsSet { ShuffleArgs b[GS_MAXB]; };

// where the key of slot g first occurs (-1: an empty slot), after the count pass: a slot that was behind another
// element asks that one, whose own first occurrence is either itself (a destination) or written there
__device__ __forceinline__ int first_occurrence(const int32_t *__restrict__ ent_mixed, int n1, int g) {
    const int e = ent_mixed[n1 + g];
    if (e >= -1) return e;
    const int at = -2 - e;
    return at < n1 ? at : ent_mixed[at];
}

__device__ __forceinline__ void shuffle_index(const ShuffleArgs &a, int S, const FanDiv &fan, int block, int n_blocks) {
    const int32_t *__restrict__ ent_mixed = a.ent_mixed;
    const int32_t *__restrict__ mixed_ent = a.mixed_ent;
    const int32_t *__restrict__ blk_indptr = a.blk_indptr;
    int32_t *__restrict__ blk_src = a.blk_src;
    int32_t *__restrict__ src_row = a.src_row;
    int32_t *__restrict__ self_row = a.self_row;
    int32_t *__restrict__ edge_row = a.edge_row;
    int32_t *__restrict__ rev_cnt = a.rev_cnt;
    const SplitOffs up = SplitOffs::load(a.meta_up->front_off, S), mixed_off = SplitOffs::load(a.meta_lo->mixed_off, S);
    const int n1 = up.n;
    const int64_t n_mixed = mixed_off.n;
    // A wide layer leaves the slots to shuffle_edges: here every mixed-frontier row also notes its row
    // of local_cat at the position where its key first occurs, beside the row the scatter pass left there.
    const int64_t n_slots = a.pos_pair ? 0 : (int64_t)n1 * fan.d;
    const int64_t total = n_mixed + n1 + n_slots;
    for (int64_t x = block * (int64_t)blockDim.x + threadIdx.x; x < total; x += (int64_t)n_blocks * blockDim.x) {
        if (x < n_mixed) {
            const int p = mixed_ent[x];
            const int r = p >= 0 ? a.row_local[p] : -1;
            src_row[x] = r;
            if (a.pos_pair) a.pos_pair[2 * (size_t)a.mixed_pos[x] + 1] = r;
        } else if (x < n_mixed + n1) {
            const int i = (int)(x - n_mixed);
            const int h = ent_mixed[i];
            const int r = h >= 0 ? a.row_local[i] : -1;
            self_row[i] = r;
            if (rev_cnt && r >= 0) atomicAdd(&rev_cnt[r], 1);
        } else {
            const int g = (int)(x - n_mixed) - n1;
            const int i = fan.div(g), q = g - i * fan.d;
            const int e = blk_indptr[i] + q;
            const int first = first_occurrence(ent_mixed, n1, g);
            if (first < 0) continue;
            const int mrow = a.row_mixed[first];
            int first_mixed;
            up.of(i, mixed_off, &first_mixed);
            const int pl = mixed_ent[first_mixed + mrow];
            const int r = pl >= 0 ? a.row_local[pl] : -1;
            blk_src[e] = mrow;                       // edges[l] as rows of the split's mixed frontier
            edge_row[e] = r;
            if (rev_cnt && r >= 0) atomicAdd(&rev_cnt[r], 1);
        }
    }
}

// The slots of a wide layer, after shuffle_index.  In one launch a slot is three dependent random
// accesses (the mixed-frontier row kept where its key first occurs -> that row's vertex entry -> its
// row of local_cat), and a wide layer runs at the rate at which the memory completes such accesses;
// once every mixed-frontier row has left its row of local_cat at that same position, a slot is one
// access of 8 bytes.
__device__ __forceinline__ void shuffle_edges(const ShuffleArgs &a, int S, const FanDiv &fan, int block, int n_blocks) {
    const int32_t *__restrict__ ent_mixed = a.ent_mixed;
    const int32_t *__restrict__ blk_indptr = a.blk_indptr;
    const int2 *__restrict__ pair = reinterpret_cast<const int2 *>(a.pos_pair);
    int32_t *__restrict__ blk_src = a.blk_src;
    int32_t *__restrict__ edge_row = a.edge_row;
    int32_t *__restrict__ rev_cnt = a.rev_cnt;
    const int n1 = a.meta_up->front_off[S];
    const int64_t n_slots = (int64_t)n1 * fan.d;
    for (int64_t g = block * (int64_t)blockDim.x + threadIdx.x; g < n_slots; g += (int64_t)n_blocks * blockDim.x) {
        const int first = first_occurrence(ent_mixed, n1, (int)g);
        if (first < 0) continue;
        const int i = fan.div((int)g), q = (int)g - i * fan.d;
        const int2 v = pair[first];
        const int e = blk_indptr[i] + q;
        blk_src[e] = v.x;
        edge_row[e] = v.y;
        if (rev_cnt && v.y >= 0) atomicAdd(&rev_cnt[v.y], 1);
    }
}

// The relabelling of the layer above (its shuffle index, or the edges of a wide one) reads nothing that the sampler
// writes, nor the other way round (ent_mixed alternates between two arrays from layer to layer): it rides on the
// sampler's launch, in workgroups behind the sampler's own.  A launch less per layer above the bottom one, 3 to 4 us each
// (the thirteen launches that sample 33 targets through three layers 66 -> 60 us).
enum { RIDE_NONE = 0, RIDE_INDEX = 1, RIDE_EDGES = 2 };
struct Ride { int what; FanDiv fan; int n_main; };

template <int G, typename IndPtrT>
__global__ __launch_bounds__(256) void k_sample_layer(const IndPtrT *__restrict__ indptr,
                                                      const int32_t *__restrict__ indices,
                                                      SampleArgsSet set, int S,
                                                      int fan, uint32_t layer, uint64_t seed,
                                                      ShuffleArgsSet above, Ride ride) {
    if ((int)blockIdx.x >= ride.n_main) {
        const int block = (int)blockIdx.x - ride.n_main, n_blocks = (int)gridDim.x - ride.n_main;
        if (ride.what == RIDE_INDEX) shuffle_index(above.b[blockIdx.y], S, ride.fan, block, n_blocks);
        else shuffle_edges(above.b[blockIdx.y], S, ride.fan, block, n_blocks);
        return;
    }
    const SampleArgs &a = set.b[blockIdx.y];
    const int32_t *__restrict__ front = a.front;
    GsLevelMeta *meta_lo = a.meta_lo;
    const GsLevelMeta *__restrict__ meta_up = a.meta_up;
    const GsTable tab = a.tab;
    const bool lines = !tab.pos;        // hashed: the keys of a vertex share lines (direct: they are neighbours in memory)
    int32_t *__restrict__ ent_mixed = a.ent_mixed;
    int32_t *__restrict__ nbr = a.nbr;
    int32_t *__restrict__ cnt = a.cnt;
    int64_t *__restrict__ epos = a.epos;
    uint64_t iter = a.iter;
    if (a.seed_iter) {      // seed and iteration counter kept in device memory (replayed graphs)
        seed = a.seed_iter[0];
        iter = a.seed_iter[1];
    }
    const SplitOffs up = SplitOffs::load(meta_up->front_off, S);
    const int n1 = up.n;
    const int bits = tab.pos ? (int)table_stamp(meta_lo - layer, layer) : table_bits(n1 * (1 + fan));
    const bool claim_first = n1 * (1 + fan) <= CLAIM_FIRST_MAX;
    const int groups_per_block = PART_BS / G;
    const int q = threadIdx.x % G;
    const int sub = lane_id() / G;
    const int stride = ride.n_main * groups_per_block;
    // every lane of a wave runs the same number of iterations (ballots/shuffles need that)
    const int first = blockIdx.x * groups_per_block + (threadIdx.x / 64) * (64 / G);
    for (int base = first; base < n1; base += stride) {
        const int row = base + sub;
        const bool active = row < n1;
        int32_t v = 0;
        int64_t beg = 0;
        uint32_t d = 0;
        if (active) {
            v = front[row];
            beg = (int64_t)indptr[v];
            d = (uint32_t)((int64_t)indptr[v + 1] - beg);
        }
        int32_t val = -1;
        const bool floyd = active && d > (uint32_t)fan;
        uint32_t chosen = 0, t = 0, j = 0;
        if (floyd && q < fan) {
            uint4 ctr = make_uint4((uint32_t)v, (uint32_t)iter, (uint32_t)(iter >> 32),
                                   (layer << 16) | ((uint32_t)q >> 2));
            uint4 r = philox4x32_10(ctr, make_uint2((uint32_t)seed, (uint32_t)(seed >> 32)));
            uint32_t w = (q & 3) == 0 ? r.x : (q & 3) == 1 ? r.y : (q & 3) == 2 ? r.z : r.w;
            j = d - (uint32_t)fan + (uint32_t)q;
            t = __umulhi(w, j + 1u);
        }
        // does any group of this wave need the sequential resolution?
        if (__ballot(floyd) != 0ull) chosen = floyd_choice<G>(t, j, fan, floyd);
        // What a lane enters into the table: its sampled neighbour (lanes q < fan) with the
        // slot's global position, or, in the first spare lane of the group, the destination vertex
        // itself with its row (destinations hold the smallest positions).  All of them go through
        // the same insert instructions, so the destination's inserts cost the wave no extra round
        // trips; only a group without a spare lane (fan == G) has lane 0 do them first.
        const bool spare = fan < G;
        int32_t key_v = -1;
        uint32_t pos_v = 0;
        int64_t out = -1;
        const uint32_t sp = active ? (uint32_t)up.of(row) : 0u;
        if (active && q < fan) {
            int64_t pos = -1;
            if (floyd) pos = beg + (int64_t)chosen;
            else if ((uint32_t)q < d) pos = beg + q;
            // (the graph is read once, at random: a load that leaves the caches to what is used again)
            if (pos >= 0) val = __builtin_nontemporal_load(&indices[pos]);
            const int64_t g = (int64_t)row * fan + q;
            nbr[g] = val;
            if (epos) epos[g] = pos;
            if (q == 0) {
                cnt[row] = d < (uint32_t)fan ? (int32_t)d : fan;
                if (!spare) {
                    int32_t none = -1;
                    ent_mixed[row] = lines ? table_insert_line(tab, bits, (uint32_t)v, (uint32_t)S, sp, (uint32_t)row,
                                                               &meta_lo->error, &none, false)
                                           : table_insert_direct(tab, (uint32_t)bits, (uint32_t)v * (uint32_t)S + sp, (uint32_t)row,
                                                                 &none);
                }
            }
            key_v = val;
            pos_v = (uint32_t)(n1 + g);
            out = n1 + g;
        } else if (active && spare && q == fan) {
            key_v = v;
            pos_v = (uint32_t)row;
            out = row;
        }
        if (out >= 0) {
            int hm = -1;
            int32_t ahead = -1;
            if (key_v >= 0)
                hm = lines ? table_insert_line(tab, bits, (uint32_t)key_v, (uint32_t)S, sp, pos_v, &meta_lo->error, &ahead, claim_first)
                           : table_insert_direct(tab, (uint32_t)bits, (uint32_t)key_v * (uint32_t)S + sp, pos_v, &ahead);
            ent_mixed[out] = (ahead >= 0 && out >= n1) ? -2 - ahead : hm;
        }
    }
}

// ------------------------------------------------------------------------------------------
// Stable multi-class partition in two launches over `nb` chunks: count per chunk, then scatter.
// Every scatter workgroup first turns the chunk histograms into its own bases (the sums over all
// chunks and over the chunks before it), so no launch sits between the two passes.
// What an element counts in is one byte, its code (PART_*), and the split its row belongs to:
//   PART_EDGE                    class 16
//   PART_WIN | owner << 3        classes `split` and 8 + owner
//   PART_FIRST (with PART_WIN)   class 17 + owner too
// A functor F describes the elements:
//   load()                       what every thread needs of the level's bookkeeping (F::Level), read once
//   n(lv)                        number of elements
//   classify(lv, g, &split)      count pass: the code of element g (and the split of a PART_WIN element);
//                                may leave the code behind for the scatter pass
//   cached(lv, g)                scatter pass: the code, the split and what else the element's emit() reads
//   heads(lv, s)                 rows that split s (owner s) puts before its class-s (class-17+s) elements
//   publish(lv, o)               writes those offsets to the batch's device bookkeeping (one
//                                workgroup of the launch; later launches read them there, this launch
//                                takes them from `o`)
//   emit(lv, g, e, segment, base, o)  base[k] + the segment's rank = bases[k] + number of class-k elements
//                                before g; called by whole waves
//   n_extra(lv, o), extra(lv, g, o)  independent element-wise work appended to the scatter pass
//   n_side(lv), side(lv, g, n)   independent work appended to the count pass: called by whole
//                                workgroups, 256 consecutive g at a time (g >= n in the last one)
// Elements keep their order inside every class (wave ballots + running chunk counters).
// Counting and ranking a segment of 64 elements takes six ballots (edge, winner, first, three bits of the
// owner) whatever the number of classes: lane k puts the count of class k together from them, an element
// its ranks.  (A shuffle tree per class took half of the count pass of a small layer, and a ballot per
// class, unrolled, made a scatter kernel of 41 KB, whose instructions arrive from memory for the first
// time in every launch.)
// ------------------------------------------------------------------------------------------
constexpr unsigned PART_EDGE = 1u, PART_WIN = 2u, PART_FIRST = 4u;
constexpr int PART_OWNER_SHIFT = 3;

struct Segment {                    // 64 elements, one per lane; all members but the lane's own code are uniform
    uint64_t edge, win, first, own0, own1, own2;
    unsigned code; int split;       // of the lane's element
    bool one_split;                 // all winners of the segment belong to split `split0`
    int split0;
    __device__ __forceinline__ static Segment make(unsigned code, int split) {
        Segment s;
        s.code = code; s.split = split;
        s.edge = __ballot(code & PART_EDGE);
        s.win = __ballot(code & PART_WIN);
        s.first = __ballot(code & PART_FIRST);
        s.own0 = __ballot(code & (1u << PART_OWNER_SHIFT));
        s.own1 = __ballot(code & (2u << PART_OWNER_SHIFT));
        s.own2 = __ballot(code & (4u << PART_OWNER_SHIFT));
        s.split0 = __builtin_amdgcn_readlane(split, s.win ? __builtin_ctzll(s.win) : 0);
        s.one_split = (__ballot(split != s.split0) & s.win) == 0ull;     // (rows are ordered by split: nearly always)
        return s;
    }
    // elements whose owner is t
    __device__ __forceinline__ uint64_t owned_by(int t) const {
        return ((t & 1) ? own0 : ~own0) & ((t & 2) ? own1 : ~own1) & ((t & 4) ? own2 : ~own2);
    }
    // winners of the segment in split s, the lane's own choice of s
    __device__ __forceinline__ uint64_t won_in(int s) const {
        if (one_split) return s == split0 ? win : 0ull;
        uint64_t m = 0ull;
#pragma unroll 1
        for (int k = 0; k < GS_MAXS; ++k) {
            const uint64_t b = __ballot(split == k) & win;
            if (s == k) m = b;
        }
        return m;
    }
    // number of elements in class k = the lane's index (anything for lanes >= PART_NK)
    __device__ __forceinline__ int count() const {
        const int k = lane_id();
        const uint64_t in_split = won_in(k);
        uint64_t m = k < 8 ? in_split : k < 16 ? win : k == 16 ? edge : first;
        if (k >= 8 && k != 16) m &= owned_by(k < 16 ? k - 8 : k - 17);
        return __popcll(m);
    }
};

// where the classes of each group start, as offsets of the splits / owners; entry S is the group's total
struct PartOffs {
    int a[GS_MAXS + 1];     // classes 0..7 with their heads: mixed_off
    int b[GS_MAXS + 1];     // classes 8..15: recv_off (front_off of the targets)
    int c[GS_MAXS + 1];     // classes 17..24 with their heads: front_off of the level below
    int total;              // class-16 total (edges)
};

// The classes as the first lanes of a wave hold them: three groups of eight lanes for the classes that have
// offsets, and the edge counter.
__device__ __forceinline__ int lane_class(int lane) { return lane < 16 ? lane : lane < 24 ? lane + 1 : 16; }
constexpr int PART_LANES = 25;

// First rank of the class of each of those lanes from its total (three steps of a scan inside the groups: row
// shifts, plain vector instructions).  Totals of splits the context does not have are zero, so entry S of an
// offset array is the total whatever S.
template <class F>
__device__ __forceinline__ int part_bases(const F &f, const typename F::Level &lv, int tot, PartOffs &o) {
    const int lane = lane_id(), grp = lane >> 3, s = lane & 7;
    const int head = grp == 0 || grp == 2 ? f.heads(lv, s) : 0;
    const int v = tot + head;
    int inc = v, below;
    below = __builtin_amdgcn_update_dpp(0, inc, 0x111, 0xF, 0xF, false);     // row_shr:1
    if (s >= 1) inc += below;
    below = __builtin_amdgcn_update_dpp(0, inc, 0x112, 0xF, 0xF, false);     // row_shr:2
    if (s >= 2) inc += below;
    below = __builtin_amdgcn_update_dpp(0, inc, 0x114, 0xF, 0xF, false);     // row_shr:4
    if (s >= 4) inc += below;
    if (grp < 3) {
        int *off = grp == 0 ? o.a : grp == 1 ? o.b : o.c;
        off[s] = inc - v;
        if (s == 7) off[GS_MAXS] = inc;
        return inc - v + head;
    }
    if (lane == 24) o.total = tot;
    return 0;
}

__device__ __forceinline__ int part_chunk(int n, int nb) {
    int c = (n + nb - 1) / nb;
    return ((c + PART_BS - 1) / PART_BS) * PART_BS;
}

// one functor and one histogram per mini-batch of the launch (blockIdx.y = batch)
template <class F>
struct PartSet { F f[GS_MAXB]; int32_t *hist[GS_MAXB]; };

// hist[chunk * PART_NK + class]; chunks past the last element have no entry
template <class F>
__global__ __launch_bounds__(PART_BS) void k_part_count(PartSet<F> set) {
    const F &f = set.f[blockIdx.y];
    int32_t *__restrict__ hist = set.hist[blockIdx.y];
    __shared__ int s_cnt[PART_BS / 64][PART_NK];
    const typename F::Level lv = f.load();
    const int n = f.n(lv);
    const int chunk = part_chunk(n, gridDim.x);
    const int64_t beg64 = (int64_t)blockIdx.x * chunk;
    const int wave = threadIdx.x >> 6;
    if (beg64 < n) {
        const int beg = (int)beg64;
        const int end = (n - beg < chunk) ? n : beg + chunk;
        int cnt = 0;                                    // lane k: class k
        for (int tile = beg; tile < end; tile += PART_BS) {
            const int g = tile + threadIdx.x;
            int split = 0;
            const unsigned code = g < end ? f.classify(lv, g, &split) : 0u;
            cnt += Segment::make(code, split).count();
        }
        if (lane_id() < PART_NK) s_cnt[wave][lane_id()] = cnt;
        __syncthreads();
        if (threadIdx.x < PART_NK) {
            int t = 0;
#pragma unroll
            for (int w = 0; w < PART_BS / 64; ++w) t += s_cnt[w][threadIdx.x];
            hist[blockIdx.x * PART_NK + threadIdx.x] = t;
        }
    }
    // every thread of the workgroup makes every call (side may synchronise the workgroup).  The
    // side work is dealt from the last workgroup backwards: in a small layer the first workgroups
    // hold all the elements and the rest are idle, so the two run side by side.
    const int64_t ns = f.n_side(lv);
    for (int64_t base = (int64_t)(gridDim.x - 1 - blockIdx.x) * PART_BS; base < ns; base += (int64_t)gridDim.x * PART_BS)
        f.side(lv, base + threadIdx.x, ns);
}

// A tile is up to PART_SUB * 256 elements, PART_SUB of them per thread (loads of all of them in flight, two
// barriers per tile).
constexpr int PART_SUB = 4;

// The kernel of a small layer is a chain: bookkeeping, histograms and codes, bases, ranks, stores.  (33 targets x 5,
// measured with clocks in the kernel: 0.8, 2.4, 0.5, 2.8 us of 6.6.  The histograms were summed class by class across
// the lanes of a wave, fourteen sums of four row rotations and four scalar reads one after the other, the first
// tile's counts waited for the bases, and a sender's bucket starts were a loop over the receivers.  Now 0.8, 1.5, 0.9, 1.2:
// 165 slots 6.5 -> 5.3 us, 30k slots 8.0 -> 6.5, 325k slots 14.0 -> 13.4.)
template <class F>
__global__ __launch_bounds__(PART_BS) void k_part_scatter(PartSet<F> set) {
    const F &f = set.f[blockIdx.y];
    const int32_t *__restrict__ hist = set.hist[blockIdx.y];
    constexpr int WAVES = PART_BS / 64, SEGS = PART_SUB * WAVES, HALVES = PART_BS / 32;
    __shared__ int s_tot[HALVES][32], s_pre[HALVES][32];
    __shared__ int s_seg[2][SEGS][PART_NK];
    __shared__ PartOffs s_o;
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const typename F::Level lv = f.load();
    const int n = f.n(lv);
    const int chunk = part_chunk(n, gridDim.x);
    const int64_t beg64 = (int64_t)blockIdx.x * chunk;
    const int beg = beg64 < n ? (int)beg64 : n;
    const int end = (n - beg < chunk) ? n : beg + chunk;
    typename F::Elem el[PART_SUB];
    // (a thread past the end reads the last element again: no branch around the loads, all of them in flight)
    auto fetch = [&](int tile) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < PART_SUB; ++j) {
            const int g = tile + j * PART_BS + (int)threadIdx.x;
            el[j] = f.cached(lv, min(g, end - 1));
            if (g >= end) el[j].code = 0u;
        }
    };
    // (uniform) 256-element parts of a tile that hold anything
    auto parts_of = [&](int tile) { return max(0, min(PART_SUB, (end - tile + PART_BS - 1) / PART_BS)); };
    // ranks where the segments' elements start (lane x of the first wave: class lane_class(x)); returns the next tile's
    auto start_ranks = [&](int parts, int buf, int run) __attribute__((always_inline)) {
        const int k = lane_class(lane);
        for (int i = 0; i < parts * WAVES; i += WAVES) {
            int c[WAVES];
#pragma unroll
            for (int w = 0; w < WAVES; ++w) c[w] = s_seg[buf][i + w][k];
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                s_seg[buf][i + w][k] = run;
                run += c[w];
            }
        }
        return run;
    };
    // the codes of the first elements do not depend on the histograms: they travel while those are read
    if (beg < end) fetch(beg);
    {
        const int k = min((int)threadIdx.x & 31, PART_NK - 1), half = threadIdx.x >> 5;
        const int live = chunk > 0 ? (n + chunk - 1) / chunk : 0;   // chunks that hold anything
        int tot = 0, pre = 0;
        // (half a wave takes a chunk's histogram, its lanes a class each; chunks past the last one are read again and not added)
        auto add = [&](auto many, int x) {
            constexpr int M = decltype(many)::value;
            int v[M];
#pragma unroll
            for (int u = 0; u < M; ++u) v[u] = hist[min(x + u * HALVES, live - 1) * PART_NK + k];
#pragma unroll
            for (int u = 0; u < M; ++u) {
                const int c = x + u * HALVES;
                tot += c < live ? v[u] : 0;
                pre += c < min(live, (int)blockIdx.x) ? v[u] : 0;
            }
        };
        int x = half;
        for (; x + 4 * HALVES < live; x += 16 * HALVES) add(std::integral_constant<int, 16>{}, x);
        for (; x < live; x += 4 * HALVES) add(std::integral_constant<int, 4>{}, x);
        s_tot[half][threadIdx.x & 31] = tot;
        s_pre[half][threadIdx.x & 31] = pre;
    }
    int run = 0, buf = 0;
    for (int tile = beg;; buf ^= 1) {       // (a workgroup without elements goes through it once, for the offsets)
        const int parts = parts_of(tile);
        // what every segment of the tile counts in every class
#pragma unroll 1
        for (int j = 0; j < parts; ++j) {       // (one copy of the code, here and below: see above)
            unsigned code = el[0].code;
            int split = el[0].split;
#pragma unroll
            for (int i = 1; i < PART_SUB; ++i)
                if (i == j) { code = el[i].code; split = el[i].split; }
            const int c = Segment::make(code, split).count();
            if (lane < PART_NK) s_seg[buf][j * WAVES + wave][lane] = c;
        }
        __syncthreads();
        if (wave == 0 && lane < PART_LANES) {
            if (tile == beg) {
                const int k = lane_class(lane);
                int tot = 0, pre = 0;
#pragma unroll
                for (int h = 0; h < HALVES; ++h) { tot += s_tot[h][k]; pre += s_pre[h][k]; }
                run = part_bases(f, lv, tot, s_o) + pre;
            }
            run = start_ranks(parts, buf, run);
        }
        __syncthreads();
        if (tile == beg && blockIdx.x == 0) f.publish(lv, s_o);
        // (the elements move up a register each time round)
#pragma unroll 1
        for (int j = 0; j < parts; ++j) {
            const int g = tile + j * PART_BS + (int)threadIdx.x;
            f.emit(lv, g, g < end, el[0], Segment::make(el[0].code, el[0].split), s_seg[buf][j * WAVES + wave], s_o);
#pragma unroll
            for (int i = 0; i + 1 < PART_SUB; ++i) el[i] = el[i + 1];
        }
        tile += PART_SUB * PART_BS;
        if (tile >= end) break;
        fetch(tile);
    }
    const PartOffs &o = s_o;
    // (dealt from the last workgroup backwards, like the count pass's side work)
    const int mine = (int)gridDim.x - 1 - (int)blockIdx.x;
    const int64_t nx = f.n_extra(lv, o);
    for (int64_t g = (int64_t)mine * PART_BS + threadIdx.x; g < nx; g += (int64_t)gridDim.x * PART_BS) f.extra(lv, g, o);
    f.clear(o, (int64_t)mine * PART_BS + threadIdx.x, (int64_t)gridDim.x * PART_BS);
}

// ---- local_front[L] = targets separated by owner, order kept ---------------------------------
struct PartTargets {
    const int32_t *targets; int n_targets; const uint8_t *pmap; int S; uint32_t n_vertices;
    int32_t *front; int32_t *perm; GsLevelMeta *meta;
    GsLevelMeta *meta_all; int n_levels;
    struct Level {};
    struct Elem { unsigned code; int split; };
    __device__ Level load() const { return Level{}; }
    __device__ int n(const Level &) const { return n_targets; }
    // An id outside the graph is in no class and so not in the batch (some vertex in its place would be there more than
    // once, and every bound on the rows of a level, which sizes buffers and tables, counts a vertex once).  It is
    // reported through the error flag, by the scatter pass only: the count pass is where the flags of the previous
    // batch are cleared.
    __device__ unsigned classify(const Level &, int g, int *) const {
        const uint32_t id = (uint32_t)targets[g];
        const unsigned owner = pmap[id < n_vertices ? id : 0u] & (GS_MAXS - 1);
        return id < n_vertices ? PART_WIN | owner << PART_OWNER_SHIFT : 0u;
    }
    __device__ Elem cached(const Level &lv, int g) const { return Elem{classify(lv, g, nullptr), 0}; }
    __device__ int heads(const Level &, int) const { return 0; }
    __device__ void publish(const Level &, const PartOffs &o) const {
        if ((int)threadIdx.x <= S) meta->front_off[threadIdx.x] = o.b[threadIdx.x];
    }
    __device__ void emit(const Level &, int g, bool in, const Elem &e, const Segment &sg, const int *base, const PartOffs &) const {
        if (!in) return;
        if (!(e.code & PART_WIN)) { meta->error = 3; return; }
        const int t = (int)(e.code >> PART_OWNER_SHIFT);
        const int r = base[8 + t] + __popcll(sg.win & sg.owned_by(t) & lanemask_lt());
        front[r] = targets[g];
        perm[r] = g;
    }
    // (the tables are clean when a batch starts: the last kernel of the previous batch cleared the
    // part a top layer of max_targets targets can use, gsplit_create all of them)
    __device__ int64_t n_extra(const Level &, const PartOffs &) const { return 0; }
    __device__ void extra(const Level &, int64_t, const PartOffs &) const {}
    __device__ void clear(const PartOffs &, int64_t, int64_t) const {}
    // the count pass is the first kernel of a batch: it clears the error flags of every level
    __device__ int64_t n_side(const Level &) const { return n_levels; }
    __device__ void side(const Level &, int64_t x, int64_t ns) const {
        if (x < ns) meta_all[x].error = 0;
        if (x == 0) meta_all[0].batches += 1;
    }
};

// A batch of at most 1024 targets takes the whole step in one workgroup, one target per thread:
// the two launches of the general partition are chains of a few dependent accesses each, and a
// launch by itself costs about as much as this kernel's work.
constexpr int TARGETS_SMALL = 1024;

struct TargetsSet { PartTargets f[GS_MAXB]; };

__global__ __launch_bounds__(TARGETS_SMALL) void k_targets_small(TargetsSet set) {
    const PartTargets &f = set.f[blockIdx.x];
    __shared__ int s_cnt[TARGETS_SMALL / 64][GS_MAXS];
    __shared__ int s_base[PART_LANES];
    __shared__ PartOffs s_o;
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    if (tid < f.n_levels) f.meta_all[tid].error = 0;
    if (tid == 0) f.meta_all[0].batches += 1;
    __syncthreads();                                   // the flags are cleared before one may be set
    int32_t id = 0;
    int k = -1;                                        // (stays so for an id outside the graph, see PartTargets)
    if (tid < f.n_targets) {
        id = f.targets[tid];
        if ((uint32_t)id < f.n_vertices) k = f.pmap[id] & (GS_MAXS - 1);
        else f.meta->error = 3;
    }
    int rank = 0;
#pragma unroll
    for (int c = 0; c < GS_MAXS; ++c) {
        const uint64_t bal = __ballot(k == c);
        if (k == c) rank = __popcll(bal & lanemask_lt());
        if (lane == 0) s_cnt[wave][c] = __popcll(bal);
    }
    __syncthreads();
    const PartTargets::Level lv{};
    if (tid < PART_LANES) {
        int acc = 0;
        if (tid >= 8 && tid < 16) {
            int c[TARGETS_SMALL / 64];
#pragma unroll
            for (int w = 0; w < TARGETS_SMALL / 64; ++w) c[w] = s_cnt[w][tid - 8];
#pragma unroll
            for (int w = 0; w < TARGETS_SMALL / 64; ++w) { s_cnt[w][tid - 8] = acc; acc += c[w]; }
        }
        s_base[tid] = part_bases(f, lv, acc, s_o);
    }
    __syncthreads();
    f.publish(lv, s_o);
    if (k >= 0) {
        const int r = s_base[8 + k] + s_cnt[wave][k] + rank;
        f.front[r] = id;
        f.perm[r] = tid;
    }
}

// ------------------------------------------------------------------------------------------
// The targets and the layers of a small batch that hang on nothing but them, in one launch: one workgroup a batch.  A layer
// of a few hundred slots is three launches of 4 to 6 us, each a chain of dependent accesses with nobody in its way, and
// the rows they hand to one another fit a workgroup's LDS, tables and all; so the chain runs on without the launch edges,
// the level's bookkeeping, the histograms and the entries that go through memory in between.  What is written is what the
// launches of the general path write, down to the order of every row (the order of a reverse-index row is free there too).
// What bounds it is the chain: the waves wait (memory, LDS, about ten barriers a layer) for 72 % of the time with 33 targets x 5 and
// 198 rows x 10, 26 us, and for 64 % with 204 targets x 10, 20 us; a SIMD's vector unit is busy for 33 and 45 %.  It grows with
// the slots all the same, one compute unit's work against a chip's, so larger layers stay with the launches that spread them.
// ------------------------------------------------------------------------------------------
constexpr int SMALL_T = 1024;
// Destinations and slots of a layer that one workgroup takes: what its LDS holds, which is right by the clock too for grouped calls
// and with hashed tables.  Sampling of a group, general launches / so, in us (1 M vertices): two, four and eight batches of 1000
// targets x 2, x 10 49.9 / 46.3, 66.5 / 53.2, 100 / 66; of 33 x 5, x 10, x 15 two 63.9 / 42, eight 117 / 60.5; eight of 409
// 214 / 177.  A batch by itself, hashed, x 5 below: 300 x 1 48.2 / 38.0, 409 x 5 50.5 / 46.2, 1000 x 2 50.8 / 50.6,
// 102 x 20 48.7 / 43.0.  Direct tables spare the general launches the clearing and most probes, and what one workgroup does grows with
// both (a destination costs about two slots), so a batch by itself with those is taken up to SMALL_ALONE.  By twice the
// destinations plus the slots, four splits, x 5 below / x 10, x 10 below / x 10, x 15 below (one split is 2 % kinder to one
// workgroup, which then looks for a vertex under one key):
//   2100: 300 x 5 38.8 / 35.8, 61.6 / 59.1, 63.9 / 62.2      2400: 600 x 2 38.4 / 37.2, 63.8 / 63.8, 68.1 / 68.8
//   2450: 350 x 5 38.4 / 37.2, 63.3 / 62.5, 66.2 / 66.2      2448: 204 x 10 38.5 / 37.5, 62.8 / 61.9, 65.1 / 65.2
//   2560: 640 x 2 38.6 / 37.7, 63.8 / 64.6, 69.4 / 70.7      2700: 450 x 4 38.9 / 37.9, 65.5 / 66.1, 73.4 / 72.2
//   2800: 700 x 2 38.8 / 38.8, 66.2 / 68.5, 71.2 / 74.0      2863: 409 x 5 38.2 / 38.8, 65.3 / 66.5, 72.1 / 73.6
//   3072: 768 x 2 38.5 / 39.4, 67.3 / 70.0, 71.4 / 74.5      4096: 1024 x 2 39.0 / 43.8, 72.8 / 82.3
constexpr int SMALL_ROWS = SMALL_T, SMALL_SLOTS = 2 * SMALL_T;
constexpr int SMALL_ALONE = 2720;                   // twice the destinations plus the slots
constexpr int SMALL_PER = SMALL_SLOTS / SMALL_T;    // slots a thread holds
constexpr int SMALL_MAX = SMALL_ROWS + SMALL_SLOTS; // elements, and rows of the level below
constexpr int SMALL_TAB_LOG = 13, SMALL_TAB = 1 << SMALL_TAB_LOG;      // entries of the table in LDS
constexpr int SMALL_LAYERS = 2 * GS_MAXB;           // layers of a launch, over all its batches

struct SmallLayer {         // of a batch; its own order of layers, top one first
    GsLevelMeta *meta_lo;
    int32_t *nbr, *cnt; int64_t *epos;
    int32_t *mixed, *blk_indptr, *blk_src, *recv, *src_row, *self_row, *edge_row, *front_lo;
    int32_t *rev_cnt, *rev_ptr, *rev_list, *rev_eid, *rev_long;     // (null: the layer has no reverse index)
};
struct SmallBatch {
    const int32_t *targets; int32_t *front, *perm; GsLevelMeta *meta;
    unsigned long long *slot;       // the hashed table, for the workgroups behind the first (null: direct)
    uint64_t iter; int n_targets;
};
struct SmallSet {
    SmallBatch b[GS_MAXB]; SmallLayer layer[SMALL_LAYERS]; FanDiv fan[GS_MAXL];
    const uint64_t *seed_iter;
    int n_layers, L;
    int64_t clear_pairs;            // pairs of table entries that the first layer of the general path can use
};
static_assert(sizeof(SmallSet) <= 3900, "argument block of a multi-batch launch too large");

struct NoHeads {
    struct Level {};
    __device__ int heads(const Level &, int) const { return 0; }
};
struct RowHeads {           // the destinations of a split in front of its rows
    struct Level { SplitOffs up; int S; };
    __device__ int heads(const Level &lv, int s) const {
        int first = 0, next = 0;
#pragma unroll
        for (int k = 0; k < GS_MAXS; ++k)
            if (k == s) { first = lv.up.o[k]; next = lv.up.o[k + 1]; }
        return s < lv.S ? next - first : 0;
    }
};

// The table in LDS: entries key << 32 | smallest position of (vertex, split) keys, hashed by the vertex and probed one after
// the other, so that a vertex's keys follow where it hashes to.  At most SMALL_MAX of its SMALL_TAB entries are taken.
__device__ __forceinline__ uint32_t small_hash(uint32_t vertex) { return (vertex * 0x9E3779B1u) >> (32 - SMALL_TAB_LOG); }
__device__ __forceinline__ int small_insert(unsigned long long *tab, uint32_t vertex, uint32_t S, uint32_t split, uint32_t pos) {
    const uint32_t key = vertex * S + split;
    const unsigned long long mine = ((unsigned long long)key << 32) | pos;
    for (uint32_t h = small_hash(vertex);; h = (h + 1) & (SMALL_TAB - 1)) {
        const unsigned long long old = atomicCAS(&tab[h], EMPTY_ENTRY, mine);
        if (old == EMPTY_ENTRY) return (int)h;
        if ((uint32_t)(old >> 32) == key) {
            if (mine < old) atomicMin(&tab[h], mine);
            return (int)h;
        }
    }
}
// smallest position among the keys of a vertex
__device__ __forceinline__ uint32_t small_first(const unsigned long long *tab, uint32_t vertex, uint32_t S) {
    uint32_t best = 0xFFFFFFFFu;
    for (uint32_t h = small_hash(vertex);; h = (h + 1) & (SMALL_TAB - 1)) {
        const unsigned long long e = tab[h];
        if (e == EMPTY_ENTRY) return best;
        if ((uint32_t)(e >> 32) - vertex * S < S) best = min(best, (uint32_t)e);
    }
}

template <typename IndPtrT>
__global__ __launch_bounds__(SMALL_T) void k_sample_small(const IndPtrT *__restrict__ indptr, const int32_t *__restrict__ indices,
                                                          const uint8_t *__restrict__ pmap, uint32_t n_vertices, int S,
                                                          SmallSet set, uint64_t seed) {
    const SmallBatch &a = set.b[blockIdx.y];
    const int tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (blockIdx.x > 0) {       // the hashed table, as far as the layer behind this launch can use it
        ulonglong2 *slot = reinterpret_cast<ulonglong2 *>(a.slot);
        for (int64_t x = (int64_t)(blockIdx.x - 1) * SMALL_T + tid; x < set.clear_pairs; x += (int64_t)(gridDim.x - 1) * SMALL_T)
            slot[x] = make_ulonglong2(EMPTY_ENTRY, EMPTY_ENTRY);
        return;
    }
    constexpr int WAVES = SMALL_T / 64, SEGS = SMALL_SLOTS / 64;
    __shared__ __align__(16) unsigned long long s_tab[SMALL_TAB];
    __shared__ int64_t s_beg[SMALL_ROWS];
    __shared__ int s_deg[SMALL_ROWS], s_front[SMALL_ROWS], s_pick[SMALL_SLOTS];
    __shared__ int s_seg[SEGS][PART_NK];
    __shared__ int s_base[PART_NK], s_wave[WAVES], s_long, s_bad;
    __shared__ PartOffs s_o;
    // (the table is done with when the rows are handed out)
    int *s_mixed = reinterpret_cast<int *>(s_tab), *s_local = s_mixed + SMALL_MAX, *s_rev = s_local + SMALL_MAX;
    static_assert(3 * SMALL_MAX * sizeof(int) <= sizeof(s_tab), "rows by position and counters in the place of the table");
    uint64_t iter = a.iter;
    if (set.seed_iter) { seed = set.seed_iter[0]; iter = set.seed_iter[1]; }

    // ranks where the elements of every segment start in every class, and the offsets of the classes
    auto start_ranks = [&](const auto &f, const auto &lv, int segs) __attribute__((always_inline)) {
        __syncthreads();
        if (wave == 0 && lane < PART_LANES) {
            const int k = lane_class(lane);
            int run = 0;
            for (int i = 0; i < segs; i += 8) {
                int c[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) c[u] = i + u < segs ? s_seg[i + u][k] : 0;
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    if (i + u < segs) s_seg[i + u][k] = run;
                    run += c[u];
                }
            }
            s_base[k] = part_bases(f, lv, run, s_o);
        }
        __syncthreads();
    };

    // targets separated by owner, order kept; their rows of the graph are asked for with the owner
    const int n_targets = a.n_targets;
    if (tid == 0) s_bad = 0;
    {
        bool bad = false;
        const bool in = tid < n_targets;
        uint32_t id = 0;
        unsigned code = 0;
        int64_t beg = 0, end = 0;
        Segment sg{};
        if (wave * 64 < n_targets) {
            id = in ? (uint32_t)a.targets[tid] : 0u;
            bad = in && id >= n_vertices;               // (left out and reported, see PartTargets)
            if (bad) id = 0u;
            const unsigned owner = pmap[id];
            beg = (int64_t)indptr[id];
            end = (int64_t)indptr[id + 1];
            code = in && !bad ? PART_WIN | (owner & (GS_MAXS - 1)) << PART_OWNER_SHIFT : 0u;
            sg = Segment::make(code, 0);
            const int c = sg.count();
            if (lane < PART_NK) s_seg[wave][lane] = c;
        }
        start_ranks(NoHeads{}, NoHeads::Level{}, (n_targets + 63) >> 6);
        if (bad) s_bad = 1;
        if (code & PART_WIN) {
            const int t = (int)(code >> PART_OWNER_SHIFT);
            const int r = s_base[8 + t] + s_seg[wave][8 + t] + __popcll(sg.win & sg.owned_by(t) & lanemask_lt());
            a.front[r] = (int32_t)id;
            a.perm[r] = tid;
            s_front[r] = (int)id;
            s_beg[r] = beg;
            s_deg[r] = (int)(end - beg);
        }
        if (tid <= S) a.meta[set.L].front_off[tid] = s_o.b[tid];
    }
    __syncthreads();
    if (tid <= set.L) a.meta[tid].error = tid == set.L && s_bad ? 3 : 0;
    if (tid == 0) atomicAdd(&a.meta[0].batches, 1u);    // (a load to wait for stood in front of everything else)
    RowHeads::Level lv{SplitOffs::load(s_o.b, S), S};

    for (int step = 0; step < set.n_layers; ++step) {
        const SmallLayer &out = set.layer[blockIdx.y * set.n_layers + step];
        const int layer = set.L - 1 - step;
        const bool last = step + 1 == set.n_layers;
        const FanDiv fan = set.fan[layer];
        const int n1 = lv.up.n, n_slots = n1 * fan.d;
        // the table empty; the random words (see k_sample_layer), four a thread
        for (int x = tid; x < SMALL_TAB / 2; x += SMALL_T) reinterpret_cast<ulonglong2 *>(s_tab)[x] = make_ulonglong2(EMPTY_ENTRY, EMPTY_ENTRY);
        if (tid == 0) s_long = 0;
        {
            int lw = 0;                 // 2^lw threads a destination
            while ((4 << lw) < fan.d) ++lw;
            for (int x = tid; x < n1 << lw; x += SMALL_T) {
                const int row = x >> lw, q = 4 * (x & ((1 << lw) - 1));
                if (q < fan.d && s_deg[row] > fan.d) {
                    const uint4 r = philox4x32_10(make_uint4((uint32_t)s_front[row], (uint32_t)iter, (uint32_t)(iter >> 32),
                                                             ((uint32_t)layer << 16) | ((uint32_t)q >> 2)),
                                                  make_uint2((uint32_t)seed, (uint32_t)(seed >> 32)));
                    int *w = s_pick + row * fan.d + q;
                    w[0] = (int)r.x;
                    if (q + 1 < fan.d) w[1] = (int)r.y;
                    if (q + 2 < fan.d) w[2] = (int)r.z;
                    if (q + 3 < fan.d) w[3] = (int)r.w;
                }
            }
        }
        __syncthreads();
        // the draws, a lane a slot
        auto draws = [&](auto lanes) __attribute__((always_inline)) {
            constexpr int G = decltype(lanes)::value;
            const int q = lane % G;
            for (int base = wave * (64 / G); base < n1; base += SMALL_T / G) {
                const int row = base + lane / G;
                const bool in = row < n1 && q < fan.d;
                const int d = row < n1 ? s_deg[row] : 0;
                const bool floyd = in && d > fan.d;
                uint32_t t = 0, j = 0;
                if (floyd) {
                    j = (uint32_t)(d - fan.d + q);
                    t = __umulhi((uint32_t)s_pick[row * fan.d + q], j + 1u);
                }
                const uint32_t chosen = __ballot(floyd) != 0ull ? floyd_choice<G>(t, j, fan.d, floyd) : 0u;
                if (in) s_pick[row * fan.d + q] = floyd ? (int)chosen : q < d ? q : -1;
                if (row < n1 && q == 0) out.cnt[row] = min(d, fan.d);
            }
        };
        if (fan.d <= 16) draws(std::integral_constant<int, 16>{});
        else if (fan.d <= 32) draws(std::integral_constant<int, 32>{});
        else draws(std::integral_constant<int, 64>{});
        __syncthreads();
        // slots: neighbour, owner, row of the graph (the next layer's), and the entry of the key
        // (segments of 64 slots, wave by wave; a wave past the last one stays out of the way of the others)
        const int segs = (n_slots + 63) >> 6;
        int id[SMALL_PER], at[SMALL_PER], row[SMALL_PER], split[SMALL_PER];
        unsigned owner[SMALL_PER];
        int64_t beg[SMALL_PER], end[SMALL_PER];
#pragma unroll
        for (int u = 0; u < SMALL_PER; ++u) {
            id[u] = -1;
            at[u] = row[u] = split[u] = 0;
            owner[u] = 0u;
            beg[u] = end[u] = 0;
            if (u * WAVES + wave < segs) {
                const int g = min(tid + u * SMALL_T, n_slots - 1);
                row[u] = fan.div(g);
                split[u] = lv.up.of(row[u]);
                const int pick = s_pick[g];
                const int64_t pos = pick >= 0 ? s_beg[row[u]] + (int64_t)(uint32_t)pick : -1;
                if (pos >= 0) id[u] = indices[pos];
                if (out.epos) out.epos[g] = pos;
                if (g != tid + u * SMALL_T) id[u] = -1;
            }
        }
        int own = 0, own_split = 0, own_first = 0;      // the thread's destination
        if (tid < n1) {
            own = s_front[tid];
            own_split = lv.up.of(tid, lv.up, &own_first);
            small_insert(s_tab, (uint32_t)own, (uint32_t)S, (uint32_t)own_split, (uint32_t)tid);
        }
#pragma unroll
        for (int u = 0; u < SMALL_PER; ++u) {
            const int g = tid + u * SMALL_T;
            if (u * WAVES + wave < segs) {
                if (id[u] >= 0) {
                    owner[u] = pmap[id[u]];
                    if (!last) { beg[u] = (int64_t)indptr[id[u]]; end[u] = (int64_t)indptr[id[u] + 1]; }
                    at[u] = small_insert(s_tab, (uint32_t)id[u], (uint32_t)S, (uint32_t)split[u], (uint32_t)(n1 + g));
                }
                if (g < n_slots) out.nbr[g] = id[u];
            }
        }
        __syncthreads();
        // the first occurrence of the key in its split and of the vertex in the layer
        int first[SMALL_PER], lfirst[SMALL_PER];
        unsigned code[SMALL_PER];
#pragma unroll
        for (int u = 0; u < SMALL_PER; ++u) {
            code[u] = 0u;
            first[u] = lfirst[u] = 0;
            if (u * WAVES + wave < segs) {
                const int pos = n1 + tid + u * SMALL_T;
                if (id[u] >= 0) {
                    first[u] = (int)(uint32_t)s_tab[at[u]];
                    lfirst[u] = S > 1 ? (int)small_first(s_tab, (uint32_t)id[u], (uint32_t)S) : first[u];
                    code[u] = PART_EDGE;
                    if (first[u] == pos) code[u] |= PART_WIN | (owner[u] & (GS_MAXS - 1)) << PART_OWNER_SHIFT | (lfirst[u] == pos ? PART_FIRST : 0u);
                }
                const int c = Segment::make(code[u], split[u]).count();
                if (lane < PART_NK) s_seg[u * WAVES + wave][lane] = c;
            }
        }
        start_ranks(RowHeads{}, lv, segs);
        const int n_lo = s_o.c[GS_MAXS];
        if (tid <= S) { out.meta_lo->mixed_off[tid] = s_o.a[tid]; out.meta_lo->recv_off[tid] = s_o.b[tid]; out.meta_lo->front_off[tid] = s_o.c[tid]; }
        if (tid == GS_MAXS + 1) { out.meta_lo->nnz = s_o.total; out.blk_indptr[n1] = s_o.total; }
        // rows: destinations first, then the winners
        int own_row = 0, own_place = 0;
        int64_t own_beg = 0;
        int own_deg = 0;
        if (tid < n1) {
            const int loc = tid - own_first, j = s_o.a[own_split] + loc;
            own_row = s_o.c[own_split] + loc;
            out.mixed[j] = own;
            out.front_lo[own_row] = own;
            out.src_row[j] = own_row;
            out.self_row[tid] = own_row;
            s_mixed[tid] = loc;
            s_local[tid] = own_row;
            own_beg = s_beg[tid];
            own_deg = s_deg[tid];
        }
        int edge[SMALL_PER], r_mixed[SMALL_PER], r_local[SMALL_PER];
#pragma unroll
        for (int u = 0; u < SMALL_PER; ++u) {
            const int g = tid + u * SMALL_T;
            r_mixed[u] = r_local[u] = -1;
            edge[u] = 0;
            if (u * WAVES + wave < segs) {
                const Segment sg = Segment::make(code[u], split[u]);
                const uint64_t below = lanemask_lt(), won = sg.won_in(split[u]);
                const int *base = s_seg[u * WAVES + wave];
                edge[u] = s_base[16] + base[16] + __popcll(sg.edge & below);
                if (g < n_slots && g == row[u] * fan.d) {
                    out.blk_indptr[row[u]] = edge[u];
                    int sender_first;
                    const int sender = lv.up.of(row[u], lv.up, &sender_first);
                    if (row[u] == sender_first) {       // where the sender's buckets start
#pragma unroll
                        for (int t = 0; t < GS_MAXS; ++t)
                            if (t < S) out.meta_lo->bucket_start[sender * GS_MAXS + t] = s_base[8 + t] + base[8 + t] + __popcll(sg.win & sg.owned_by(t) & below);
                    }
                }
                if (code[u] & PART_WIN) {
                    const int t = (int)(code[u] >> PART_OWNER_SHIFT);
                    const uint64_t same = sg.owned_by(t) & below;
                    r_mixed[u] = s_base[split[u]] + base[split[u]] + __popcll(won & below);
                    out.mixed[r_mixed[u]] = id[u];
                    out.recv[s_base[8 + t] + base[8 + t] + __popcll(sg.win & same)] = id[u];
                    s_mixed[n1 + g] = r_mixed[u] - s_o.a[split[u]];
                    if (code[u] & PART_FIRST) {
                        r_local[u] = s_base[17 + t] + base[17 + t] + __popcll(sg.first & same);
                        out.front_lo[r_local[u]] = id[u];
                        s_local[n1 + g] = r_local[u];
                    }
                }
            }
        }
        const bool rev = out.rev_cnt != nullptr;
        if (rev)
            for (int x = tid; x < n_lo; x += SMALL_T) s_rev[x] = 0;
        __syncthreads();
        // the level below as the next layer reads it
        if (!last) {
            if (tid < n1) { s_front[own_row] = own; s_beg[own_row] = own_beg; s_deg[own_row] = own_deg; }
#pragma unroll
            for (int u = 0; u < SMALL_PER; ++u)
                if (r_local[u] >= 0) { s_front[r_local[u]] = id[u]; s_beg[r_local[u]] = beg[u]; s_deg[r_local[u]] = (int)(end[u] - beg[u]); }
        }
        // the shuffle index, and each entry's place in its row of the reverse index
        int src[SMALL_PER], place[SMALL_PER];
#pragma unroll
        for (int u = 0; u < SMALL_PER; ++u) {
            src[u] = place[u] = 0;
            if (id[u] >= 0) {
                src[u] = s_local[lfirst[u]];
                out.blk_src[edge[u]] = s_mixed[first[u]];
                out.edge_row[edge[u]] = src[u];
                if (r_mixed[u] >= 0) out.src_row[r_mixed[u]] = src[u];
                if (rev) place[u] = atomicAdd(&s_rev[src[u]], 1);
            }
        }
        if (rev) {
            if (tid < n1) own_place = atomicAdd(&s_rev[own_row], 1);
            __syncthreads();
            // segments in the order of the rows
            constexpr int PER = SMALL_MAX / SMALL_T;
            int c[PER], sum = 0;
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const int x = tid * PER + u;
                c[u] = x < n_lo ? s_rev[x] : 0;
                sum += c[u];
            }
            int inc = sum;
            if (wave * 64 * PER < n_lo) {
                for (int o = 1; o < 64; o <<= 1) {
                    const int below = __shfl_up(inc, o);
                    if (lane >= o) inc += below;
                }
            }
            if (lane == 63) s_wave[wave] = inc;
            __syncthreads();
            if (wave * 64 * PER < n_lo) {
                int p = inc - sum;
                for (int w = 0; w < wave; ++w) p += s_wave[w];
#pragma unroll
                for (int u = 0; u < PER; ++u) {
                    const int x = tid * PER + u;
                    if (x < n_lo) {
                        out.rev_cnt[x] = c[u];
                        out.rev_ptr[x] = p;
                        s_rev[x] = p;
                        if (c[u] > GS_REV_LONG) out.rev_long[atomicAdd(&s_long, 1)] = x;
                    }
                    p += c[u];
                }
            }
            __syncthreads();
            if (tid == 0) { out.meta_lo->rev_cursor = n1 + s_o.total; out.meta_lo->n_long = s_long; }
            if (tid < n1) {
                const int p = s_rev[own_row] + own_place;
                out.rev_list[p] = 2 * tid;
                if (out.rev_eid) out.rev_eid[p] = -1;
            }
#pragma unroll
            for (int u = 0; u < SMALL_PER; ++u)
                if (id[u] >= 0) {
                    const int p = s_rev[src[u]] + place[u];
                    out.rev_list[p] = 2 * row[u] + 1;
                    if (out.rev_eid) out.rev_eid[p] = edge[u];
                }
        }
        lv.up = SplitOffs::load(s_o.c, S);
        __syncthreads();
    }
}

// The scatter side of the shuffle index of the sampling layer above (layer l+1) is finished while
// layer l is partitioned: its rows are this layer's destination vertices, and its counters are
// complete once the shuffle-index kernel of layer l+1 has run.  The count pass hands every row a
// segment of rev_list (segments need not be in row order: one atomic per workgroup of 256 rows
// on the cursor, a single address), the scatter pass lists, for every source row, the destination
// rows it feeds (slot q of destination i is a sampled edge when q < cnt[i]).
struct RevUp {
    int on;
    const int32_t *rev_cnt; int32_t *rev_ptr; int32_t *rev_fill; int32_t *rev_list; int32_t *rev_eid;
    const int32_t *cnt; const int32_t *blk_indptr; const int32_t *self_row; const int32_t *edge_row;
    FanDiv fan; int32_t *cursor; const GsLevelMeta *meta_up2; int32_t *rev_long; int32_t *n_long;
    __device__ void alloc(int64_t x, int64_t n_rows) const {
        __shared__ int s_wave[PART_BS / 64];
        __shared__ int s_base;
        const int lane = lane_id(), wave = threadIdx.x >> 6;
        const int c = x < n_rows ? rev_cnt[x] : 0;
        int inc = c;
        for (int o = 1; o < 64; o <<= 1) {
            const int below = __shfl_up(inc, o);
            if (lane >= o) inc += below;
        }
        if (lane == 63) s_wave[wave] = inc;
        __syncthreads();
        if (threadIdx.x == 0) {
            int tot = 0;
            for (int w = 0; w < PART_BS / 64; ++w) { const int t = s_wave[w]; s_wave[w] = tot; tot += t; }
            s_base = tot > 0 ? atomicAdd(cursor, tot) : 0;
        }
        __syncthreads();
        if (x < n_rows) {
            rev_ptr[x] = s_base + s_wave[wave] + inc - c;
            rev_fill[x] = 0;
            if (c > GS_REV_LONG) rev_long[atomicAdd(n_long, 1)] = (int32_t)x;      // (rare: one atomic per such row)
        }
        __syncthreads();
    }
    __device__ int n_dst(int S) const { return on ? meta_up2->front_off[S] : 0; }
    __device__ void fill(int64_t x, int n_dst) const {
        int u, code, eid = -1;
        if (x < n_dst) {
            u = self_row[x];
            code = 2 * (int)x;
        } else {
            const int g = (int)x - n_dst;
            const int i = fan.div(g), q = g - i * fan.d;
            if (q >= cnt[i]) return;
            eid = blk_indptr[i] + q;
            u = edge_row[eid];
            code = 2 * i + 1;
        }
        if (u < 0) return;
        const int p = atomicAdd(&rev_fill[u], 1);
        rev_list[rev_ptr[u] + p] = code;
        if (rev_eid) rev_eid[rev_ptr[u] + p] = eid;
    }
};

// ---- the partition of a sampling layer: mixed frontiers, block CSR offsets, owner buckets and
// next local frontiers in one pass over the slots.  A slot that is the first occurrence of its
// vertex inside its split s ("winner") gets
//   class s       -> its row in mixed_front_s (destination vertices occupy the rows before)
//   class 8 + t   -> its place in bucket[s -> t], t = f_G(vertex): partitioning the sender-ordered
//                    slot stream by owner yields, for each receiver t, bucket[0->t] | bucket[1->t]
//                    | ...: on one GPU the send buffers and the received concatenation are the
//                    same memory.
// Class 16 counts valid slots: its exclusive rank is the edge number (block CSR offsets).
// A slot that is the first occurrence of its vertex in the whole stream (and whose vertex is not a
// destination vertex, which the table decides: destinations hold the smallest positions) gets
//   class 17 + t  -> its row in local_front[l]_t (the owner's own destination vertices come first).
struct PartLayer {
    GsTable tab; int32_t *row_mixed; int32_t *row_local;
    const int32_t *front; const int32_t *nbr; const uint8_t *pmap;
    int32_t *ent_mixed; int32_t *first_any; uint8_t *cls; int32_t *mixed_ent;
    int32_t *mixed; int32_t *blk_indptr; int32_t *recv; int32_t *front_lo; int32_t *rev_cnt;
    GsLevelMeta *meta_lo; const GsLevelMeta *meta_up; int S; FanDiv fan; int rev;
    RevUp up;
    int layer;
    int32_t *pos_pair; int32_t *mixed_pos;      // a wide layer's (null otherwise)
    int fan_next; int64_t top_cap;              // hashed: what the next sampling layer can use of the table (see extra)
    struct Level { SplitOffs up; int n_up2; };      // split offsets of the destinations; rows two levels up
    struct Elem { unsigned code; int split; int32_t id, first; };
    __device__ Level load() const { return Level{SplitOffs::load(meta_up->front_off, S), up.n_dst(S)}; }
    __device__ int n(const Level &lv) const { return lv.up.n * fan.d; }
    // From here on an element's ent_mixed no longer names a table entry but the position
    // of the first occurrence of its key (what the entry holds), and first_any that of a winner's vertex in the
    // whole stream: the rows are handed out by position (row_mixed, row_local), so the later passes read
    // small dense arrays instead of following every element into the table again.  A slot that was behind
    // another element when it was sampled is no winner and is left as it is: no access to the table for it here, one
    // to ent_mixed in the relabelling (count pass of 266k skewed destinations x 20 136 -> 86 us, relabelling 79 -> 95;
    // 567k x 10 187 -> 159, 87 -> 93; eight batches of 21.6k x 15 91 -> 80, 43 -> 47).
    __device__ unsigned classify(const Level &lv, int g, int *split) const {
        const int at = lv.up.n + g;
        const int h = ent_mixed[at];
        const int32_t id = nbr[g];                          // -1 in an empty slot
        const uint32_t pos = (uint32_t)at;
        unsigned m = h != -1 ? PART_EDGE : 0u;
        if (h >= 0) {
            // One table of (vertex, split) keys.  Direct: the vertex's entries for the single splits lie
            // side by side; the slot's own one tells where its key first occurs, the smallest of those
            // that carry this layer's stamp where the vertex first occurs in the whole stream.  Hashed:
            // the slot's own entry, and for a winner the smallest position in the vertex's lines.
            const int s = lv.up.of(fan.div(g));
            uint32_t first = pos, lfirst = pos;
            unsigned t = 0u;
            if (tab.pos) {
                // (what the answer needs is fetched side by side, the owner byte beside the entries although only
                // a winner wants it: the kernel of a small layer is a chain of dependent accesses)
                t = pmap[id] & (GS_MAXS - 1);
                const uint32_t stamp = table_stamp(meta_lo - layer, (uint32_t)layer);
                const unsigned long long *e = tab.pos + (size_t)(uint32_t)id * (uint32_t)S;
                // (an entry the context does not have reads as empty, whose upper half is no stamp)
                unsigned long long v[GS_MAXS];
#pragma unroll
                for (int ss = 0; ss < GS_MAXS; ++ss) v[ss] = ss < S ? e[ss] : EMPTY_ENTRY;
#pragma unroll
                for (int ss = 0; ss < GS_MAXS; ++ss) {
                    if (ss == s) first = (uint32_t)v[ss];
                    if ((uint32_t)(v[ss] >> 32) == stamp) lfirst = min(lfirst, (uint32_t)v[ss]);
                }
            } else {
                // (the form of the large layers, which run at the rate of their random accesses, not of the chain:
                // the owner is fetched for the winners alone)
                first = (uint32_t)tab.slot[h];
                if (first == pos) {
                    t = pmap[id] & (GS_MAXS - 1);
                    if (S > 1) lfirst = table_line_first(tab, table_bits(lv.up.n * (1 + fan.d)), (uint32_t)id, (uint32_t)S, pos);
                }
            }
            ent_mixed[at] = (int32_t)first;
            if (first == pos) {
                m |= PART_WIN | t << PART_OWNER_SHIFT;
                *split = s;
                first_any[at] = (int32_t)lfirst;
                if (lfirst == pos) m |= PART_FIRST;
            }
        }
        cls[g] = (uint8_t)m;
        return m;
    }
    // the id and the vertex's first occurrence are wanted of the winners only, but asked for with the mask:
    // one level of the chain less, in lines that the winners among the neighbours read anyway
    __device__ Elem cached(const Level &lv, int g) const {
        return Elem{cls[g], lv.up.of(fan.div(g)), nbr[g], first_any[lv.up.n + g]};
    }
    // destination vertices are the first rows of their split's mixed frontier and of their owner's next
    // local frontier
    __device__ int heads(const Level &lv, int s) const {
        int first = 0, next = 0;
#pragma unroll
        for (int k = 0; k < GS_MAXS; ++k)
            if (k == s) { first = lv.up.o[k]; next = lv.up.o[k + 1]; }
        return s < S ? next - first : 0;
    }
    __device__ void publish(const Level &lv, const PartOffs &o) const {
        const int s = threadIdx.x;
        if (s <= S) { meta_lo->mixed_off[s] = o.a[s]; meta_lo->recv_off[s] = o.b[s]; meta_lo->front_off[s] = o.c[s]; }
        if (s == GS_MAXS + 1) { meta_lo->nnz = o.total; blk_indptr[lv.up.n] = o.total; }
    }
    __device__ void emit(const Level &lv, int g, bool in, const Elem &e, const Segment &sg, const int *base, const PartOffs &o) const {
        const uint64_t below = lanemask_lt();
        const int i = fan.div(g), q = g - i * fan.d;
        bool starts = false;        // the first slot of a split
        int sender = 0;
        if (in && q == 0) {
            blk_indptr[i] = base[16] + __popcll(sg.edge & below);
            int first;
            sender = lv.up.of(i, lv.up, &first);
            starts = i == first;
        }
        // the first row of a sender marks where its buckets start at every receiver
        // (senders are consecutive in the slot stream); sizes follow by subtraction on the host
        if (starts) {
#pragma unroll
            for (int t = 0; t < GS_MAXS; ++t)
                if (t < S) meta_lo->bucket_start[sender * GS_MAXS + t] = base[8 + t] + __popcll(sg.win & sg.owned_by(t) & below);
        }
        const uint64_t won = sg.won_in(e.split);
        if (!(e.code & PART_WIN)) return;
        const int t = (int)(e.code >> PART_OWNER_SHIFT);
        const uint64_t same = sg.owned_by(t) & below;
        const int at = lv.up.n + g;            // a winner: the first occurrence of its (vertex, split) key
        const int r_mixed = base[e.split] + __popcll(won & below);
        const int r_recv = base[8 + t] + __popcll(sg.win & same);
        const int row = r_mixed - o.a[e.split];
        mixed[r_mixed] = e.id;
        if (pos_pair) { pos_pair[2 * (size_t)at] = row; mixed_pos[r_mixed] = at; }
        else row_mixed[at] = row;
        mixed_ent[r_mixed] = e.first;          // where the vertex first occurs in the whole stream
        recv[r_recv] = e.id;
        if (e.code & PART_FIRST) {             // that place is this one
            const int r_local = base[17 + t] + __popcll(sg.first & same);
            front_lo[r_local] = e.id;
            row_local[at] = r_local;
        }
    }
    // scatter pass extras: destination vertices are rows 0 .. n_dst-1 of their split's mixed
    // frontier and of their owner's next local frontier; then (layers that have one) the counters
    // of this layer's reverse index are zeroed; then the reverse index of the layer above is filled
    __device__ int64_t n_extra(const Level &lv, const PartOffs &o) const {
        return (int64_t)lv.up.n + (rev ? o.c[S] : 0) + (int64_t)lv.n_up2 * (1 + up.fan.d);
    }
    // then a hashed table, which the count pass was the last to read, is cleared as far as the next sampling layer
    // can use it (after the bottom layer: as far as a top layer of max_targets targets can); a power of two of entries
    __device__ void clear(const PartOffs &o, int64_t x, int64_t stride) const {
        if (tab.pos) return;
        const int64_t pairs = (fan_next > 0 ? 1ll << table_bits(o.c[S] * (1 + fan_next)) : top_cap) >> 1;
        ulonglong2 *slot = reinterpret_cast<ulonglong2 *>(tab.slot);
#pragma unroll 4
        for (; x < pairs; x += stride) slot[x] = make_ulonglong2(EMPTY_ENTRY, EMPTY_ENTRY);
    }
    __device__ void extra(const Level &lv, int64_t x, const PartOffs &o) const {
        const int64_t own = lv.up.n + (rev ? o.c[S] : 0);
        if (x >= own) {
            up.fill(x - own, lv.n_up2);
            return;
        }
        if (x >= lv.up.n) {
            rev_cnt[x - lv.up.n] = 0;
            if (x == lv.up.n) { meta_lo->rev_cursor = 0; meta_lo->n_long = 0; }
            return;
        }
        const int i = (int)x;
        int first;
        const int s = lv.up.of(i, lv.up, &first);
        const int loc = i - first;
        const int32_t id = front[i];
        const int h = ent_mixed[i];
        const int j = o.a[s] + loc, rowp = o.c[s] + loc;
        // a destination vertex holds the smallest position of its key and of its vertex: position i
        mixed[j] = id;
        if (pos_pair) { pos_pair[2 * (size_t)i] = loc; mixed_pos[j] = i; }
        else row_mixed[i] = loc;
        mixed_ent[j] = h >= 0 ? i : -1;
        front_lo[rowp] = id;
        row_local[i] = rowp;
    }
    // count pass side work: segments of the reverse index of the layer above
    __device__ int64_t n_side(const Level &lv) const { return up.on ? lv.up.n : 0; }
    __device__ void side(const Level &, int64_t x, int64_t ns) const { up.alloc(x, ns); }
};

// the relabelling of a layer as launches of its own: the bottom layer's, and the index of a wide layer, whose edges wait
// for it (static arrays of gsplit_sample_split_noalloc: every layer's)
__global__ __launch_bounds__(256) void k_shuffle_index(ShuffleArgsSet set, int S, FanDiv fan) {
    shuffle_index(set.b[blockIdx.y], S, fan, blockIdx.x, gridDim.x);
}
__global__ __launch_bounds__(256) void k_shuffle_edges(ShuffleArgsSet set, int S, FanDiv fan) {
    shuffle_edges(set.b[blockIdx.y], S, fan, blockIdx.x, gridDim.x);
}

// reverse index as two launches of its own (blockIdx.y = layer - first): used for the bottom layer,
// which has no partition below it; same steps as RevUp::alloc / RevUp::fill
struct RevArgs {
    const int32_t *rev_cnt; int32_t *rev_ptr; int32_t *rev_fill; int32_t *rev_list; int32_t *rev_eid; int32_t *rev_long;
    const int32_t *cnt; const int32_t *blk_indptr; const int32_t *self_row; const int32_t *edge_row;
    GsLevelMeta *meta;          // the batch's level bookkeeping, [L + 1]
};
struct RevArgsSet { RevArgs b[GS_MAXB]; };

// step 2: give every row of local_cat[l] a segment of rev_list (segments need not be in row order:
// one atomic per workgroup of 1024 rows hands out space; the cursor is a single address, and an
// atomic on it from every wave of a million-row level took longer than the rest of the kernel)
__global__ __launch_bounds__(1024) void k_rev_alloc(RevArgsSet set, int l, int S) {
    __shared__ int s_wave[16];
    __shared__ int s_base;
    const RevArgs &a = set.b[blockIdx.y];
    GsLevelMeta *meta_lo = a.meta + l;
    const int32_t *__restrict__ rev_cnt = a.rev_cnt;
    int32_t *__restrict__ rev_ptr = a.rev_ptr;
    int32_t *__restrict__ rev_fill = a.rev_fill;
    const int n_lo = meta_lo->front_off[S];
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int stride = gridDim.x * blockDim.x;
    const int rounds = (n_lo + stride - 1) / stride;
    for (int it = 0; it < rounds; ++it) {
        const int u = it * stride + blockIdx.x * blockDim.x + threadIdx.x;
        const int c = u < n_lo ? rev_cnt[u] : 0;
        int inc = c;
        for (int o = 1; o < 64; o <<= 1) {
            int up = __shfl_up(inc, o);
            if (lane >= o) inc += up;
        }
        if (lane == 63) s_wave[wave] = inc;
        __syncthreads();
        if (threadIdx.x == 0) {
            int tot = 0;
            for (int w = 0; w < 16; ++w) { const int x = s_wave[w]; s_wave[w] = tot; tot += x; }
            s_base = tot > 0 ? atomicAdd(&meta_lo->rev_cursor, tot) : 0;
        }
        __syncthreads();
        if (u < n_lo) {
            rev_ptr[u] = s_base + s_wave[wave] + inc - c;
            rev_fill[u] = 0;
            if (c > GS_REV_LONG) a.rev_long[atomicAdd(&meta_lo->n_long, 1)] = u;
        }
        __syncthreads();
    }
}

// step 3: list, for every source row, the destination rows it feeds (slot q of destination i is a
// sampled edge when q < cnt[i])
__global__ __launch_bounds__(256) void k_rev_fill(RevArgsSet set, int l, FanDiv fan, int S) {
    const RevArgs &a = set.b[blockIdx.y];
    const int32_t *__restrict__ cnt = a.cnt;
    const int32_t *__restrict__ blk_indptr = a.blk_indptr;
    const int32_t *__restrict__ self_row = a.self_row;
    const int32_t *__restrict__ edge_row = a.edge_row;
    const int32_t *__restrict__ rev_ptr = a.rev_ptr;
    int32_t *__restrict__ rev_fill = a.rev_fill;
    int32_t *__restrict__ rev_list = a.rev_list;
    int32_t *__restrict__ rev_eid = a.rev_eid;
    const int n1 = a.meta[l + 1].front_off[S];
    const int64_t total = (int64_t)n1 * (1 + fan.d);
    for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < total;
         x += (int64_t)gridDim.x * blockDim.x) {
        int u, code, eid = -1;
        if (x < n1) {
            u = self_row[x];
            code = 2 * (int)x;
        } else {
            const int g = (int)x - n1;
            const int i = fan.div(g), q = g - i * fan.d;
            if (q >= cnt[i]) continue;
            eid = blk_indptr[i] + q;
            u = edge_row[eid];
            code = 2 * i + 1;
        }
        if (u < 0) continue;
        const int p = atomicAdd(&rev_fill[u], 1);
        rev_list[rev_ptr[u] + p] = code;
        if (rev_eid) rev_eid[rev_ptr[u] + p] = eid;
    }
}

int part_blocks(int64_t upper_items) {
    return upper_items <= (1 << 18) ? 256 : upper_items <= (1 << 20) ? 512 : PART_MAX_NB;
}

// kernel arguments are limited to 4 KiB
static_assert(sizeof(PartSet<PartLayer>) <= 4096 && sizeof(PartSet<PartTargets>) <= 4096 && sizeof(TargetsSet) <= 4096 &&
              sizeof(SampleArgsSet) + sizeof(ShuffleArgsSet) + sizeof(Ride) <= 4000 && sizeof(RevArgsSet) <= 3072,
              "argument block of a multi-batch launch too large");

template <class F>
void run_partition(gsplit_ctx *const *ctxs, int nbat, const PartSet<F> &set, int64_t upper_items, hipStream_t st,
                   const char *name, int layer) {
    gsplit_ctx *ctx = ctxs[0];
    const int nb = part_blocks(upper_items);
    const std::string nm(name);
    {
        GsTimeScope ts(ctx, (nm + "_count").c_str(), layer, st);
        hipLaunchKernelGGL(k_part_count<F>, dim3(nb, nbat), dim3(PART_BS), 0, st, set);
    }
    GsTimeScope ts(ctx, (nm + "_scatter").c_str(), layer, st);
    hipLaunchKernelGGL(k_part_scatter<F>, dim3(nb, nbat), dim3(PART_BS), 0, st, set);
}

// entry indices of layer l's elements: two arrays in turn, so that the layer above can still be read
int32_t *ent_mixed_of(const gsplit_ctx *c, int l) { return (l & 1) && c->ent_mixed_odd ? c->ent_mixed_odd : c->ent_mixed; }

// grid of a grid-stride kernel over upper_items elements; with several batches in the launch the
// cap on resident workgroups is shared between them
int grid_for(const gsplit_ctx *ctx, int64_t upper_items, int nbat = 1) {
    int64_t want = gs_ceil_div(upper_items, 256);
    int64_t cap = std::max<int64_t>(1, (int64_t)ctx->n_cu * ctx->sampler_blocks_per_cu / nbat);
    if (want < 1) want = 1;
    return (int)(want < cap ? want : cap);
}

// the relabelling of layer l + 1 that rides on the sampler of layer l
struct RideAbove { int what = RIDE_NONE; ShuffleArgsSet args{}; };

template <typename IndPtrT>
void launch_sample(gsplit_ctx *const *ctxs, int nbat, int l, uint64_t seed, const uint64_t *iters,
                   const uint64_t *d_seed_iter, const RideAbove &above, hipStream_t st) {
    gsplit_ctx *ctx = ctxs[0];
    const int fan = ctx->fan[l];
    const int64_t ub = ctx->ub_front[l + 1];
    const IndPtrT *ip = (const IndPtrT *)ctx->graph.d_indptr;
    SampleArgsSet set{};
    for (int b = 0; b < nbat; ++b) {
        gsplit_ctx *c = ctxs[b];
        GsLayerBuf &B = c->layer[l];
        set.b[b] = SampleArgs{c->front[l + 1], c->d_meta + l, c->d_meta + (l + 1), c->tab_mixed, ent_mixed_of(c, l), B.nbr, B.cnt,
                              B.epos, iters[b], d_seed_iter};
    }
    Ride ride{above.what, FanDiv::make(1), 0};
    int riders = 0;
    if (above.what != RIDE_NONE) {
        const int fan_up = ctx->fan[l + 1];
        ride.fan = FanDiv::make(fan_up);
        riders = grid_for(ctx, ctx->ub_front[l + 2] * (above.what == RIDE_INDEX ? 2 + 2 * fan_up : fan_up), nbat);
    }
    GsTimeScope ts(ctx, "sample_layer", l, st);
#define GS_SAMPLE(G)                                                                                                     \
    do {                                                                                                                 \
        ride.n_main = grid_for(ctx, ub * G, nbat);                                                                       \
        hipLaunchKernelGGL((k_sample_layer<G, IndPtrT>), dim3(ride.n_main + riders, nbat), dim3(256), 0, st, ip,         \
                           ctx->graph.d_indices, set, ctx->S, fan, (uint32_t)l, seed, above.args, ride);                 \
    } while (0)
    if (fan <= 16) GS_SAMPLE(16);
    else if (fan <= 32) GS_SAMPLE(32);
    else GS_SAMPLE(64);
#undef GS_SAMPLE
}

// Layers from the top that k_sample_small takes, by the bound on their elements that follows from the targets at hand.
// The bound, not the live rows: the host does not know them.
int small_layers(const gsplit_ctx *ctx, int64_t n_targets, int nbat, int64_t *rows_below) {
    int64_t rows = n_targets;
    int n = 0;
    const bool alone = nbat == 1 && ctx->tab_mixed.pos;
    while (n < ctx->L && n < SMALL_LAYERS / nbat && rows <= SMALL_ROWS) {
        const int64_t slots = rows * ctx->fan[ctx->L - 1 - n];
        if (slots > SMALL_SLOTS || (alone && 2 * rows + slots > SMALL_ALONE)) break;
        rows = std::min(ctx->graph.n_vertices, rows + slots);
        ++n;
    }
    *rows_below = rows;
    return n;
}

void launch_small(gsplit_ctx *const *ctxs, int nbat, int n_layers, int64_t rows_below, const int32_t *const *d_targets,
                  const int64_t *n_targets, uint64_t seed, const uint64_t *iters, const uint64_t *d_seed_iter, hipStream_t st) {
    gsplit_ctx *ctx = ctxs[0];
    const int L = ctx->L, below = L - 1 - n_layers;     // the first layer of the general path (-1: none is left)
    SmallSet set{};
    set.seed_iter = d_seed_iter;
    set.n_layers = n_layers;
    set.L = L;
    for (int l = 0; l < L; ++l) set.fan[l] = FanDiv::make(ctx->fan[l]);
    for (int b = 0; b < nbat; ++b) {
        gsplit_ctx *c = ctxs[b];
        set.b[b] = SmallBatch{d_targets[b], c->front[L], c->target_perm, c->d_meta, c->tab_mixed.slot, iters[b], (int)n_targets[b]};
        for (int i = 0; i < n_layers; ++i) {
            const int l = L - 1 - i;
            const GsLayerBuf &B = c->layer[l];
            SmallLayer &o = set.layer[b * n_layers + i];
            o = SmallLayer{c->d_meta + l, B.nbr, B.cnt, B.epos, B.mixed, B.blk_indptr, B.blk_src, B.recv, B.src_row, B.self_row,
                           B.edge_row, c->front[l], nullptr, nullptr, nullptr, nullptr, nullptr};
            if (l >= c->rev_from) { o.rev_cnt = B.rev_cnt; o.rev_ptr = B.rev_ptr; o.rev_list = B.rev_list; o.rev_eid = B.rev_eid; o.rev_long = B.rev_long; }
        }
    }
    int riders = 0;
    if (below >= 0 && !ctx->tab_mixed.pos) {
        int64_t cap = 1024;                             // = 1 << table_bits(rows_below * (1 + fan))
        while (cap < 2 * rows_below * (1 + ctx->fan[below])) cap <<= 1;
        set.clear_pairs = cap >> 1;
        riders = (int)std::min<int64_t>(ctx->n_cu, gs_ceil_div(set.clear_pairs, 4 * SMALL_T));
    }
    GsTimeScope ts(ctx, "sample_small", L - 1, st);
    const dim3 grid(1 + riders, nbat), block(SMALL_T);
    if (ctx->graph.indptr_is_64)
        hipLaunchKernelGGL((k_sample_small<int64_t>), grid, block, 0, st, (const int64_t *)ctx->graph.d_indptr, ctx->graph.d_indices,
                           ctx->graph.d_pmap, (uint32_t)ctx->graph.n_vertices, ctx->S, set, seed);
    else
        hipLaunchKernelGGL((k_sample_small<int32_t>), grid, block, 0, st, (const int32_t *)ctx->graph.d_indptr, ctx->graph.d_indices,
                           ctx->graph.d_pmap, (uint32_t)ctx->graph.n_vertices, ctx->S, set, seed);
}

// One event behind the batches of a call, in all their contexts.  It is one of their own that no other context still
// waits for the previous record of; where there is none (they were grouped otherwise before), a new one.
int record_done(gsplit_ctx *const *ctxs, int nbat, hipStream_t st) {
    for (int b = 0; b < nbat; ++b) ctxs[b]->sample_done.reset();
    std::shared_ptr<GsEvent> done;
    for (int b = 0; b < nbat && !done; ++b)
        if (ctxs[b]->own_done.use_count() == 1) done = ctxs[b]->own_done;
    if (!done) {
        done = GsEvent::make();
        if (!done) return gs_fail(ctxs[0], GSPLIT_EHIP, "gsplit_sample_split: no event");
        ctxs[0]->own_done = done;
    }
    GS_HIP(ctxs[0], hipEventRecord(done->ev, st));
    for (int b = 0; b < nbat; ++b) ctxs[b]->sample_done = done;
    return GSPLIT_OK;
}

// Algorithm 1 for nbat mini-batches at once, one context each (same graph, same configuration)
int sample_split(gsplit_ctx *const *ctxs, int nbat, const int32_t *const *d_targets, const int64_t *n_targets,
                 uint64_t seed, const uint64_t *iters, const uint64_t *d_seed_iter, void *stream) {
    gsplit_ctx *ctx = ctxs[0];
    for (int b = 0; b < nbat; ++b) {
        if (n_targets[b] < 0 || (n_targets[b] > 0 && !d_targets[b]))
            return gs_fail(ctx, GSPLIT_EINVAL, "gsplit_sample_split: bad targets");
        if (n_targets[b] > ctxs[b]->max_targets)
            return gs_fail(ctx, GSPLIT_ECAPACITY, "gsplit_sample_split: n_targets exceeds max_targets");
    }
    hipStream_t st = (hipStream_t)stream;
    const int S = ctx->S, L = ctx->L;
    // Under stream capture the calls of a step become nodes of a graph: no event is recorded for the
    // host-side queries (they synchronise the device instead) and no timing events are taken.
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cap) != hipSuccess) {
        (void)hipGetLastError();
        cap = hipStreamCaptureStatusNone;
    }
    bool all_small = true;
    for (int b = 0; b < nbat; ++b) {
        gsplit_ctx *c = ctxs[b];
        c->captured = cap == hipStreamCaptureStatusActive;
        c->batch_id += 1;
        c->n_targets = n_targets[b];
        c->h_meta_valid = false;
        c->sage.fwd_done = false;
        c->last_stream = st;
        all_small = all_small && n_targets[b] <= TARGETS_SMALL;
    }

    int64_t top_cap = 1024;                             // = 1 << table_bits(max_targets * (1 + fan_top))
    while (top_cap < 2 * ctx->max_targets * (1 + ctx->fan[L - 1])) top_cap <<= 1;
    int64_t rows_below = 0;
    const int n_small = small_layers(ctx, *std::max_element(n_targets, n_targets + nbat), nbat, &rows_below);
    if (n_small > 0) {
        launch_small(ctxs, nbat, n_small, rows_below, d_targets, n_targets, seed, iters, d_seed_iter, st);
    } else {
        auto targets_of = [&](int b) {
            gsplit_ctx *c = ctxs[b];
            return PartTargets{d_targets[b], (int)n_targets[b], c->graph.d_pmap, S, (uint32_t)c->graph.n_vertices,
                               c->front[L], c->target_perm, c->d_meta + L, c->d_meta, L + 1};
        };
        if (all_small) {
            TargetsSet set{};
            for (int b = 0; b < nbat; ++b) set.f[b] = targets_of(b);
            GsTimeScope ts(ctx, "targets", -1, st);
            hipLaunchKernelGGL(k_targets_small, dim3(nbat), dim3(TARGETS_SMALL), 0, st, set);
        } else {
            PartSet<PartTargets> set{};
            for (int b = 0; b < nbat; ++b) { set.f[b] = targets_of(b); set.hist[b] = ctxs[b]->part_hist; }
            run_partition(ctxs, nbat, set, ctx->ub_front[L], st, "targets", -1);
        }
    }

    bool may_ride = true;       // (not with the static arrays, which have no second one for the entry indices)
    for (int b = 0; b < nbat; ++b) may_ride = may_ride && (L == 1 || ctxs[b]->ent_mixed_odd);
    RideAbove above;
    for (int l = L - 1 - n_small; l >= 0; --l) {
        const int fan = ctx->fan[l];
        const int64_t ub1 = ctx->ub_front[l + 1];

        if (ctx->graph.indptr_is_64) launch_sample<int64_t>(ctxs, nbat, l, seed, iters, d_seed_iter, above, st);
        else launch_sample<int32_t>(ctxs, nbat, l, seed, iters, d_seed_iter, above, st);

        PartSet<PartLayer> pset{};
        ShuffleArgsSet &sset = above.args;
        bool wide = ub1 * fan >= ctx->wide_slots;
        for (int b = 0; b < nbat; ++b) wide = wide && ctxs[b]->pos_pair && ctxs[b]->mixed_pos;
        for (int b = 0; b < nbat; ++b) {
            gsplit_ctx *c = ctxs[b];
            GsLayerBuf &B = c->layer[l];
            GsLevelMeta *ml = c->d_meta + l;
            const GsLevelMeta *mu = c->d_meta + (l + 1);
            PartLayer pa{c->tab_mixed, c->tab_mixed.row, c->row_local, c->front[l + 1], B.nbr, c->graph.d_pmap,
                         ent_mixed_of(c, l), c->first_any, c->cls, c->mixed_ent,
                         B.mixed, B.blk_indptr, B.recv, c->front[l], B.rev_cnt,
                         ml, mu, S, FanDiv::make(fan), l >= c->rev_from ? 1 : 0, RevUp{}, l,
                         wide ? c->pos_pair : nullptr, wide ? c->mixed_pos : nullptr,
                         l > 0 ? ctx->fan[l - 1] : 0, l == 0 ? top_cap : 0};
            if (l + 1 < L - n_small && l + 1 >= c->rev_from) {
                const GsLayerBuf &U = c->layer[l + 1];
                pa.up = RevUp{1, U.rev_cnt, U.rev_ptr, U.rev_fill, U.rev_list, U.rev_eid, U.cnt, U.blk_indptr,
                              U.self_row, U.edge_row, FanDiv::make(c->fan[l + 1]), &c->d_meta[l + 1].rev_cursor, c->d_meta + (l + 2),
                              U.rev_long, &c->d_meta[l + 1].n_long};
            }
            pset.f[b] = pa;
            pset.hist[b] = c->part_hist;
            sset.b[b] = ShuffleArgs{c->tab_mixed.row, c->row_local, ent_mixed_of(c, l), c->mixed_ent, B.blk_indptr,
                                    B.blk_src, B.src_row, B.self_row, B.edge_row, l >= c->rev_from ? B.rev_cnt : nullptr,
                                    ml, mu, wide ? c->pos_pair : nullptr, wide ? c->mixed_pos : nullptr};
        }
        run_partition(ctxs, nbat, pset, ub1 * fan, st, "mixed_buckets", l);
        const bool rides = may_ride && l > 0;
        if (wide || !rides) {
            GsTimeScope ts(ctx, "shuffle_index", l, st);
            hipLaunchKernelGGL(k_shuffle_index, dim3(grid_for(ctx, ub1 * (2 + 2 * fan), nbat), nbat), dim3(256), 0, st,
                               sset, S, FanDiv::make(fan));
        }
        if (wide && !rides) {
            GsTimeScope ts(ctx, "shuffle_edges", l, st);
            hipLaunchKernelGGL(k_shuffle_edges, dim3(grid_for(ctx, ub1 * fan, nbat), nbat), dim3(256), 0, st, sset, S, FanDiv::make(fan));
        }
        above.what = !rides ? RIDE_NONE : wide ? RIDE_EDGES : RIDE_INDEX;
    }
    // the bottom layer's reverse index (contexts that keep one) has no partition below it to ride on
    if (ctx->rev_from == 0 && n_small < L) {
        RevArgsSet ra{};
        for (int b = 0; b < nbat; ++b) {
            const GsLayerBuf &B = ctxs[b]->layer[0];
            ra.b[b] = RevArgs{B.rev_cnt, B.rev_ptr, B.rev_fill, B.rev_list, B.rev_eid, B.rev_long, B.cnt, B.blk_indptr,
                              B.self_row, B.edge_row, ctxs[b]->d_meta};
        }
        const int64_t rows = std::max<int64_t>(1, ctx->ub_front[0]);
        const int64_t items = std::max<int64_t>(1, ctx->ub_front[1] * (1 + ctx->fan[0]));
        {
            GsTimeScope ts(ctx, "rev_alloc", -1, st);
            hipLaunchKernelGGL(k_rev_alloc, dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>(
                                   (int64_t)ctx->n_cu * 2, gs_ceil_div(rows, 1024))), nbat), dim3(1024), 0, st, ra, 0, S);
        }
        GsTimeScope ts(ctx, "rev_fill", -1, st);
        hipLaunchKernelGGL(k_rev_fill, dim3(grid_for(ctx, items, nbat), nbat), dim3(256), 0, st, ra, 0, FanDiv::make(ctx->fan[0]), S);
    }
    GS_HIP(ctx, hipGetLastError());
    return ctx->captured || !ctx->own_done ? GSPLIT_OK : record_done(ctxs, nbat, st);
}

// ------------------------------------------------------------------------------------------
// The same step without any allocation: everything a context would own (tables, per-element entry
// indices, class codes, histograms, level bookkeeping) lives in one static device array, carved up
// per call.  Each GPU holds its own copy of the array at its own address, taken once per device.
// ------------------------------------------------------------------------------------------
constexpr size_t NOALLOC_SCRATCH_BYTES = (size_t)GSPLIT_NOALLOC_SCRATCH_MIB << 20;
constexpr int NOALLOC_MAX_DEVICES = 64;

static __device__ __align__(256) unsigned char scratch[NOALLOC_SCRATCH_BYTES];

struct NoAllocDevice { unsigned char *ptr = nullptr; int n_cu = 0; };
NoAllocDevice g_noalloc[NOALLOC_MAX_DEVICES];
std::mutex g_noalloc_mutex;

// device address of this GPU's copy of the array (and its compute-unit count), taken on the first
// call with that device current
int noalloc_device(NoAllocDevice **out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= NOALLOC_MAX_DEVICES)
        return gs_fail(nullptr, GSPLIT_EHIP, "gsplit_sample_split_noalloc: no current HIP device");
    std::lock_guard<std::mutex> lock(g_noalloc_mutex);
    NoAllocDevice &d = g_noalloc[dev];
    if (!d.ptr) {
        void *p = nullptr;
        hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return gs_fail(nullptr, GSPLIT_EHIP, std::string("gsplit_sample_split_noalloc: hipGetSymbolAddress: ") +
                                                     hipGetErrorString(e));
        int n_cu = 0;
        if (hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu <= 0) n_cu = 256;
        d.n_cu = n_cu;
        d.ptr = (unsigned char *)p;
    }
    *out = &d;
    return GSPLIT_OK;
}

// every table entry of the part a call can use starts empty, the level bookkeeping at zero (a fill
// kernel, not a memset: the call may be recorded into a graph)
__global__ __launch_bounds__(256) void k_noalloc_reset(GsTable a, int64_t n_entries, int32_t *meta_words, int n_meta_words) {
    for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < n_entries; x += (int64_t)gridDim.x * blockDim.x)
        a.slot[x] = EMPTY_ENTRY;
    if (blockIdx.x == 0)
        for (int x = threadIdx.x; x < n_meta_words; x += blockDim.x) meta_words[x] = 0;
}

// split offsets of every level and layer, from the internal bookkeeping to the caller's arrays
__global__ void k_noalloc_export(const GsLevelMeta *__restrict__ meta, int L, int S, int32_t *local_off,
                                 int32_t *mixed_off, int32_t *recv_off) {
    const int per = S + 1;
    for (int x = threadIdx.x; x < (L + 1) * per; x += blockDim.x) local_off[x] = meta[x / per].front_off[x % per];
    for (int x = threadIdx.x; x < L * per; x += blockDim.x) {
        mixed_off[x] = meta[x / per].mixed_off[x % per];
        recv_off[x] = meta[x / per].recv_off[x % per];
    }
}

}  // namespace

extern "C" int gsplit_sample_split_noalloc(const gsplit_graph *g, const gsplit_config *c, const int32_t *d_targets,
                                           int64_t n_targets, uint64_t seed, uint64_t iter,
                                           const gsplit_batch_out *out, void *stream) {
    const char *who = "gsplit_sample_split_noalloc: ";
    if (!g || !c || !out) return gs_fail(nullptr, GSPLIT_EINVAL, std::string(who) + "NULL argument");
    if (g->n_vertices <= 0 || g->n_vertices >= (1ll << 31) || g->n_edges < 0 || !g->d_indptr ||
        (g->n_edges > 0 && !g->d_indices) || !g->d_pmap || g->n_splits < 1 || g->n_splits > GSPLIT_MAX_SPLITS ||
        (unsigned long long)g->n_vertices * (unsigned long long)g->n_splits >= 0xFFFFFFFFull)
        return gs_fail(nullptr, GSPLIT_EINVAL, std::string(who) + "bad graph");
    if (c->n_layers < 1 || c->n_layers > GSPLIT_MAX_LAYERS || !c->fanouts || c->max_targets < 1 ||
        c->max_targets > g->n_vertices)
        return gs_fail(nullptr, GSPLIT_EINVAL, std::string(who) + "bad config");
    if (c->keep_edge_ids || c->gat_index)
        return gs_fail(nullptr, GSPLIT_EINVAL, std::string(who) + "keep_edge_ids and gat_index need a context");
    for (int l = 0; l < c->n_layers; ++l)
        if (c->fanouts[l] < 1 || c->fanouts[l] > GSPLIT_MAX_FANOUT)
            return gs_fail(nullptr, GSPLIT_EINVAL, std::string(who) + "fanout out of range");
    if (n_targets < 0 || (n_targets > 0 && !d_targets)) return gs_fail(nullptr, GSPLIT_EINVAL, std::string(who) + "bad targets");
    if (n_targets > c->max_targets) return gs_fail(nullptr, GSPLIT_ECAPACITY, std::string(who) + "n_targets exceeds max_targets");
    const int L = c->n_layers, S = g->n_splits;
    if (!out->d_local_off || !out->d_mixed_off || !out->d_recv_off)
        return gs_fail(nullptr, GSPLIT_EINVAL, std::string(who) + "NULL output");
    for (int l = 0; l <= L; ++l)
        if (!out->d_local_cat[l]) return gs_fail(nullptr, GSPLIT_EINVAL, std::string(who) + "NULL output");
    for (int l = 0; l < L; ++l)
        if (!out->d_nbr[l] || !out->d_cnt[l] || !out->d_mixed_cat[l] || !out->d_blk_indptr[l] || !out->d_blk_src[l] ||
            !out->d_shuffle_src_row[l] || !out->d_recv_cat[l])
            return gs_fail(nullptr, GSPLIT_EINVAL, std::string(who) + "NULL output");

    // a context on the host stack whose buffers are the caller's outputs and pieces of the static array
    gsplit_ctx ctx;
    ctx.graph = *g;
    ctx.L = L; ctx.S = S;
    ctx.max_targets = c->max_targets;
    ctx.sampler_blocks_per_cu = c->sampler_blocks_per_cu > 0 ? std::min(c->sampler_blocks_per_cu, 8) : 8;
    ctx.rev_from = L;                     // no scatter side: it serves the training passes of a context
    for (int l = 0; l < L; ++l) ctx.fan[l] = c->fanouts[l];
    ctx.ub_front[L] = c->max_targets;
    int64_t tab_cap = 1024, max_items = 1024;
    for (int l = L - 1; l >= 0; --l) {
        const int64_t grown = ctx.ub_front[l + 1] * (1 + ctx.fan[l]);
        max_items = std::max(max_items, grown);
        ctx.ub_front[l] = std::min<int64_t>(g->n_vertices, grown);
        while (tab_cap < 2 * grown) tab_cap <<= 1;
        if (grown >= (1ll << 29)) { max_items = 1ll << 40; break; }
    }
    ctx.tab_cap = tab_cap;
    size_t need = 0;
    auto carve = [&](size_t bytes) { const size_t at = need; need += (bytes + 255) & ~(size_t)255; return at; };
    const size_t o_meta = carve(sizeof(GsLevelMeta) * (L + 1));
    const size_t o_mslot = carve(sizeof(unsigned long long) * tab_cap), o_mrow = carve(sizeof(int32_t) * max_items);
    const size_t o_lrow = carve(sizeof(int32_t) * max_items);
    const size_t o_em = carve(sizeof(int32_t) * max_items), o_el = carve(sizeof(int32_t) * max_items);
    // (four bytes per class code, of which one is used: the documented capacity counts 32 bytes per element)
    const size_t o_me = carve(sizeof(int32_t) * max_items), o_cls = carve(sizeof(uint32_t) * max_items);
    const size_t o_self = carve(sizeof(int32_t) * max_items), o_edge = carve(sizeof(int32_t) * max_items);
    const size_t o_hist = carve(sizeof(int32_t) * PART_MAX_NB * PART_NK);
    const size_t o_perm = carve(sizeof(int32_t) * ctx.ub_front[L]);
    if (max_items >= (1ll << 29) || need > NOALLOC_SCRATCH_BYTES)
        return gs_fail(nullptr, GSPLIT_ECAPACITY,
                       std::string(who) + "max_targets and fanouts need " + std::to_string(need >> 10) +
                           " KiB of working memory, the static array holds " +
                           std::to_string(NOALLOC_SCRATCH_BYTES >> 10) + " KiB; use a context (gsplit_create)");
    NoAllocDevice *dev = nullptr;
    int rc = noalloc_device(&dev);
    if (rc != GSPLIT_OK) return rc;
    unsigned char *base = dev->ptr;       // this GPU's copy of the array (never the array's name on the host)
    ctx.n_cu = dev->n_cu;
    ctx.d_meta = (GsLevelMeta *)(base + o_meta);
    ctx.tab_mixed = GsTable{(unsigned long long *)(base + o_mslot), (int32_t *)(base + o_mrow), nullptr};
    ctx.row_local = (int32_t *)(base + o_lrow);
    ctx.ent_mixed = (int32_t *)(base + o_em); ctx.first_any = (int32_t *)(base + o_el);
    ctx.mixed_ent = (int32_t *)(base + o_me); ctx.cls = (uint8_t *)(base + o_cls);
    ctx.part_hist = (int32_t *)(base + o_hist);
    ctx.target_perm = (int32_t *)(base + o_perm);
    for (int l = 0; l <= L; ++l) ctx.front[l] = out->d_local_cat[l];
    for (int l = 0; l < L; ++l) {
        GsLayerBuf &B = ctx.layer[l];
        B.nbr = out->d_nbr[l]; B.cnt = out->d_cnt[l]; B.mixed = out->d_mixed_cat[l]; B.blk_indptr = out->d_blk_indptr[l];
        B.blk_src = out->d_blk_src[l]; B.recv = out->d_recv_cat[l]; B.src_row = out->d_shuffle_src_row[l];
        // the shuffle index composed with edges[l] is a by-product nobody reads here: one region for all layers
        B.self_row = (int32_t *)(base + o_self); B.edge_row = (int32_t *)(base + o_edge);
    }
    hipStream_t st = (hipStream_t)stream;
    // the array keeps what the last call left: clear the table entries this call can touch and the
    // level bookkeeping before the first kernel reads them
    hipLaunchKernelGGL(k_noalloc_reset, dim3((unsigned)std::min<int64_t>(1024, gs_ceil_div(tab_cap, 256))), dim3(256), 0, st,
                       ctx.tab_mixed, tab_cap, (int32_t *)ctx.d_meta,
                       (int)(sizeof(GsLevelMeta) * (L + 1) / sizeof(int32_t)));
    gsplit_ctx *one = &ctx;
    rc = sample_split(&one, 1, &d_targets, &n_targets, seed, &iter, nullptr, stream);
    if (rc != GSPLIT_OK) return gs_fail(nullptr, rc, std::string(who) + ctx.err);
    hipLaunchKernelGGL(k_noalloc_export, dim3(1), dim3(64), 0, st, ctx.d_meta, L, S, out->d_local_off, out->d_mixed_off,
                       out->d_recv_off);
    if (hipGetLastError() != hipSuccess) return gs_fail(nullptr, GSPLIT_EHIP, std::string(who) + "kernel launch failed");
    return GSPLIT_OK;
}

extern "C" int gsplit_sample_split(gsplit_ctx *ctx, const int32_t *d_targets, int64_t n_targets,
                                   uint64_t seed, uint64_t iter, void *stream) {
    if (!ctx) return GSPLIT_EINVAL;
    return sample_split(&ctx, 1, &d_targets, &n_targets, seed, &iter, nullptr, stream);
}

extern "C" int gsplit_sample_split_multi(gsplit_ctx *const *ctxs, int32_t n_batches, const int32_t *const *d_targets,
                                         const int64_t *n_targets, uint64_t seed, const uint64_t *iters, void *stream) {
    if (!ctxs || n_batches < 1 || !ctxs[0]) return GSPLIT_EINVAL;
    gsplit_ctx *first = ctxs[0];
    if (n_batches > GSPLIT_MAX_MULTI)
        return gs_fail(first, GSPLIT_ECAPACITY, "gsplit_sample_split_multi: more than GSPLIT_MAX_MULTI batches");
    if (!d_targets || !n_targets || !iters) return gs_fail(first, GSPLIT_EINVAL, "gsplit_sample_split_multi: NULL argument");
    for (int b = 0; b < n_batches; ++b) {
        const gsplit_ctx *c = ctxs[b];
        if (!c) return gs_fail(first, GSPLIT_EINVAL, "gsplit_sample_split_multi: NULL context");
        for (int a = 0; a < b; ++a)
            if (ctxs[a] == c) return gs_fail(first, GSPLIT_EINVAL, "gsplit_sample_split_multi: a context is listed twice");
        bool same = c->L == first->L && c->S == first->S && c->max_targets == first->max_targets &&
                    c->keep_edge_ids == first->keep_edge_ids && c->gat_index == first->gat_index &&
                    c->sampler_blocks_per_cu == first->sampler_blocks_per_cu && c->direct_tables == first->direct_tables &&
                    c->graph.d_indptr == first->graph.d_indptr && c->graph.d_indices == first->graph.d_indices &&
                    c->graph.d_pmap == first->graph.d_pmap && c->graph.n_vertices == first->graph.n_vertices &&
                    c->graph.indptr_is_64 == first->graph.indptr_is_64;
        for (int l = 0; same && l < first->L; ++l) same = c->fan[l] == first->fan[l];
        if (!same)
            return gs_fail(first, GSPLIT_EINVAL, "gsplit_sample_split_multi: the contexts differ in graph or configuration");
    }
    return sample_split(ctxs, n_batches, d_targets, n_targets, seed, iters, nullptr, stream);
}

extern "C" int gsplit_sample_split_dev(gsplit_ctx *ctx, const int32_t *d_targets, int64_t n_targets,
                                       const uint64_t *d_seed_iter, void *stream) {
    if (!ctx) return GSPLIT_EINVAL;
    if (!d_seed_iter) return gs_fail(ctx, GSPLIT_EINVAL, "gsplit_sample_split_dev: NULL seed / iteration buffer");
    const uint64_t zero = 0;
    return sample_split(&ctx, 1, &d_targets, &n_targets, 0, &zero, d_seed_iter, stream);
}
