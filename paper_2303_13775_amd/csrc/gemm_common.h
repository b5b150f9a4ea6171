// Pieces shared by the matrix products of the GraphSAGE and GAT translation units (included inside their
// anonymous namespaces): the bfloat16 conversions, the plain row-major operand accessor, the tiling of
// persistent row-block products and the split-K geometry of the weight gradients.
#pragma once

typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int BK = 32;                  // k granularity of a split-K chunk
constexpr int GNT = 512;                // threads of a workgroup of the bf16 products
struct TileMid { static constexpr int BM = 64, BN = 128, OCC = 2; };     // their tile; workgroups a compute unit holds

__device__ __forceinline__ uint16_t f2bf(float f) {          // round to nearest, ties to even
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint32_t h) { return __uint_as_float(h << 16); }

// Accessors return an address that is always safe to read VW floats from (indices are clamped into
// the matrix; matrices have at least one row and VW columns) and say whether the element exists.
// plain row-major matrix
struct MatRows {
    const float *p; int rows; int cols;
    template <int VW>
    __device__ __forceinline__ const float *at(int o, int i, bool &in) const {
        in = o < rows && i < cols;
        const int oc = min(o, rows - 1), ic = min(i, cols - VW);
        return p + (int64_t)oc * cols + ic;
    }
    // K-major use, 16-byte pieces: tok() clamps the M/N index once, km() addresses row k < rows
    __device__ __forceinline__ int tok(int i) const { return min(i, cols - 4); }
    __device__ __forceinline__ const float *km(int k, int t) const { return p + (int64_t)k * cols + t; }
};
// partial [dW_self; dW_neigh; db] of one chunk of destination rows, written to the chunk's slab
// (rows = 2 * D + 1: the last one holds the bias gradient)
struct EpiGradW {
    float *part; int rows; int N;
    __device__ __forceinline__ float col(int) const { return 0.f; }
    __device__ __forceinline__ float row(int) const { return 0.f; }
    __device__ __forceinline__ void store(int c, int n, float v, float, float) const {
        if (n < N && c < rows) part[(int64_t)c * N + n] = v;
    }
};
// Row-block products run as persistent workgroups: the launch has at most as many workgroups as the
// chip holds at once (the host only knows an upper bound on the rows; workgroups without a tile
// would otherwise queue behind the working ones and drain after them) and each walks the tiles
// gid = blockIdx.x, + gridDim.x, ...  The id is decoded so that the column tiles of one row block
// run on the same XCD (workgroups are dealt round-robin to the 8 XCDs) and share its L2.
template <class T>
__device__ __forceinline__ bool next_tile(int gid, int tiles_m, int tiles_n, int &m0, int &n0) {
    const int xcd = gid & 7, j = gid >> 3;
    const int tm = (j / tiles_n) * 8 + xcd;
    m0 = tm * T::BM; n0 = (j % tiles_n) * T::BN;
    return tm < tiles_m;
}

// Split-K geometry of the weight-gradient product, decided on the device from the actual number
// of destination rows n1: as many chunks (nchunk, or a smaller multiple of 8) as keep rows_min rows
// in each, every chunk a multiple of the k-tile.
__device__ __forceinline__ int grad_w_chunk_rows(int n1, int nchunk, int rows_min) {
    const int want = min(nchunk, max(8, ((n1 + rows_min - 1) / rows_min + 7) & ~7));
    const int per = (n1 + want - 1) / want;
    return max(BK, (per + BK - 1) & ~(BK - 1));
}

constexpr int GRAD_W_ROWS_MIN = 256;

// Sum of the per-chunk slabs of partials, in a fixed order: a workgroup of 256 threads takes 64 words at a time, its
// four waves a quarter of the slabs each, sixteen loads in flight, added as trees (fewer roundings than in a row).
// (One thread per word left the loads of 128 slabs in eight rounds one after the other: 11.4 us for the 45 MB of a
// training step of the medium workload.)
template <class Store>
__device__ __forceinline__ void sum_slabs(const float *__restrict__ part, int64_t words, int64_t slab, int chunks, const Store &store) {
    __shared__ float s_sum[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int per = (chunks + 3) / 4, z1 = min(chunks, (wave + 1) * per);
    for (int64_t base = blockIdx.x * (int64_t)64; base < words; base += gridDim.x * (int64_t)64) {
        const int64_t x = base + lane;
        const float *p = part + (x < words ? x : words - 1);
        float acc = 0.f;
        int z = wave * per;
        for (; z + 16 <= z1; z += 16) {
            float v[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) v[j] = p[(z + j) * slab];
#pragma unroll
            for (int d = 8; d > 0; d >>= 1)
#pragma unroll
                for (int j = 0; j < d; ++j) v[j] += v[j + d];
            acc += v[0];
        }
        for (; z + 4 <= z1; z += 4) {
            const float v0 = p[z * slab], v1 = p[(z + 1) * slab], v2 = p[(z + 2) * slab], v3 = p[(z + 3) * slab];
            acc += (v0 + v2) + (v1 + v3);
        }
        for (; z < z1; ++z) acc += p[z * slab];
        s_sum[wave][lane] = acc;
        __syncthreads();
        if (wave == 0 && x < words) store(x, (s_sum[0][lane] + s_sum[1][lane]) + (s_sum[2][lane] + s_sum[3][lane]));
        __syncthreads();
    }
}
inline unsigned sum_slabs_grid(int64_t words) { return (unsigned)std::min<int64_t>(2048, gs_ceil_div(words, 64)); }

// persistent launch: no more workgroups than the chip holds, a multiple of 8
template <class T>
unsigned row_block_grid(const gsplit_ctx *ctx, int64_t ub, int n_out) {
    const int64_t want = gs_ceil_div(gs_ceil_div(ub, T::BM), 8) * 8 * gs_ceil_div(n_out, T::BN);
    return (unsigned)std::min<int64_t>(want, (int64_t)ctx->n_cu * T::OCC / 8 * 8);
}
