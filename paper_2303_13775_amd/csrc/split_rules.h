// Which form a split product takes: rules on sizes alone, shared by the launches, the kernels and their tests (included by
// gemm_split.h; a host program defines __host__ and __device__ away).
//
// Products of rows (rows x K x N; the products of a launch, its heads, count together), in us (wide tiles of 64 x 128 /
// narrow tiles of 64 x 64 / few rows, 32 x 32):
//   up to one few-rows workgroup per compute unit the few-rows form: 800 x 64 x 256 5.5 / 4.2 / 3.7, 800 x 512 x 256
//   14.0 / 9.5 / 5.7, 1500 x 100 x 132 6.4 / 4.6 / 4.1; up to two with a long contraction: 1100 x 512 x 256 14.0 / 9.6 / 8.9,
//   1100 x 256 x 256 9.1 / 6.4 / 6.5, 1100 x 128 x 256 6.7 / 4.9 / 6.5;
//   then narrow tiles while the chip holds all of them at once, three per compute unit: 2600 x 512 x 256 14.4 / 10.1 / 12.9,
//   3300 x 256 x 512 10.3 / 9.8 / 18.6, 11000 x 200 x 256 13.1 / 11.4, 16000 x 200 x 256 14.5 / 16.3; and whatever the rows
//   where they cover the columns with less padding: 24000 x 512 x 172 38.5 / 35.8, 24000 x 100 x 132 12.3 / 11.5.
//   Rows read float by float (`pieces` false: not whole 16-byte pieces) cost a narrow tile nearly what they cost a wide one:
//   there one narrow tile per compute unit is the bar, and padding does not move it: 3300 x 254 x 256 12.2 / 10.4, 6000 x
//   254 x 256 12.8 / 16.0, 11000 x 254 x 256 18.8 / 22.7, 11000 x 202 x 100 12.0 / 15.7, 8000 x 70 x 260 10.8 / 13.0.
#pragma once

enum : int { FORM_FEW = 1, FORM_NARROW = 2, FORM_WIDE = 4 };

__host__ __device__ inline bool split_few(int64_t rows, int N, int K, int heads) {
    return ((rows + 31) / 32) * ((N + 31) / 32) * heads <= (K > 256 ? 512 : 256);
}
__host__ __device__ inline bool split_narrow(int64_t rows, int N, int heads, bool pieces, int n_cu) {
    if (N <= 64) return true;
    const int64_t tiles = ((rows + 63) / 64) * ((N + 63) / 64) * heads;
    return pieces ? tiles <= 3 * n_cu || ((N - 1) & 127) < 64 : tiles <= n_cu;
}

// The host knows a bound on the rows only, twice to three times their number in the lower layers, their number in the
// top one.  A kernel holds the forms that the rows may call for between a quarter of the bound (half of it for the
// few-rows form) and the bound: one that holds more is slower in each (a kernel of all forms: 4 % in the wide tiles).
inline int split_forms(int64_t ub, int N, int K, int heads, bool pieces, int n_cu) {
    return (split_few(ub / 2, N, K, heads) ? FORM_FEW : 0) | (split_narrow(ub / 4, N, heads, pieces, n_cu) ? FORM_NARROW : 0) |
           (split_narrow(ub, N, heads, pieces, n_cu) ? 0 : FORM_WIDE);
}
// the form a kernel that holds `forms` takes for the rows of the batch
__host__ __device__ inline int split_form(int forms, int64_t rows, int N, int K, int heads, bool pieces, int n_cu) {
    if ((forms & FORM_FEW) && split_few(rows, N, K, heads)) return FORM_FEW;
    if ((forms & FORM_NARROW) && (!(forms & FORM_WIDE) || split_narrow(rows, N, heads, pieces, n_cu))) return FORM_NARROW;
    return FORM_WIDE;
}

// Weight gradients (M x N, summed over rows).  Blocks of 128 for levels with enough rows (half their bound) to give every
// team of waves 96 of them, two teams a compute unit; blocks of 64 below that and where an operand is at most 64 wide.  In us with the
// reduction (64 / 128), at a quarter of the bar, at half, at three quarters, at the bar and at twice its rows:
//   512 x 256 16.1 / 17.5, 23.2 / 21.9, 24.2 / 23.3, 26.8 / 23.5, 38.1 / 28.5;  256 x 256 14.8 / 16.6, 20.9 / 19.7, 24.5 / 22.5,
//   25.4 / 21.2, 37.8 / 28.7;  1204 x 256 17.6 / 17.8, 22.4 / 21.7, 25.3 / 23.9, 28.2 / 25.0, 42.0 / 30.0.
// (From half the bar on blocks of 128 are ahead where the gradients are a launch of their own; above the bottom layer most such
// levels' go, as blocks of 64, with the pull of the input gradients.)
// Rows of a chunk at least (256 instead: 24k x 200 x 256 32 against 27 us, 3500 x 512 x 256 19 against 15).
constexpr int SGW_ROWS_MIN = 96;
inline int split_grad_block(int64_t ub_rows, int M, int N) {
    return M > 64 && N > 64 && (int64_t)((M + 127) / 128) * ((N + 127) / 128) * (ub_rows / 2 / SGW_ROWS_MIN) >= 512 ? 128 : 64;
}

// Chunks of rows of the weight gradients (of all `heads` of a launch): as many as give every workgroup a place at once, one a
// compute unit for blocks of 128 and, in eights, four for blocks of 64.  Blocks of 128 rounded down to eights as well left
// 96 and 112 of 256 compute units without one at 20 and 18 blocks, and a second round of workgroups in their place costs its
// first rows and the trade of the sums once more (22k x 1204 x 256: 8 chunks 93 us, 24 in two rounds 79, 12 76.5; 22k x 768 x
// 384: 8 93, 24 76, 14 70.7; 22k x 768 x 256: 16 52.6, 40 in two rounds 53.7, 21 49).  More than a quarter of the chip a chunk: eight chunks,
// in as many rounds as it takes.
inline int split_grad_chunks(int64_t ub_rows, int M, int N, int heads, int n_cu) {
    const int B = split_grad_block(ub_rows, M, N);
    const int tiles = ((M + B - 1) / B) * ((N + B - 1) / B) * heads;
    if (B == 128) return 4 * tiles <= n_cu ? n_cu / tiles : 8;
    return 4 * n_cu / tiles >= 8 ? 4 * n_cu / tiles / 8 * 8 : 8;
}
