// Which of the two copies of a matrix a GEMM of few token rows reads: the rows as they lie (the kernels for few rows) or the packed order (the
// kernels that stream weights into registers).  Host arithmetic on sizes and nothing else, so that the rules can be read and tested on their own.
#pragma once

namespace samp {

// From this many padded token rows on the LayerNorm steps ask for the weights that come next (api.hip), so that a GEMM finds them in the
// memory-side cache; below, a GEMM waits for memory beyond it.
constexpr int FETCH_AHEAD_MIN_ROWS = 256;

// FP16: the rows as they lie while the 32 x 32 tiles of gemm_nt_small_f16_kernel are all on the chip at once, two to a CU, and one to a CU where the
// weights have been fetched ahead.  The packed kernel's narrowest tile is 128 channels wide: 32 rows of 1024 x 4096 are 8 blocks of it, 32 of the small
// one, and what bounds such a GEMM is how many CUs ask for its weights.  Us per launch, rows as they lie / packed, weights from memory:
// 2304 x 768 at 19 rows 5.70 / 6.63, 96 5.72 / 6.65, 224 6.43 / 6.60, 240 (no longer two to a CU) 8.63 / 6.47; 4096 x 1024 at 19 rows 6.62 / 7.93, 64
// 6.78 / 8.08, 128 7.70 / 7.97, 144 10.20 / 7.83; 768 x 3072 at 19 rows 13.3 / 18.1, 255 13.3 / 18.0; 1024 x 4096 at 32 rows 16.4 / 24.4, 255
// 16.5 / 22.8; 2048 x 8192 at 19 rows 29.8 / 46.0.  Weights in the memory-side cache: 768 x 3072 at 256 rows 11.45 / 12.21, 320 (240 tiles) 11.68 / 12.55,
// 384 12.92 / 12.41; 1024 x 4096 at 256 rows 14.66 / 15.50, 320 16.01 / 15.63; 768 x 768 at 320 rows 4.90 / 5.09, 384 5.25 / 5.08.  (Below 256 rows the wide
// matrices are faster packed when a single model keeps its weights cached: 2304 x 768 at 19 rows 5.04 / 4.87, 192 5.66 / 5.13.)  Forward of
// BERT-large FP16, one sequence, all packed / one to a CU / two to a CU below 256 rows: 19 tokens 1404 / 1178 / 1178, 96 tokens - / 1267 / 1234, 144
// 1442 / 1268 / 1257; from 256 rows on two to a CU loses: 512 tokens 1386 / 1386 / 1407.
// K that is no multiple of 256 has no small kernel: 384 x 384 at 128 rows 4.82 / 3.99, 640 x 640 10.5 / 6.2.
inline long f16_small_tiles(long rows, int N) { return (rows + 31) / 32 * (N / 32); }
inline bool f16_reads_rows(long rows, int N, int K, long cus)
{
    return K % 256 == 0 && f16_small_tiles(rows, N) <= (rows < FETCH_AHEAD_MIN_ROWS ? 2 : 1) * cus;
}

}  // namespace samp
