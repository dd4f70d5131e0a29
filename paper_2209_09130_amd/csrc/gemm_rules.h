// Which of the two copies of a matrix a GEMM of few token rows reads: the rows as they lie (the kernels for few rows) or the packed order (the
// kernels that stream weights into registers).  And which kernels ask for the weights that come next,
// and the tiles of the INT8 GEMMs on packed weights.  Host arithmetic on sizes and nothing else, so that the rules can be read and tested on their
// own.
#pragma once

namespace samp {

// From this many padded token rows on the LayerNorm steps ask for the weights that come next where the attention kernels do not (api.hip), so that a
// GEMM finds them in the memory-side cache.  (Below, only attention kernels ask; the figures here are of GEMMs that wait for memory.)
constexpr int FETCH_AHEAD_MIN_ROWS = 256;

// The kernels of QKV GEMM and attention in one on packed weights, which exist with blocks that ask; those on rows as they lie exist without.
inline bool qkv_attention_packed(bool i8, bool has_packed, int max_len, int H) { return has_packed && max_len <= 128 && H % (i8 ? 256 : 128) == 0; }

// Of a layer: its attention asks for attention output, FFN1, FFN2 and the next layer's QKV; or its LayerNorm steps ask, the first for FFN1 and FFN2, the
// second for the next layer's QKV and attention output, each for what no attention kernel does.  attention_may, norm_may: whether they do so at all in
// this forward; here_can, next_can: whether the attention kernels of this layer and the next exist with blocks that ask.  Forward, us, three encoders in
// turn, nobody asks / the LayerNorm steps do, where the attention cannot: 12 Fully-Quant layers of width 896, 10 x 128 tokens 819 / 754, 17 x 100 with
// FP16 FFN 1037 / 939; with the weights in the memory-side cache anyway, width 640 13 x 128 607 / 610, width 384 24 x 64 392 / 395, 32 x 128 502 / 508.
struct Asks { bool attention, norm1, norm2_qkv, norm2_out; };
inline Asks who_asks(bool attention_may, bool norm_may, bool here_can, bool next_can)
{
    const bool here = attention_may && here_can, next = attention_may && next_can;
    return {here, norm_may && !here, norm_may && !here, norm_may && !next};
}

// FP16: the rows as they lie while the 32 x 32 tiles of gemm_nt_small_f16_kernel are all on the chip at once.  The packed kernel's narrowest tile is
// 128 channels wide: 32 rows of 1024 x 4096 are 8 blocks of it, 32 of the small one, and what bounds such a GEMM is how many CUs ask for its weights.
// One small tile per CU is always worth it, two where the weights come from memory and the packed kernel waits longest for them: up to 96 rows (of
// its 64 x 128 tiles, at most two in a column), and with the longer chain of loads of K from 1024 on (models of that width do not fit the memory-side
// cache).  Us per launch, rows as they lie / packed, weights from memory: 2304 x 768 at 19 rows 5.70 / 6.63, 96 5.72 / 6.65, 128 (288 small tiles)
// 6.53 / 6.59, 240 (576) 8.63 / 6.47; 3072 x 768 at 96 rows (288) 6.20 / 6.71, 97 (384) 6.19 / 6.34; 3072 x 1024 at 96 rows (288) 7.08 / 7.93, 160 (480)
// 7.34 / 7.93, 192 (576) 10.22 / 7.95; 4096 x 1024 at 19 rows 6.62 / 7.93, 96 (384) 7.38 / 8.00, 128 (512) 7.70 / 7.97, 144 (640) 10.20 / 7.83; 768 x 3072
// at 19 rows 13.3 / 18.1, 255 13.3 / 18.0; 1024 x 4096 at 32 rows 16.4 / 24.4, 255 16.5 / 22.8; 2048 x 8192 at 19 rows 29.8 / 46.0, 255 (512) 35 / 46.
// Weights in the memory-side cache: 2304 x 768 at 19 rows 5.04 / 4.87, 96 5.18 / 5.01, 128 5.62 / 5.08, 192 (432) 5.66 / 5.13; 768 x 3072 at 256 rows
// 11.45 / 12.21, 320 (240) 11.68 / 12.55, 384 (288) 12.92 / 12.41; 1024 x 4096 at 256 rows 14.66 / 15.50, 320 (320) 16.01 / 15.63; 768 x 768 at 320 rows 4.90 / 5.09,
// 384 5.25 / 5.08.  Forward, one sequence, all packed / one tile per CU / two below 256 rows: BERT-large FP16 19 tokens 1408 / 1178 / 1176, 96
// tokens - / 1267 / 1234, 144 1442 / 1268 / 1257, 512 (two there as well) 1386 / 1386 / 1407; BERT-base FP16 96 tokens - / 540 / 538, 128 609 / 552 / 557, and
// with its weights in the memory-side cache 128 474 / 462 / 472, 192 - / 478 / 499; one layer of 128 rows, Quant-FFN-Only, 33.4 / 33.4 / 33.9.
// K that is no multiple of 256 has no small kernel: 384 x 384 at 128 rows 4.82 / 3.99, 640 x 640 10.5 / 6.2.
inline long f16_small_tiles(long rows, int N) { return (rows + 31) / 32 * (N / 32); }
inline bool f16_reads_rows(long rows, int N, int K, long cus)
{
    const bool from_memory = rows <= 96 || (rows < FETCH_AHEAD_MIN_ROWS && K >= 1024);
    return K % 256 == 0 && f16_small_tiles(rows, N) <= (from_memory ? 2 : 1) * cus;
}

// INT8: the rows as they lie where the kernel that splits K over a block's waves (gemm_nt_small_kernel) is the faster one: it asks for the whole of K at once
// and has tiles of 16 channels.  It exists for K of whole slabs of eight or of six waves (128 bytes each) and for no other: those are always faster
// packed than on what is left for them (us, 19 rows: 512 x 512 5.07 / 2.95, 1024 x 512 5.24 / 3.03, 640 x 2560 13.2 / 4.8, 1280 x 1280 11.0 / 6.0).
// Us per launch, K split / packed weights, at most 1024 channels: 768 x 768 at 128 rows 3.05 / 3.29, 255 3.50 / 3.36, 400 3.89 / 3.41; 768 x 3072 at 128 rows
// 5.43 / 7.27, 320 5.15 / 6.33, 400 6.13 / 6.32; 1024 x 1024 at 255 rows 4.20 / 5.06, 448 4.33 / 4.64; 1024 x 4096 at 128 rows 6.03 / 8.52, 256 5.91 / 6.36, 320
// 7.15 / 6.38.  Up to 2048 channels, long K: 1280 x 5120 at 128 rows 8.6 / 10.5, 192 8.4 / 10.4, 256 11.0 / 10.4; 1536 x 6144 at 160 rows 9.5 / 11.8, 192
// 12.4 / 11.8; 2048 x 8192 at 64 rows 9.6 / 15.5, 160 13.3 / 15.2, 192 15.0 / 15.2; K no longer than N: 2048 x 2048 at 128 rows 5.47 / 5.71, 160
// 6.05 / 5.65; 1536 x 1536 at 64 rows 4.39 / 5.13, 128 5.27 / 5.20, 192 5.94 / 5.35.  Wider: 2304 x 768 at 32 rows 3.55 / 4.20, 40 4.05 / 3.91; 3072 x 768
// at 32 rows 3.61 / 4.23, 40 4.08 / 3.90; 4096 x 1024 at 32 rows 4.00 / 4.47, 40 4.37 / 4.34; 6144 x 2048 at 32 rows 6.07 / 6.19, 64 7.09 / 6.17.
// (from 256 rows weights in the memory-side cache, below from memory)
inline int i8_small_waves(int K) { return K % 1024 == 0 ? 8 : K % 768 == 0 ? 6 : 0; }
inline bool i8_reads_rows(long rows, int N, int K)
{
    return i8_small_waves(K) && rows * N <= (N <= 1024 ? 300000 : N > 2048 ? 128000 : K > N ? 330000 : 262144);
}

// INT8 GEMMs on packed weights (gemm_nt_stream_kernel): the tile is the one whose estimated time is least.  The estimate, in us, is a fit to the times of these tiles at 16 to 16384 rows of eight
// N x K from 768 x 768 to 4096 x 1024 (each alone on the chip, in chains over other weights at every launch, as in a forward; the choice
// costs 1 % on average over the best of all tiles and depths): per 128-byte stage of K the products and the operand bytes of the blocks
// that the busiest CU gets, and their epilogues.  Beside another batch group all CUs count as well: larger tiles for half of them lose (forward, us, all /
// half: BERT-base 32 x 128 Fully-Quant 756 / 795, FP16 1144 / 1345, 6 x 500..1100 1695 / 1829, 33 x 40..301 1436 / 1418).  Smallest first.
struct StreamShape { int mt, ntw; };
constexpr StreamShape STREAM_TILES[] = {{2, 1}, {4, 1}, {4, 2}, {4, 3}, {4, 4}, {8, 2}, {8, 3}};
constexpr int STREAM_TILE_COUNT = sizeof(STREAM_TILES) / sizeof(STREAM_TILES[0]);
// with as many rows as the host counts, or `percent` of them
inline double stream_cost(StreamShape tile, long rows, int percent, int N, int K)
{
    const int bm = 16 * tile.mt, bn = 64 * tile.ntw;
    const double area = bm * bn / 8192.0, sides = (bm + bn) / 256.0;
    const long tiles = (long)(N / bn) * ((rows * percent / 100 + bm - 1) / bm);
    return (double)((tiles + 255) / 256) * (K / 128 * (0.016 * area + 0.30 * sides) + 0.81 * area);
}
// fewer: a batch with a mask, of whose rows only the device knows how many there are.  Lengths spread evenly up to the longest make 50 to 100 % of them, and a
// mask may also leave out nothing, so the full batch counts as much as 55, 70 and 85 % together: a tile that suits fewer rows is taken where it saves them
// more than it costs a full batch.  Forward, us, three encoders in turn, at 100, 90, 75 and 55 % of the rows, tiles for all rows / for the plain average of 55
// to 100 % / these: BERT-base Fully-Quant 12 x 128 517, 517, 513, 501 / 518, 513, 476, 464 / 520, 519, 479, 469; 7 x 61 358, 356, 348, 342 / 358, 357, 333, 325 /
// 352, 351, 329, 323; 40 x 48 529, 522, 516, 505 / 558, 534, 523, 462 / 529, 523, 515, 495; 9 x 200 558, 550, 539, 519 / 588, 558, 530, 477 / 560, 550,
// 538, 512; 24 x 100 612, 593, 564, 536 / 634, 615, 555, 537 / 612, 593, 564, 536; 8 x 256 575, 564, 552, 541 / 581, 573, 539, 528 / 574, 564, 552, 539;
// BERT-large 7 x 200 1380, 1349, 1317, 1213 / 1438, 1367, 1322, 1072 / 1369, 1339, 1308, 1190; 6 x 256 1433, 1380, 1354, 1227 / 1384, 1371, 1339,
// 1205 / 1435, 1383, 1356, 1228.  Beside another batch group the larger tiles that padded rows ask for are the better ones (64 x 16..128 846 / 908, 33 x
// 40..301 1078 / 1109), and the FP16 tiles come out the same.
inline int stream_tile(long rows, bool fewer, int N, int K)
{
    int best = -1;
    double best_cost = 0.0;
    for (int i = 0; i < STREAM_TILE_COUNT; i++) {
        if (N % (64 * STREAM_TILES[i].ntw)) continue;
        double cost = (fewer ? 3 : 1) * stream_cost(STREAM_TILES[i], rows, 100, N, K);
        for (int percent = 55; fewer && percent < 100; percent += 15) cost += stream_cost(STREAM_TILES[i], rows, percent, N, K);
        if (best < 0 || cost < best_cost) { best = i; best_cost = cost; }
    }
    return best;
}

}  // namespace samp
