// Which kernel a projection of more than 16 rows goes to, and which tile it takes there: rules on M rows, N columns and K alone.
// Plain C++ (no HIP types): launch_gemm asks them, the layer's workspace is sized by them, and tests/tile_rules_audit.cpp asks
// them on the host, so that a test that names a tile can be held to it.
#pragma once

#include <cstddef>
#include <cstdint>

namespace eet {

constexpr int kGemmCutMaxM = 1024;            // rows of the largest projection that is cut along K
constexpr int kFinishRowsMaxWidth = 16384;    // columns of the widest one: finish_rows holds a row in registers

// ---- 17 to 1024 rows: a weight stream through the tile kernel ----
// A decode step of 17 to 128 sequences (or as short a prompt) reads every weight once, and what bounds it is how fast the
// weights come in.  The general tile choice below makes that slow in two ways: a narrow output with a long K has only N/64
// workgroups (48 x 4096 x 16384: 64 of them, 71 us, 1.9 TB/s), and 128-row tiles pull twice the activations through L2 that
// 33 to 64 rows need.  Here one row tile of 32, 64 or 128 rows covers all rows, the columns come in tiles of 64, four waves
// of a workgroup (two or four K groups) keep two K steps each in flight, and a bias + residual projection whose columns leave
// CUs idle has K cut into 2 to 8 ranges, whose fp32 sums finish_rows adds up.  Measured on cold weights, before -> now, us
// (cut ones with finish_rows): 48 rows: 4096 x 16384 70.8 -> 29.0, 4096 x 4096 21.0 -> 13.2 (and the LayerNorm launch behind it
// gone), 12288 x 4096 27.9 -> 23.9, 16384 x 4096 32.8 -> 25.1, 49152 x 12288 251 -> 212, 12288 x 49152 280 -> 248, 8192 x
// 32768 166 -> 102; 24 rows: 16384 x 4096 32.4 -> 23.4; 128 rows: 4096 x 16384 73.5 -> 36.2, 36864 x 12288 267 -> 235.
// More rows (129 to 1024) take it only for the cut, and with the plain K walk and plain loads, since several row tiles then
// share the weights: 200 x 2048 x 8192 33.8 -> 20.6, 512 x 2048 x 8192 47.5 -> 32.4, 512 x 1024 x 4096 19.5 -> 16.7.
constexpr int kRowsStreamMaxM = 128;
inline int rows_tile(int M) { return M <= 32 ? 32 : M <= 64 ? 64 : 128; }
// K ranges that fill the CUs without a second round, up to 8; at least 512 columns each (below that a range is all start-up: 32 x
// 1024 x 1024 gains nothing in two).
inline int rows_ranges(int M, int N, int K) {
    const int tiles = (M + rows_tile(M) - 1) / rows_tile(M) * ((N + 63) / 64);
    int s = 256 / tiles;
    s = s < K / 512 ? s : K / 512;
    return s < 1 ? 1 : s > 8 ? 8 : s;
}
// Weights below 18 MB (24 MB for at most 32 rows) stay with the row slices (48 x 2048 x 2048 7.9 us in slices, 9.1 here; 17 x 1536 x
// 6144 8.6 and 10.5; but 48 x 1536 x 6144 13.3 and 11.2, 64 x 3072 x 3072 17.9 and 11.9).  At most 32 rows want no cut in eight
// (32 x 2048 x 8192 11.7 against 13.4), more than 64 rows without a cut a long K (96 x 6144 x 2048 12.1 against 16.0).  These floors
// are measured on calls that the slices can take, a decode step's and the operators' (prompts: prompt_k_ranges).
inline bool rows_stream_pays(int M, int N, int K, int ranges) {
    if (M <= 16 || K % 128 != 0 || N % 64 != 0) return false;
    // a cut that still leaves half of the CUs idle: 20 to 31 x 1984 x 7936 in two ranges (62 workgroups) took half again as long as the slices
    if (ranges > 1 && (M + rows_tile(M) - 1) / rows_tile(M) * ((N + 63) / 64) * ranges < 128) return false;
    const int64_t weights = (int64_t)N * K;
    if (M > kRowsStreamMaxM) return M <= kGemmCutMaxM && ranges > 1 && K >= 4096 && weights >= ((int64_t)4 << 20);
    if (weights < ((int64_t)(M <= 32 ? 12 : 9) << 20)) return false;
    if (M <= 32 && ranges >= 8) return false;
    return ranges > 1 || K >= (M <= 64 ? 2048 : 4096);
}
inline int gemm_k_ranges(int M, int N, int K) {
    const int s = N <= kFinishRowsMaxWidth ? rows_ranges(M, N, K) : 1;
    return s > 1 && rows_stream_pays(M, N, K, s) ? s : 1;
}
// A prompt's output and second feed-forward projection carry row maps, so the row slices cannot take them: with up to 256 rows and weights
// below the floors above they ran on N/64 or 2N/64 workgroups through the whole K (37 x 1024 x 4096: 16 of them, 15 us).  The cut
// pays there for much smaller weights, with ranges of 256 columns up to 64 rows, and it takes the LayerNorm launch behind the output
// projection along.  us per layer of a prompt, before -> now (stacks of 8): hidden 768, 20 rows 44 -> 36, 64 47 -> 39, 128 50 ->
// 47, 250 51 -> 47; 1024, 37 rows 50 -> 40, 100 53 -> 47; 1536, 20 rows 69 -> 48, 64 61 -> 55; 2048, 20 rows 81 -> 56, 64 72 -> 63, 250
// 88 -> 84; one layer of 1280 x 5120, 64 rows 63 -> 49.  Where it stops: 20 to 64 rows of hidden 256 (a quarter of a million weights: 32 -> 34);
// 65 to 128 of 640 x 1664 (one million: 44.2 -> 45.3); 160 of hidden 1024 (output projection, one million: 47 -> 48.5); 400 and 700 rows
// (1024 54 -> 55, 63 -> 66; 768 and 2048 gain 4 % at 400 and nothing at 700).
// (Most prompts of layers of up to 1024 x 4096 are one launch by now, prompt_step.hip, which asks nothing here; their layers' capacity does.)
inline int prompt_k_ranges(int M, int N, int K) {
    if (M > 16 && M <= 256 && K % 128 == 0 && N % 64 == 0 && N <= kFinishRowsMaxWidth && (int64_t)N * K >= (M <= 64 ? (int64_t)1 << 19 : (int64_t)2 << 20)) {
        const int tiles = (M + rows_tile(M) - 1) / rows_tile(M) * ((N + 63) / 64), least = M <= 64 ? 256 : 512;
        int s = 256 / tiles;
        s = s < K / least ? s : K / least;
        if (s > 1) return s > 8 ? 8 : s;
    }
    return gemm_k_ranges(M, N, K);
}
// The largest fp32 sums, in bytes, that a cut N x K projection of up to max_rows rows leaves (0: never cut).  The number of ranges
// depends on the row tiles alone, so the most rows of each number of them are all there is to ask (a walk over every row
// count made the creation of a layer handle take 17 us instead of 1, and a stack does it for every layer).
inline int64_t gemm_cut_bytes(int M, int N, int K) {
    const int p = prompt_k_ranges(M, N, K), ranges = p > 1 ? p : gemm_k_ranges(M, N, K);
    return ranges > 1 ? (int64_t)ranges * M * N * (int64_t)sizeof(float) : 0;
}
inline int64_t gemm_cut_bytes_up_to(int64_t max_rows, int N, int K) {
    int64_t most = 0;
    for (int m = 32; ; m = m < 128 ? 2 * m : m + 128) {
        const int64_t b = gemm_cut_bytes((int)(m < max_rows ? m : max_rows), N, K);
        if (b > most) most = b;
        if (m >= max_rows || m >= kGemmCutMaxM) return most;
    }
}
// Without the cut (outputs other than bias + residual, and callers without room for the sums), by column tiles.  us, the kernels
// below / as a stream, on weights out of HBM with the non-temporal hint (read_once); then the same on weights that the
// memory-side cache holds, with plain loads:
//   at most 32 rows: a narrow output stays where it was (17 x 6144 x 2048, 96 tiles: 11.5 / 10.0; 32 x 4096 x 4096 no better);
//   33 to 64 rows: 33 x 7168 x 4096, 112 tiles 21.7 / 23.0; 64 x 8192 x 4096, 128 tiles 26.0 / 24.2, 20.9 / 18.9; x 16384, 256 tiles 34.4 / 26.7,
//     23.4 / 22.3; x 20480, 320 tiles 52.5 / 47.1, 33.5 / 37.6; x 32768, 512 tiles 68.4 / 53.9; 64 x 36864 x 2048 48.1 / 41.3, 29.9 / 33.6;
//   65 to 128 rows are more arithmetic than the four waves of a workgroup hide behind the loads: cached weights never take it (100
//     x 8192 x 4096 21.0 / 28.5, x 16384 24.5 / 29.1), others where the CUs are full: 100 x 7168 x 4096, 112 tiles 22.1 / 29.6; x 8192
//     28.8 / 28.9; x 10240 31.5 / 29.8; 128 x 16384 x 4096 41.9 / 34.9; 100 x 20480 x 8192 110 / 108; with fewer than 96 rows in well filled
//     rounds only: 68 x 8192 x 8192 47.7 / 52.0; x 16384 66.2 / 59.5; x 18432, 288 tiles 98 / 104; 66 x 36864 x 4096, 576 tiles 82.0 / 89.1;
//   more than 768 tiles (a vocabulary) fill two 128 x 128 tiles per CU: 100 x 49152 x 4096 107 / 103, x 50304 109 / 121, x 65536 x 8192 209 /
//     242; 52 x 50304 x 7552, 786 tiles 155 / 171; 64 x 65536 x 4096 135 / 101; 24 x 50304 x 2048 plain 52.5 / 50.5, 33.1 / 40.8.
// (17 to 32 rows run in the 64-row tile where K is no multiple of 256: 26 x 19968 x 4992 plain 39.6 / 45.6, as 33 to 64 rows do.)
inline bool rows_stream_uncut(int M, int N, int K, bool read_once) {
    if (M > kRowsStreamMaxM || !rows_stream_pays(M, N, K, 1)) return false;
    const int tiles = (N + 63) / 64, rounds = (tiles + 255) / 256;
    if (M <= 32 && K % 256 == 0) return tiles >= 96 && (read_once || tiles <= 768);
    if (M <= 64) return tiles >= (M <= 32 ? 96 : 128) && (read_once ? tiles <= 768 || rounds * 208 <= tiles : tiles <= 256);
    return read_once && tiles >= 128 && tiles <= 768 && (M >= 96 || rounds * 208 <= tiles);
}
// The operator entry points do not know what else runs between two of their calls.  Up to 16 rows weights of this size or more
// are taken to come from HBM every time and are read with the non-temporal hint.  Calls of more rows ask more of a second read: where
// the memory-side cache can hold the weights they are read with plain loads, which costs a caller whose weights do come from HBM
// 3 to 9 % (64 x 16384 x 4096 26.7 -> 29.3 us, 34.4 without the stream) and spares the others 10 to 35 % (25.1 -> 22.3).
constexpr size_t kReadOnceOperandBytes = (size_t)64 << 20;
constexpr size_t kMemorySideCacheBytes = (size_t)256 << 20;   // of the part
inline bool operator_weights_read_once(int64_t M, int N, int K) {
    return (size_t)N * K * 2 >= (M <= 16 ? kReadOnceOperandBytes : kMemorySideCacheBytes);
}
// Up to 64 rows over a wide output with a short K (the vocabulary): a workgroup is mostly start-up and epilogue, so two per
// CU, of 64 x 128 with three stages (47 x 50304 x 1024: 22.1 us, as a rows stream 30.0, 128 x 128 tiles 25.8; 24 x 50304 x 256
// 8.0, 16.9 and 9.4; even at K = 2048: 47.9 and 49.6).  More rows than 64: 128 x 128 tiles (68 x 50304 x 1024 24.7, 64 x 128 29.5).
inline bool short_k_wide(int M, int N, int K) { return M > 16 && M <= 64 && K < 2048 && N > 256 * 128; }

// ---- 17 to 512 rows: slices of 16 rows ----
// Row slices of the weight-streaming kernels against the tile kernels for a problem of 17 to 512 rows, from two cost
// estimates in microseconds whose constants are measured (projections of 2 to 400 MB, 17 to 1024 rows).  Slices: the
// first reads the weights at about 4 TB/s, every further one reads them again out of L2 or the memory-side cache at about
// 7.5 TB/s.  Tiles: the time does not depend on the row count while all workgroups are resident at once; it is the larger
// of the weights at about 3 TB/s and of the K loop (0.33 us per step of 64 columns, 0.23 us where two groups of waves
// share it; longer in proportion once the tiles no longer fit the chip at once).  Wide outputs with a short K go
// to the tiles from about 33 rows on, narrow outputs with a long K (the output and second feed-forward projections)
// stay with the slices for up to a few hundred rows.
//
// K = 640 to 896 with 33 rows and more: the tiles have the shared loop there, and its price holds where the slices run on the general
// kernel (K no multiple of 256) or on 8-column workgroups (fewer than 2048 columns): slices / tiles 352 x 640 x 640 9.7 / 6.6, 144 x
// 1536 x 640 9.8 / 6.7, 80 x 2560 x 640 9.7 / 6.8, 480 x 768 x 768 9.3 / 7.2, 176 x 1920 x 768 8.7 / 7.4, 224 x 896 x 896 9.7 / 7.7; the least,
// weights out of HBM: 49 x 2304 x 896 7.4 / 8.0, out of the memory-side cache 6.7 / 6.5.  Not where they run on 16-column ones: 96 x 3072 x 768 6.2 /
// 7.4, 64 x 4096 x 768 5.9 / 7.8, nor below 33 rows (24 x 4096 x 896 6.2 / 7.8).
inline bool two_k_groups(int K) { return K % 128 == 0 && K >= 640; }    // what tile_for shares between two groups of waves
inline bool slices_beat_tiles(int M, int N, int K) {
    const int slices = (M + 15) / 16;
    if (slices > 32) return false;
    const double w_mb = (double)N * K * 2e-6;
    const bool streams = K % 256 == 0 && N % 32 == 0;        // else the slower general kernel: 2.5 and 4.5 TB/s
    const double again = w_mb / (streams ? 7.5 : 4.5);
    const double est_slices = 2.0 + w_mb / (streams ? 4.0 : 2.5) + (slices - 1) * (again > 0.1 ? again : 0.1);
    const double wg64 = (double)((M + 63) / 64) * ((N + 63) / 64);
    const bool k_split = two_k_groups(K) && wg64 <= 256.0 && (K >= 1024 || (M > 32 && (K % 256 != 0 || N < 2048)));
    const double k_loop = (K / 64) * (k_split ? 0.23 : 0.33) * (wg64 > 768.0 ? wg64 / 768.0 : 1.0);
    const double est_tiles = 3.0 + (w_mb / 3.0 > k_loop ? w_mb / 3.0 : k_loop);
    return est_slices < est_tiles;
}

// ---- the tile kernel ----
// One workgroup of the large-tile kernels fills a CU, so the tiles run in rounds of 256, and a launch whose last round is
// part-filled pays for more than that round: 25082 x 12288 x 49152 (18.4 rounds) 26.3 ms, 24832 rows (18.2 rounds) 26.35 ms,
// 24576 rows (18 rounds) 24.6 ms; 25082 x 36864 x 12288 (55.1 rounds) 19.1 ms, 24576 rows (54 rounds) 18.2 ms.  Where some
// number of row tiles gives whole rounds and leaves at most 16 row tiles, the launch is cut there and the rest is a launch
// of its own, with whatever tile its size takes (506 x 12288 x 49152: 128 x 256).  The rest is priced in large tiles, at 0.6
// of their rate below 150 of them, and against one launch of large tiles.  (62 sizes that are cut, K = 768 to 6144, as one launch of full_tile's choice: 1.012 of the
// time, between 0.96 and 1.10; 8246 x 4096 x 1024 76.5 cut, 79.2 in one.)  Returns the rows of the first part, 0 for no cut.  The whole rounds are also what the tile order that lets the XCDs share operand panels
// needs (pipe::tile_of_block): 20000 x 12288 x 12288, 14.8 rounds, 4.92 ms as one launch.
inline int rows_in_whole_rounds(int M, int N) {
    constexpr int kCUs = 256;
    const int tm = (M + 255) / 256, tn = (N + 255) / 256, big_tiles = tm * tn;
    if (big_tiles < 2 * kCUs || big_tiles % kCUs == 0) return 0;
    for (int c = tm - 1; c >= 1 && c >= tm - 16; --c) {
        if ((c * tn) % kCUs != 0) continue;
        if (M - c * 256 <= 16) return 0;                 // the rest would be a decode-sized problem: other kernels, no row strides
        const int rest = (tm - c) * tn;                   // large tiles' worth of rows left over
        const double rest_rounds = rest < 150 ? rest / (0.6 * kCUs) : (double)((rest + kCUs - 1) / kCUs);
        const double rounds_now = (big_tiles + kCUs - 1) / kCUs - c * tn / kCUs + 0.27;   // what the part-filled round costs on top
        return rest_rounds + 0.1 < rounds_now ? c * 256 : 0;
    }
    return 0;
}

// The tile of a launch of more than 128 rows, by the time its rounds take: an odd multiple of 64 columns, K below 768, and what full_tile below leaves to the
// pairs.  (Prices and examples are from when every size came here and the loads of a step were not spread; the one-per-CU tiles are 1 to 10 % faster since.)  Measured, us, K in thousands (of 1024):
//   256 x 256, one workgroup per CU                    10 + 21.5 K   per round of up to 256 tiles
//   128 x 256 (three stages), 192 x 128 (three stages), 128 x 128 (three), 96 x 128 (four), one per CU
//                                       9 + 12 K, 7 + 9.2 K, 5 + 7.9 K, 4.5 + 6.9 K   for up to 256 tiles (one round only)
//   192 x 128, 128 x 128, 128 x 64, two per CU         8 + 21.3 K, 6 + 14.5 K, 4.5 + 9 K   per whole round of 512; a last round
//                                                      that gives every CU at most one takes 0.76, 0.58, 0.75 of that, a
//                                                      fuller one 0.92 (128 x 128 in one such round alone: three stages, above)
// So the large tile, the best per flop, gives way where its last round would leave much of the chip idle, to whichever tile
// fills the CUs once (or twice) with the least on top.  us, 256 x 256 / two per CU (192 x 128, 128 x 128, 128 x 64) / one per CU (its
// tile): 3054 x 3072 x 1024 31 / 25, 32, 30 / 32; 2140 x 4096 x 1024 34 / 27, 33, 33; 1200 x 16384 x 4096 188 / 173, 190, 225;
// 2140 x 1024 x 4096 83 / 68, 55, 35 / 29.5 (96 x 128); 1200 x 2048 x 8192 - / -, -, 81 / 54 (96 x 128); 700 x 4096 x 16384 302 / 263,
// 215, 173 / 112 (96 x 128); 700 x 6144 x 2048 - / -, 32, 38 / 25 (192 x 128); 400 x 12288 x 4096 - / -, 64, 74 / 56.5 (128 x 256);
// 2500 x 1280 x 5120 - / -, 50, 58 / 47 (128 x 128); and not where it would not: 6758 x 6144 x 2048 149 / 157, 162; 3262 x 12288 x 4096
// 276 / 306, 315.  All of the one-per-CU tiles run the one-wave-per-SIMD schedule, a tenth ahead of the shared one at every
// depth (700 x 4096 x 16384, 128 x 128: 141 with the shared schedule and 3, 4 or 5 stages, 130 and 123 with this one and 3 and 4).
enum TileChoice { kTile64, kTile64Split, kTile128x64Split, kTile128x64, kTile128PairShared, kTile128Pair, kTile192Pair, kTile96, kTile128, kTile192, kTile128x256, kTile256 };
inline double two_per_cu(double n, double two, double one) {         // n tiles, `two` the time of both of a CU, `one` the share of one
    const double whole = (double)(int64_t)(n / 512), rest = n - whole * 512;
    return two * (whole + (rest == 0 ? 0.0 : rest <= 256 ? one : 0.92));
}
inline double pair_us(int M, int N, double k, int rows) {            // 192 x 128 or 128 x 128
    const double n = (double)((M + rows - 1) / rows) * ((N + 127) / 128);
    return rows == 192 ? two_per_cu(n, 8 + 21.3 * k, 0.76) : two_per_cu(n, 6 + 14.5 * k, 0.58);
}
inline TileChoice choose_tile(int M, int N, int K) {
    auto tiles = [&](int bm, int bn) { return (double)((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
    const double k = K / 1024.0;
    double best = 1e30;
    TileChoice choice = kTile128x64;
    auto offer = [&](TileChoice c, double us) {
        if (us < best) { best = us; choice = c; }
    };
    // (the large tile first and with 3 % in hand: past the first round the others' tails are rougher estimates than its own)
    offer(kTile256, (double)(int64_t)((tiles(256, 256) + 255) / 256) * (10 + 21.5 * k) / 1.03);
    offer(kTile192Pair, pair_us(M, N, k, 192));
    if (tiles(128, 128) > 256) offer(kTile128Pair, pair_us(M, N, k, 128));
    offer(kTile128x64, two_per_cu(tiles(128, 64), 4.5 + 9 * k, 0.75));
    if (tiles(128, 256) <= 256) offer(kTile128x256, 9 + 12 * k);
    if (tiles(192, 128) <= 256) offer(kTile192, 7 + 9.2 * k);
    if (tiles(128, 128) <= 256) offer(kTile128, 5 + 7.9 * k);
    if (tiles(96, 128) <= 256) offer(kTile96, 4.5 + 6.9 * k);
    return choice;
}

// Few tiles (short prompts, narrow layers): smaller tiles put more workgroups on the chip; the K loop of each is a chain
// of dependent steps, so what counts there is how many run side by side and how far ahead the loads run (rows x K x N,
// against two-stage register-staged tiles of the same sizes: 256 x 4096 x 4096 29.9 -> 23.8 us, 2048 x 4096 x 1024 37.6 -> 28.5
// us, 768 x 8192 x 2048 69.5 -> 51.9 us, 128 x 1600 x 6400 16.3 -> 11.8 us).  A long K with all tiles resident at one workgroup
// per CU: two groups of waves per tile, each with half of the K steps and LDS stages of its own, put twice the loads in
// flight (rows x K x N: 128 x 4096 x 4096 23.8 -> 16.5 us, 96 x 16384 x 4096 101.7 -> 67.7 us, 512 x 4096 x 1024 23.3 -> 16.5 us; 1959 x
// 4096 x 1024 24.8 against 30.1 with the best of the tiles below; four groups with two stages each were slower than two with
// three).  From K = 640 on, five steps per group: prompts of 20 to 900 rows through layers of 640, 768 and 896 take 0.88 to 0.98 of the time
// that they took with one group (768: 160 rows 46.8 -> 44.4 us per layer, 600 57.9 -> 53.7); at 256 and 384 there is nothing to gain.
inline bool few_tiles(int M, int N, int K) {
    const int wg128 = ((M + 127) / 128) * ((N + 63) / 64);
    return wg128 < 128 || (two_k_groups(K) && wg128 <= 256);
}
inline TileChoice tile_for(int M, int N, int K) {
    const bool k_split = two_k_groups(K);
    const int wg128 = ((M + 127) / 128) * ((N + 63) / 64), wg64 = ((M + 63) / 64) * ((N + 63) / 64);
    if (few_tiles(M, N, K)) {
        if (k_split && wg64 <= 256) return kTile64Split;              // (1000 x 1024 x 4096: 25.1 -> 20.1)
        return wg128 >= 128 ? kTile128x64Split : kTile64;
    }
    // The one-wave-per-SIMD schedule serves two 128 x 128 workgroups per CU better than the one the two-stage kernels share (6000 x 768 x
    // 3072 48.5 -> 45.3 us, 1200 x 4096 x 16384 238 -> 221, 3054 x 3072 x 1024 32.7 -> 31.0, 5007 x 960 x 832 16.4 -> 15.7), but for a short K (9831 x
    // 576 x 320 10.5 -> 11.2 us, 4120 x 1728 x 192 9.7 -> 10.1; at 576 14.47 -> 14.42 and 13.7 -> 14.2) and for the wide outputs that at most 128
    // rows come here with (68 x 50304 x 256 10.5 -> 11.2, x 1280 33.3 -> 34.6).
    if (M > 128) {
        const TileChoice choice = choose_tile(M, N, K);
        return choice == kTile128Pair && K < 512 ? kTile128PairShared : choice;
    }
    // at most 128 rows: half of a taller tile would be idle
    const int tiles128 = (N + 127) / 128;
    return tiles128 > 256 ? kTile128PairShared : tiles128 == 256 ? kTile128 : kTile128x64;
}

// The tiles with two groups of waves spread the loads of a step over both of its halves, but for one row tile over more weights than the
// eight L2s hold (32 MB): each is then read once, from the memory-side cache or HBM, and what counts is how early it is asked for, all of a step at once.  us,
// at once / spread, weights in the memory-side cache: 114 x 16256 x 1152 10.9 / 12.3, 86 x 14080 x 1536 11.3 / 12.2, 105 x 13440 x 2176 14.8 / 16.0, 21 x
// 14144 x 1408 9.9 / 10.5, 50 x 14016 x 1280 9.2 / 9.9; out of HBM level.  Below
// the line spread is 2 to 16 % ahead (46 x 11264 x 1408, 30 MB 8.7 / 7.5; 32 x 11200 x 1536, 33 MB 9.6 / 8.6).
inline bool reads_weights_past_l2(int M, int N, int K, int tile_rows) {
    return M <= tile_rows && (size_t)N * K * 2 > ((size_t)33 << 20);
}

// More than 128 rows over outputs of a multiple of 128 columns with K from 768 on (what the projections of a layer mostly are): one tile per CU in any
// number of rounds, of the height that leaves the least of them idle.  Since the loads of a K step are spread over both of its halves and the
// output goes straight to memory a tile alone on its CU is faster than two that share it, so what is left to choose is the size.  Measured, us, K in
// thousands, a launch of one round / each of several rounds (540 sizes, hidden 512 to 4096, 300 to 10000 rows; mean error 6 and 3 %):
//   256 x 256  12 + 18.9 K   10.5 + 21.4 K      128 x 256  8.3 + 10.8 K  6.8 + 12 K
//   224 x 256  11.7 + 17.3 K  8.9 + 19.2 K      192 x 128  6.9 + 8.5 K   5.2 + 9.7 K
//   192 x 256  10.2 + 15.5 K  7.4 + 17.3 K      128 x 128  5.6 + 6.4 K   3.9 + 7.1 K
//   160 x 256  9.6 + 13 K     7.3 + 14.7 K       96 x 128  5.5 + 5.2 K   3.6 + 5.8 K
// a part-filled last round takes 0.7 of a full one and 0.3 of what it fills.  Over those sizes the time falls to 0.967 of what tile_for's choice
// takes (the best tile of each: 0.962; the worst of them 1.09, before the pairs below came first), us: 3054 x 3072 x 12288 239 -> 198 (160 x 256), 2140 x 4096 x 4096 82 -> 70, 1700 x 12288 x 4096
// 167 -> 144, 6758 x 2048 x 2048 60 -> 54 (224 x 256), 700 x 5120 x 1280 16.2 -> 13.3 (128 x 128).  Where it stops: at K = 512 the pairs of tile_for
// are level or ahead (8200 x 2048 x 512 27.8 / 30.8, 3800 x 2048 x 512 14.4 / 15.3); 64 columns left over keep tile_for's choice (110 such sizes, K = 768 to 6144, with these tiles
// instead: 0.963 of the time, between 0.79 and 1.085); the tiles shared by two groups of waves are ahead of all of these (900 x 1280 x 5120 28.2 / 31.3, 700 x 2048 x
// 8192 39.4 / 43.6).  Tiles of 128 columns are for one round: where they would be the cheapest in more, and 192 x 128 below K = 1024 throughout, the pairs of tile_for
// come first if their own price is the lower one (one round of 128 x 128 or 192 x 128 in two / as pairs: 1031 x 10880 x 1152 40.9 / 34.7, 4290 x 1920 x 1408 33.2 / 28.4, 3302
// x 2432 x 832 21.3 / 18.9, 8223 x 896 x 1856 35.5 / 33.5; 161 sizes of the first kind 1.04 / 0.98 of what tile_for's choice took before; below K = 1024, 2275 x 10880 x 896
// 56.1 / 51.4, 4802 x 2432 x 832 29.0 / 27.6).  Up to K = 1152 taller tiles in more than one round give way as well where the general choice has pairs: its prices
// are short of their part-filled rounds there (5377 x 6016 x 768 with a residual 72.3 / 66.9, 6000 x 3072 x 768 38.2 / 35.2; 127 sizes 1.018 / 1; K = 1216 to 1536, 41 sizes, 0.984, from
// 1600 on 0.95).  224 rows only where at most one in sixteen of their rows is padding: beyond that 256 are as fast or the next smaller height is.
enum FullTile { kFullNone, kFull256, kFull224x256, kFull192x256, kFull160x256, kFull128x256, kFull192, kFull128, kFull96 };
inline FullTile full_tile(int M, int N, int K) {
    if (M <= 128 || N % 128 != 0 || K < 768 || few_tiles(M, N, K)) return kFullNone;
    constexpr struct { FullTile tile; int rows, cols; double one, one_k, each, each_k; } kTiles[] = {
        {kFull256, 256, 256, 12, 18.9, 10.5, 21.4},     {kFull224x256, 224, 256, 11.7, 17.3, 8.9, 19.2}, {kFull192x256, 192, 256, 10.2, 15.5, 7.4, 17.3},
        {kFull160x256, 160, 256, 9.6, 13, 7.3, 14.7},   {kFull128x256, 128, 256, 8.3, 10.8, 6.8, 12},    {kFull192, 192, 128, 6.9, 8.5, 5.2, 9.7},
        {kFull128, 128, 128, 5.6, 6.4, 3.9, 7.1},       {kFull96, 96, 128, 5.5, 5.2, 3.6, 5.8}};
    const double k = K / 1024.0;
    double best = 1e30, best_narrow = 1e30;
    FullTile choice = kFullNone;
    int64_t choice_tiles = 0;
    for (const auto& t : kTiles) {
        const int64_t tm = (M + t.rows - 1) / t.rows, tiles = tm * ((N + t.cols - 1) / t.cols), whole = tiles / 256, rest = tiles % 256;
        if (t.tile == kFull224x256 && (tm * t.rows - M) * 16 > tm * t.rows) continue;
        const double us = tiles <= 256 ? t.one + t.one_k * k : ((double)whole + (rest == 0 ? 0.0 : 0.7 + 0.3 * (double)rest / 256)) * (t.each + t.each_k * k);
        if (t.cols == 128 && tiles > 256) best_narrow = us < best_narrow ? us : best_narrow;
        else if (us < best) { best = us; choice = t.tile; choice_tiles = tiles; }
    }
    if ((best_narrow < best || K < 1024) && pair_us(M, N, k, 192) < best) return kFullNone;
    if (best_narrow < best && pair_us(M, N, k, 128) < best) return kFullNone;
    if (K <= 1152 && choice_tiles > 256) {
        const TileChoice t = choose_tile(M, N, K);
        if (t == kTile192Pair || t == kTile128Pair) return kFullNone;
    }
    return choice;
}

// ---- weights pulled into the memory-side cache during a prefill's attention ----
// The workgroups of a projection walk K side by side, so weights that come from HBM hold all of them up at every K step (8 prompts of 256 to
// 512 tokens, 24 x hidden 1024: 3011 us, with one layer's weights in all layers 2765).  The attention leaves HBM idle: extra workgroups of its launch
// touch the output projection's and the second feed-forward matrix.  (The first one and the next layer's QKV matrix as well: nothing more, although
// both are read as coldly: their launches have few K steps.)  us without / with, `ahead` bytes of those two matrices:
//   stacks up to hidden 1536 (24 MB): those prompts 3167 / 3012, as an encoder's sentences of 64 to 192 2550 / 2360; 24 x 512 1720 / 1634; 12 x 768 1249
//     / 1140; 12 x 1280 2069 / 1945; 10 x 1536 2266 / 2206; 24 x 1024, one prompt of 37 tokens 1015 / 988, 128 of 8 to 32 2797 / 2612, two of 2000 to 4000
//     (12 layers) 3783 / 3710; nothing to gain beyond 6000 rows (12 x 1024, 12000 rows 4730 / 4740; 10 x 1536, 8200 rows 4657 / 4685);
//   nor where the weights are still cached from the call before: by the weights of all layers and the K/V that the call writes, drawn stacks of 1 to 24 layers, hidden 256
//     to 1600, 20 to 6000 rows, without / with: up to 100 MB 0.994 (127 of them, down to 0.963), 100 to 180 0.999 (61), 180 to 210 1.007 (19), 210 to 240 1.017, 240 to
//     270 1.028, more 1.04;
//   up to 72 MB, stacks that no cache holds, 129 to 2048 rows: 8 x 2048, 600 rows 1080 / 986, 1500 1694 / 1615 (of heads of 128, 900 rows, 1183 / 1190);
//     5 x 2560, 600 887 / 852; 4 x 3072 x 8192 705 / 692; 3054 rows of 2048 2640 / 2674, 60 rows 472 / 514;
//   more take longer to read than the attention lasts (2 x 4096, 500 rows 625 / 656).
constexpr int kAheadBlocks = 128;      // (64: 3051 us for those prompts, 256 and 512 as 128; one prompt of 200 tokens 1231, with 256 1244)
inline bool prefill_touches_weights(int64_t rows, size_t ahead, size_t stack, size_t kv) {
    if (rows <= 16) return false;          // (7 x 1024, 9 rows 191 / 194)
    if (stack + kv <= kMemorySideCacheBytes / 4 * 3) return false;
    if (ahead <= (size_t)24 << 20) return rows <= 6144;
    return ahead <= (size_t)72 << 20 && stack > kMemorySideCacheBytes && rows > 128 && rows <= 2048;
}

// ---- decode attention: the longest sequences first ----
// With more pairs than CUs a pair is one workgroup, and the launch ends with those of the longest sequences, wherever the batch has them; so they
// start first.  us per pass of decode steps, in the order of the batch / longest first (lengths): "server tokens 4096" (48 x 32 heads of 128, 100 to
// 1500) 3219 / 3134; 12 x 32 of 128 (100 to 2000) 1982 / 1895; 24 layers of 24 x 16 of 64 (100 to 1000) 4071 / 3913; four of 100 x 16 of 64 2508 / 2423; 16 x 96 of
// 128 (1024 to 2104) 5902 / 5885.  Sequences of one length gain nothing and pay nothing that stands out of the noise: 24 layers of 64 x 16 of 64, 500 and 900
// keys 5445 / 5439, 6888 / 6902; 48 x 32 of 128, 800 keys 1541 / 1538; four of 100 x 16 of 64, 508 keys 2367 / 2363.  (They paid 0.2 us per workgroup as long as the
// length was read a second time and equal lengths were counted too.)  Measured then: short sequences, 128 x 16 of 64, 200 keys 879 / 888, 128 x 8 of at most 30
// 3870 / 3996, 24 x 32 of 128, 40 to 400 1716 / 1708, so not below 512 slots; and all bits of the lengths instead of the four upper ones, 905 and 3960.
// A wave counts two lengths per lane and no more (attention.hip: sequence_at_place), so the operators' calls with more sequences than that keep the order of the batch.
constexpr int kOrderedSequences = 128;
inline bool decode_longest_first(int splits, int batch, int heads, int capacity) {
    return splits == 1 && batch > 1 && batch <= kOrderedSequences && (int64_t)batch * heads > 256 && capacity >= 512;
}

}  // namespace eet
