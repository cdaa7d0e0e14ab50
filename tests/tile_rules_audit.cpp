// Host-side questions to the dispatch rules of the projections (paper_2104_12470_amd/csrc/tile_rules.hpp, plain C++): the very
// functions that launch_gemm and the layer's workspace compile.  tests/test_tile_rules.py asks.
//
// Usage: one question per line of the standard input, one answer per line of the standard output
//   route M N K       where a dense operator call of M > 16 rows with an activation or a residual goes ("rows 64": the weight
//                     stream with a tile of 64 rows, "slices", "192x128 x3": tile and LDS stages, "8192 + 128x64 x3": whole rounds
//                     of large tiles, then the rest)
//   bias M N K        the same with neither
//   mapped M N K      the same for a projection whose rows are mapped (a prompt inside a layer), which is never sliced
//   mapped_once M N K and whose weights come from HBM every time
//   ranges M N K      K ranges of a bias + residual projection
//   sums M N K        bytes that the sums of such a cut projection of up to M rows need at most; then the same from a walk over
//                     every row count
//   longest_first B H C  whether the decode attention of B sequences, H heads, C slots and one key range takes the longest first
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <string>

#include "../paper_2104_12470_amd/csrc/tile_rules.hpp"

namespace {

const char* tile_name(eet::TileChoice t) {
    switch (t) {
        case eet::kTile64: return "64x64 x3";
        case eet::kTile64Split: return "64x64 x3, two K groups";
        case eet::kTile128x64Split: return "128x64 x3, two K groups";
        case eet::kTile128x64: return "128x64 x3";
        case eet::kTile128PairShared: return "128x128 x2, shared schedule";
        case eet::kTile128Pair: return "128x128 x2";
        case eet::kTile192Pair: return "192x128 x2";
        case eet::kTile96: return "96x128 x4";
        case eet::kTile128: return "128x128 x3";
        case eet::kTile192: return "192x128 x3";
        case eet::kTile128x256: return "128x256 x3";
        case eet::kTile256: return "256x256 x2";
    }
    return "?";
}

std::string route(int M, int N, int K, bool sliceable, bool once) {
    if (eet::rows_stream_uncut(M, N, K, once)) return "rows " + std::to_string(M <= 32 && K % 256 != 0 ? 64 : eet::rows_tile(M));
    if (sliceable && eet::slices_beat_tiles(M, N, K)) return "slices";
    if (const int head = eet::rows_in_whole_rounds(M, N)) return std::to_string(head) + " + " + route(M - head, N, K, sliceable, once);
    const char* full[] = {nullptr, "256x256 x2", "224x256 x2", "192x256 x2", "160x256 x3", "128x256 x3", "192x128 x3", "128x128 x3", "96x128 x4"};
    if (const eet::FullTile t = eet::full_tile(M, N, K)) return full[t];
    return tile_name(eet::tile_for(M, N, K));
}

}  // namespace

int main() {
    char what[16];
    int M, N, K;
    while (std::scanf("%15s %d %d %d", what, &M, &N, &K) == 4) {
        if (!std::strcmp(what, "route")) std::printf("%s\n", route(M, N, K, true, eet::operator_weights_read_once(M, N, K)).c_str());
        else if (!std::strcmp(what, "bias")) {
            const bool once = eet::operator_weights_read_once(M, N, K), stream = eet::rows_stream_uncut(M, N, K, once);
            std::printf("%s\n", !stream && eet::short_k_wide(M, N, K) ? "64x128 x3" : route(M, N, K, true, once).c_str());
        }
        else if (!std::strcmp(what, "mapped")) std::printf("%s\n", route(M, N, K, false, false).c_str());
        else if (!std::strcmp(what, "mapped_once")) std::printf("%s\n", route(M, N, K, false, true).c_str());
        else if (!std::strcmp(what, "ranges")) std::printf("%d\n", eet::gemm_k_ranges(M, N, K));
        else if (!std::strcmp(what, "sums")) {
            int64_t most = 0;
            for (int m = 1; m <= M; ++m) {
                const int64_t b = eet::gemm_cut_bytes(m, N, K);
                if (b > most) most = b;
            }
            std::printf("%lld %lld\n", (long long)eet::gemm_cut_bytes_up_to(M, N, K), (long long)most);
        } else if (!std::strcmp(what, "longest_first")) std::printf("%d\n", eet::decode_longest_first(1, M, N, K));
        else return 1;
    }
    return 0;
}
