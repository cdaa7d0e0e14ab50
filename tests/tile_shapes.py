"""Shapes of the projection tests and the kernel each of them is there for.

tests/test_tile_rules.py holds every entry to the rules the library compiles, so that moving a line of a rule cannot take a
kernel out of its test unnoticed; the GPU tests run them.  Routes as tests/tile_rules_audit.cpp writes them."""
from paper_2104_12470_amd import workloads as wl

# (M, K, N) of operator calls with GELU and with a residual; ragged row and column tails
LARGE_TILES = [
    (3000, 1024, 4160, "256x256 x2"), (4099, 192, 3136, "256x256 x2"), (2049, 4096, 6144, "256x256 x2"), (961, 64, 12352, "256x256 x2"),
    (800, 128, 12352, "192x128 x2"), (801, 128, 12352, "192x128 x2"), (960, 64, 12352, "192x128 x2"),               # two per CU
    (400, 1088, 12352, "128x128 x2"), (2006, 576, 3136, "128x128 x2"),
    (300, 128, 12352, "128x128 x2, shared schedule"), (1480, 320, 3136, "128x128 x2, shared schedule"),
    (1500, 64, 2112, "128x64 x3"), (1500, 128, 2112, "128x64 x3"), (2500, 1280, 1344, "128x64 x3"),
    (1190, 1088, 2112, "96x128 x4"), (2011, 2112, 1088, "96x128 x4"),                                                # one per CU
    (2500, 2560, 1344, "128x128 x3"),
    (1480, 1088, 3136, "192x128 x3"), (700, 2112, 6208, "192x128 x3"),
    (400, 4160, 12352, "128x256 x3"),
]

# operator calls without activation and residual, then with GELU
ROWS_STREAM = [
    (17, 2048, 8192, "rows 32", "rows 32"), (32, 2176, 6144, "rows 64", "rows 64"),            # four K groups, two where K is no multiple of 256
    (33, 2048, 8256, "rows 64", "rows 64"), (64, 2176, 8192, "rows 64", "rows 64"),
    (64, 2176, 6144, "64x64 x3, two K groups", "64x64 x3, two K groups"),
    (20, 64, 33024, "64x128 x3", "128x128 x2, shared schedule"), (64, 192, 32832, "64x128 x3", "128x128 x2, shared schedule"),   # a wide output with a short K
    (97, 8192, 16448, "rows 128", "rows 128"),                                                 # weights no cache holds
    (352, 640, 640, "64x64 x3, two K groups", "64x64 x3, two K groups"), (33, 640, 3584, "64x64 x3, two K groups", "64x64 x3, two K groups"),    # K shared from 640 on
    (480, 768, 768, "64x64 x3, two K groups", "64x64 x3, two K groups"), (225, 896, 896, "64x64 x3, two K groups", "64x64 x3, two K groups"),
    (96, 768, 3072, "slices", "slices"), (24, 896, 4096, "slices", "slices"),
    (65, 4096, 16384, "128x64 x3, two K groups", "128x64 x3, two K groups"), (128, 4224, 16384, "128x64 x3, two K groups", "128x64 x3, two K groups"),
]

# (M, K, N, halfs between rows of x and y beyond K and N) of strided operator calls
STRIDED = [
    (3000, 1024, 4160, 64, 72, "256x256 x2"),
    (300, 512, 640, 8, 64, "64x64 x3"),
    (2049, 4096, 6144, 64, 0, "256x256 x2"),
    (8492, 256, 4096, 64, 72, "8192 + 128x64 x3"),       # 544 large tiles: two whole rounds, then 300 rows
    (2648, 256, 16384, 64, 0, "2048 + 192x128 x2"),      # 704 large tiles: two whole rounds, then 600 rows
    (40, 2048, 8256, 64, 72, "rows 64"),
]


def _layer(hidden, heads, ffn, batch, S, **routes):
    return wl.Workload(f"tiles{hidden}x{batch * S}", 41, hidden, heads, ffn, 1, batch, S, max(1, S - S // 8), S, 1, S + 2), routes


# prompts through a layer: cache rows (qkv) and mapped rows (o, ffn2) out of the one-per-CU tiles
LAYERS = [
    _layer(2048, 16, 2048, 2, 370, qkv="192x128 x3"),
    _layer(2048, 16, 2048, 6, 400, o="192x128 x3", ffn2="192x128 x3"),
    _layer(3072, 24, 3072, 2, 190, qkv="128x128 x3", ffn1="128x64 x3, two K groups"),
    _layer(4096, 32, 12288, 2, 210, qkv="128x256 x3", ffn1="128x256 x3"),
]
