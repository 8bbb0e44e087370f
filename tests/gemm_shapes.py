"""Shapes at which the GPU tests run the bf16 GEMMs, with the form that each one is there for.

(mode, M, N, K, tile rows, which tiles are cut along K, prefetch) and, for the projection with its rotary epilogue, (rows, K,
query heads, KV heads, ...): every form of the wide kernel at ragged rows and columns.  The forms are asserted on the CPU, apart
from the results: a change of the rule that chooses them shows which form is left without a test, and breaks no comparison."""

WIDE_SHAPES = [
    (0, 131, 72, 192, 128, "none", False), (0, 129, 72, 1088, 128, "all", False), (0, 150, 65800, 1088, 160, "tail", False),
    (0, 185, 16392, 2048, 128, "none", False), (0, 192, 65800, 1088, 192, "none", False),
    (0, 185, 32776, 192, 192, "none", False), (0, 223, 32776, 192, 224, "none", False),
    (0, 200, 16392, 2048, 128, "none", False), (0, 193, 65800, 1088, 224, "none", False),
    (0, 225, 32776, 64, 256, "none", False), (0, 225, 16392, 2048, 128, "none", False),
    (0, 500, 32776, 1088, 192, "none", False), (0, 2047, 1000, 64, 256, "none", True),
    (0, 2001, 3000, 2048, 128, "none", True), (0, 2001, 4000, 2048, 128, "none", True),
    (0, 2001, 10240, 1088, 192, "none", False), (2, 131, 72, 192, 128, "none", False), (2, 160, 72, 1088, 128, "all", False),
    (2, 300, 16392, 1088, 128, "none", False), (2, 185, 8200, 2048, 128, "none", False),
    (2, 370, 16392, 1088, 128, "none", True), (2, 185, 16392, 192, 192, "none", False),
    (2, 223, 16392, 192, 224, "none", False), (2, 223, 8200, 2048, 128, "none", False),
    (2, 440, 16392, 1088, 160, "none", False), (2, 225, 16392, 64, 256, "none", False),
    (2, 225, 8200, 2048, 128, "none", False), (2, 500, 16392, 1088, 192, "none", False),
    (2, 2047, 512, 64, 256, "none", True), (2, 2001, 2040, 2048, 128, "none", True),
    (2, 2001, 5120, 1088, 192, "none", False),
    # forms that none of these takes
    (0, 384, 72, 2048, 128, "all", True), (0, 381, 72, 576, 128, "none", True), (0, 162, 32928, 1088, 192, "none", False),
    (0, 129, 10808, 3072, 128, "all", False), (0, 777, 4624, 3072, 128, "none", False),
    (0, 130, 33416, 64, 160, "none", False), (0, 448, 16440, 64, 160, "none", True),
    (0, 259, 33304, 2048, 128, "none", False), (0, 779, 16824, 1536, 128, "none", False),
    (0, 165, 16520, 4096, 192, "all", False), (0, 644, 27176, 3072, 192, "none", False),
    (0, 673, 27152, 4096, 192, "none", False), (0, 1983, 10128, 2048, 192, "none", False),
    (2, 361, 80, 1088, 128, "all", True), (2, 383, 72, 64, 128, "none", True), (2, 165, 16456, 3072, 192, "none", False),
    (2, 132, 5480, 3072, 128, "all", False), (2, 1564, 1160, 3072, 128, "none", True),
    (2, 130, 16864, 192, 160, "none", False), (2, 773, 4728, 64, 160, "none", True),
    (2, 132, 32912, 1088, 160, "tail", False), (2, 770, 8224, 4096, 128, "none", False),
    (2, 161, 8256, 4096, 192, "all", False), (2, 165, 32904, 1024, 192, "none", False),
    (2, 645, 13728, 3072, 192, "none", False), (2, 683, 13672, 4096, 192, "none", False),
    (2, 1932, 5048, 3072, 192, "none", False),
    # forms with three stages of W that none of these takes
    (0, 254, 32920, 4096, 128, "tail", False), (0, 130, 11032, 4096, 160, "all", False),
    (0, 770, 18896, 3072, 160, "tail", True), (0, 515, 26448, 3072, 192, "tail", False),
    (0, 388, 33208, 3072, 224, "tail", False), (0, 482, 33288, 4096, 256, "tail", False),
    (0, 1924, 12136, 3072, 256, "tail", True), (2, 226, 16640, 4096, 128, "tail", False),
    (2, 134, 5408, 4096, 160, "all", False), (2, 793, 2376, 3072, 128, "none", False),
    (2, 514, 13096, 3072, 192, "tail", False), (2, 404, 16424, 3072, 224, "tail", False),
    (2, 484, 16568, 4096, 256, "tail", False), (2, 1926, 6024, 3072, 256, "tail", True),
    (0, 2424, 2346, 8192, 224, "all", False), (0, 233, 16480, 6144, 256, "all", False),
    (0, 2251, 1040, 5120, 160, "all", True), (2, 2251, 520, 5120, 160, "all", True), (2, 780, 9376, 2560, 160, "tail", True),
    # what the suite has run all along, whatever the height
    (0, 160, 520, 192, None, None, None), (0, 161, 72, 1088, None, None, None), (0, 192, 512, 64, None, None, None),
    (0, 193, 250, 320, None, None, None), (0, 224, 264, 2048, None, None, None), (0, 257, 128, 704, None, None, None),
    (0, 320, 512, 576, None, None, None), (0, 170, 65800, 1024, None, None, None), (2, 224, 264, 2048, None, None, None),
]

QKV_SHAPES = [
    (256, 256, 2, 2, 128, "none", False), (300, 512, 4, 1, 128, "none", False), (77, 1024, 8, 2, 128, "none", False),
    (2048, 2048, 64, 8, 192, "none", False), (2048, 2048, 64, 1, 160, "none", True), (2304, 1024, 64, 8, 192, "none", False),
    (256, 2048, 16, 4, 128, "all", False), (512, 1024, 8, 8, 128, "none", True), (77, 8192, 64, 8, 128, "all", False),
    (150, 192, 2, 1, 128, "none", False), (129, 1088, 2, 1, 128, "all", False), (161, 2048, 112, 16, 128, "none", False),
    (193, 2048, 112, 16, 128, "none", False), (225, 2048, 112, 16, 128, "none", False),
    # forms that none of these takes
    (354, 1088, 1, 1, 128, "all", True), (1604, 3072, 64, 16, 192, "none", False), (131, 3072, 64, 16, 128, "all", False),
    (1543, 3072, 16, 2, 128, "none", True), (1282, 64, 16, 16, 160, "none", False), (1541, 64, 32, 4, 160, "none", True),
    (2054, 3072, 64, 8, 192, "none", False), (961, 64, 64, 8, 192, "none", False), (961, 64, 64, 16, 224, "none", False),
    (1025, 64, 64, 16, 224, "none", False), (1794, 64, 4, 2, 128, "none", True), (1838, 64, 4, 2, 256, "none", True),
    (2305, 64, 112, 16, 256, "none", False), (1983, 3072, 80, 8, 256, "tail", True),
    (1601, 3584, 16, 2, 160, "all", False), (2252, 5120, 8, 1, 160, "all", True), (1921, 6144, 16, 2, 192, "all", False),
    (1319, 3072, 64, 16, 192, "tail", False), (1539, 5120, 64, 8, 224, "tail", False)
]

# at most 128 rows: (rows, K, query heads, KV heads, columns of the narrow kernel's tiles, whether K is cut)
FEW_ROWS_QKV_SHAPES = [(1, 64, 1, 1, 64, False), (128, 4096, 32, 32, 96, True), (100, 8192, 64, 8, 128, True),
                       (65, 192, 112, 16, 96, False), (128, 512, 8, 1, 64, False), (33, 1088, 4, 2, 64, False),
                       (100, 1536, 1, 1, 64, True), (100, 64, 128, 64, 128, False)]

# The narrow kernel at every number of row blocks, (mode, N, K) or (3, K, query heads, KV heads), then columns of a tile and
# whether K is cut, the same at any number of rows: K of one slab, of less than the stages hold, of one slab more than they
# hold twice over; ragged columns, rows of Y that are whole quads and not
NARROW_SHAPES = [
    (0, 72, 64, 64, False), (0, 250, 1536, 64, True), (1, 1000, 2048, 64, True), (0, 250, 704, 64, False),
    (0, 16500, 192, 128, False), (1, 8257, 4096, 128, True), (2, 40, 64, 64, False), (2, 1500, 4096, 64, True),
    (2, 8200, 192, 96, False), (2, 2760, 4096, 96, True), (2, 14000, 320, 128, False), (2, 4132, 5120, 128, True),
]
NARROW_QKV_SHAPES = [
    (3, 64, 1, 1, 64, False), (3, 1536, 1, 1, 64, True), (3, 192, 112, 16, 96, False), (3, 5120, 32, 8, 96, True),
    (3, 64, 128, 64, 128, False), (3, 6144, 64, 8, 128, True),
]
# 4-bit products (N, K, group) and models of one layer (d_model, query heads, KV heads, d_ffn), whose products pair their columns
W4_SHAPES = [
    (250, 384, 128, 64, False), (3072, 4096, 512, 64, True), (20500, 512, 64, 96, False), (10884, 4096, 128, 96, True),
    (30010, 256, 256, 128, False), (10200, 8192, 128, 128, True),
]
W4_PAIR_SHAPES = [
    (128, 1, 1, 128, 64, False), (2048, 1, 1, 128, 64, True), (128, 128, 16, 8320, 96, False), (4096, 64, 16, 5504, 96, True),
    (128, 128, 64, 12416, 128, False), (3072, 64, 8, 4224, 128, True),
]
ROW_BLOCK_EDGES = [1, 16, 17, 32, 33, 64, 65, 80, 81, 112, 113, 128]
