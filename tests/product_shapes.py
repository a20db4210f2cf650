"""Sizes that reach every kernel of the any-size product: each tile side, load width, operand layout and element type, and of
the ring kernel each tile, way of storing and element type."""

# (rows, columns) whose tiles are 128, 64 and 32 wide; units divide every size: 16 elements make 16-byte loads of any type, 4
# make 4-byte loads of bf16 and fp8, 1 single elements (fp8 then has no tile of 128)
OUTPUTS = {16: ((1936, 2000), (400, 1600), (48, 1040)), 4: ((1940, 2004), (404, 1604), (44, 1036)),
           1: ((1937, 2001), (401, 1601), (33, 1041))}
# less than the loads in flight and a partial K-tile; the loop over whole K-tiles, several passes
CONTRACTIONS = {16: (176, 656, 1968), 4: (180, 660, 1972), 1: (177, 661, 1969)}

# in place, q = 3: shards that end inside a K-tile, longer and shorter than the K-tiles in flight; all three products on
# tiles of 128 and of 64
CUBES = {16: ((9 * 216, 3 * 656, 9 * 224), (9 * 64, 3 * 336, 9 * 144)),
         4: ((9 * 220, 3 * 660, 9 * 228), (9 * 60, 3 * 332, 9 * 140)),
         1: ((9 * 217, 3 * 661, 9 * 227), (9 * 59, 3 * 331, 9 * 139))}

# in place, q = 8: shards of the contraction index that are shorter than a K-tile (32 fp32, 64 bf16 or 128 fp8 indices) keep
# a product off the ring kernel: the 16-byte kernels through registers
SHORT_SHARDS = {"bf16": ((3584, 2112, 3584), (2112, 448, 2048), (192, 448, 3584), (64, 448, 3584), (576, 448, 1024)),
                "fp8_e4m3": ((7168, 896, 4096), (2112, 896, 4096), (576, 896, 2048), (64, 896, 7168), (576, 128, 1024)),
                "f32": ((1792, 2112, 1792), (1792, 1056, 1792), (1792, 160, 1792), (1088, 224, 1792), (64, 224, 1792))}

# ring kernel: (rows, columns, blocks per side of the cube, contractions).  Multiples of 16 wherever an operand may be
# contiguous there; output rows that are not whole cache lines
RING = [(48, 1040, 1, (272, 1040, 2064)), (816, 1040, 1, (400, 1040)), (400, 1040, 1, (144, 1040, 8208)), (1616, 2064, 1, (272, 400, 1040)),
        (2064, 4112, 1, (2064,)), (4112, 2064, 1, (1040, 2064)), (4112, 4112, 1, (80, 1040)), (272, 144, 3, (1040,)),
        (3088, 1168, 1, (1040, 4624)), (1136, 7152, 1, (1040, 4112)), (2064, 3088, 1, (4112,))]
# fp8 with bf16 results on each tile with the 64-deep MFMA, in every layout; with 400 and 48 rows on smaller ones
RING_DEEP = [(1616, 2064, 1040), (1136, 7152, 4112), (1552, 8256, 400)]
# more than 16 MB of results in rows of whole cache lines: streaming stores
RING_LINES = [(1552, 8256, 1, (144, 400)), (2064, 7232, 1, (144,)), (592, 1088, 3, (144,))]
# A B^T of an odd number of columns: results are stored element by element
RING_ODD = [(45, 33, 1, (784,)), (3001, 145, 1, (784,)), (4001, 145, 1, (784,)), (1105, 1041, 1, (6160,)), (4001, 1041, 1, (8208,)),
            (2049, 1041, 1, (8208,)), (3001, 4111, 1, (4112,)), (1105, 7151, 1, (8208,))]
# in place (q, M, K, N): shards that end inside a K-tile, in every direction
RING_CUBES = [(3, 9 * 272, 3 * 656, 9 * 368), (3, 9 * 304, 3 * 272, 9 * 272), (3, 9 * 16, 3 * 1040, 9 * 272)]
# whole cache lines and more than 16 MB; shards of an odd number of columns or rows
RING_CUBES_LINES = [(3, 9 * 272, 3 * 1344, 9 * 576), (3, 9 * 464, 3 * 1344, 9 * 64)]
RING_CUBES_ODD = [(2, 4 * 528, 2 * 1041, 4 * 2064), (2, 4 * 272, 2 * 337, 4 * 336), (2, 4 * 136, 2 * 200, 4 * 68), (2, 4 * 1552, 2 * 2048, 4 * 516)]
# an operand [rows, columns] at most and just above 1 GiB, the ring kernel's limit: (columns, rows at most, rows above)
ONE_GB = {"f32": (1040, 258096, 258112), "bf16": (1040, 516208, 516224), "fp8_e4m3": (1040, 1032432, 1032448)}

# an operand [rows, columns] just below and just above 4 GB: (columns, rows below, rows above), multiples of 16
FOUR_GB = {"f32": (1040, 1032432, 1048640), "bf16": (1040, 2064880, 2097280), "fp8_e4m3": (1040, 4129760, 4194000)}
