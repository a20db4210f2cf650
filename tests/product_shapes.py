"""Sizes that reach every kernel of the any-size product: each tile side, load width, operand layout and element type."""

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

# an operand [rows, columns] just below and just above 4 GB: (columns, rows below, rows above), multiples of 16
FOUR_GB = {"f32": (1040, 1032432, 1048640), "bf16": (1040, 2064880, 2097280), "fp8_e4m3": (1040, 4129760, 4194000)}
