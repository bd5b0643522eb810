"""Problems that reach each tile of the kernels and each way a tile may end, as data for
test_plan_host.py, which checks on the CPU that the plan takes that tile (so that a change of
its estimates cannot move a case away unseen), and test_gpu_tiles.py, which runs them."""


def even(V, P):
    per = -(-V // P)
    return [per] * (P - 1) + [V - per * (P - 1)]


# Backward: (class, dtype, T, d, shard rows, strip_elems).  Class 0: 256 x 256 tiles reading W
# and H transposed; 1: 128 x 64; 2: 128 x 128; 3: 256 x 256 on transposed copies.  Column
# blocks of d are 256 (128) wide, a remainder of at most 64 joining the last 256-wide one; a
# remainder of at most half a block skips its dead rows.  d % 64 (32 in float32) is the part
# slice of the logits.
BACKWARD = [
    (0, "bf16", 1333, 456, [9000, 4000], 0),       # 200 columns in the last block, a part slice
    (0, "bf16", 2500, 448, [9000, 4000], 0),       # 192, whole slices
    (0, "bf16", 2500, 616, [9000, 4000], 0),       # 104
    (0, "bf16", 1333, 552, [9000, 4000], 0),       # 40 joined to the block before
    (0, "bf16", 3000, 576, [13000], 0),            # 64 joined, one shard
    (0, "bf16", 4000, 2000, [2999, 3001], 0),      # one dH job over two shards
    (1, "bf16", 257, 1000, [700, 3001], 0),        # 104 columns in the last block
    (1, "f32", 257, 1000, [700, 3001], 0),
    (1, "bf16", 333, 320, [100, 0, 257, 131, 612], 0),  # 64
    (1, "f32", 333, 320, [100, 0, 257, 131, 612], 0),
    (2, "bf16", 1333, 360, [9000, 4000], 0),       # 104
    (2, "f32", 1100, 616, [9000, 300, 5000], 0),   # 104
    (2, "bf16", 200, 264, [30000], 0),             # 8
    (2, "f32", 1100, 520, [9000, 300, 5000], 0),   # 8
    (3, "bf16", 9481, 304, even(16588, 8), 0),     # 48 joined, a part slice, four shards a strip
    (3, "bf16", 13509, 464, [13475], 1 << 26),     # 208; two token chunks, a shard in two pieces
    (3, "bf16", 17088, 616, [6300, 6336], 1 << 26),  # 104
    (3, "f32", 9654, 3128, [3976, 3975], 0),       # 56 joined, a part slice, two shards a strip
    (3, "f32", 6573, 7312, even(7414, 8), 0),      # 144
    (3, "f32", 8332, 7016, even(7981, 8), 0),      # 104
]

# Forward: (kind of the whole forward, kinds of the shards folded one by one, dtype, T, d, shard
# rows).  Kind 0: 256 x 256 tiles; 1: streamed 256 x 128; 2: streamed 128 x 64.
FORWARD = [
    (1, [1], "bf16", 230, 2672, [21915]),          # a part slice, the last tile 155 rows
    (1, [2] * 16, "bf16", 198, 1664, even(17677, 16)),
    (1, [1], "bf16", 164, 2048, [61184]),          # whole slices and tiles
    (1, [1, 2, 2], "f32", 65, 2056, [50000, 1, 300]),
    (1, [1], "f32", 128, 2048, [51200]),
    (2, [2, 2, 2], "bf16", 65, 2056, [50000, 1, 300]),
    (2, [0, 2, 2], "f32", 1100, 520, [9000, 300, 5000]),
    (0, [0, 2, 0], "bf16", 1100, 520, [9000, 300, 5000]),
    (0, [0, 0], "bf16", 2048, 448, [9000, 4000]),
]
