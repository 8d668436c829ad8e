"""Shapes that reach every instantiation of the product kernel.

Key: (workgroup tile rows, tile columns, paired scale fetch (K a multiple of 256), K split); value: (M, N, K) for which
the planner picks exactly that variant.  All are ragged (M not a multiple of 64, N not a multiple of 4).  A test without
a GPU checks the planner's choice for each, so the GPU parity test over this table is known to run all of them.
"""

VARIANT_SHAPES = {
    (128, 128, False, False): (77, 6, 64),
    (128, 128, False, True): (71, 6, 1152),
    (128, 128, True, False): (16751, 578, 256),
    (128, 128, True, True): (12226, 17, 4096),
    (128, 192, True, False): (12, 5, 256),
    (128, 192, True, True): (13, 7, 1024),
    (128, 256, False, False): (2593, 2955, 64),
    (128, 256, False, True): (888, 1595, 3136),
    (128, 256, True, False): (2860, 2774, 256),
    (128, 256, True, True): (521, 2377, 3328),
    (256, 128, False, False): (18382, 131, 64),
    (256, 128, False, True): (16416, 5, 1216),
    (256, 128, True, False): (16951, 201, 256),
    (256, 128, True, True): (4857, 7, 3584),
    (256, 256, False, False): (19641, 521, 64),
    (256, 256, False, True): (2461, 1622, 4160),
    (256, 256, True, False): (14086, 783, 256),
    (256, 256, True, True): (17890, 201, 3840),
}

# The same for operands with 1 x 128 outer blocks (K a multiple of 128; no 256 x 256 tile there: that mode keeps two
# accumulator sets per wave).
VARIANT_SHAPES_BLOCK128 = {
    (128, 128, False, False): (13242, 73, 128),
    (128, 128, False, True): (731, 137, 1152),
    (128, 128, True, False): (2085, 1363, 512),
    (128, 128, True, True): (13657, 41, 3584),
    (128, 192, True, False): (2444, 1547, 256),
    (128, 192, True, True): (126, 2773, 2048),
    (128, 256, False, False): (6452, 2450, 1408),
    (128, 256, False, True): (6439, 171, 2944),
    (128, 256, True, False): (2628, 2958, 512),
    (128, 256, True, True): (10813, 206, 3072),
    (256, 128, False, False): (18350, 263, 1408),
    (256, 128, False, True): (1293, 970, 2432),
    (256, 128, True, False): (6332, 2378, 512),
    (256, 128, True, True): (3661, 225, 3584),
}

# Ragged outputs of other sizes, (outer mode, M, N, K), whatever tile they get: narrow and short ones, reductions with and
# without a split
RAGGED_SHAPES = [(0, 10762, 150, 1856), (0, 3105, 393, 2560), (0, 11069, 134, 2880), (0, 16564, 193, 3072), (0, 3000, 770, 2304),
                 (0, 700, 760, 8192), (0, 1000, 520, 3072), (1, 16897, 2141, 512), (1, 181, 1495, 256), (1, 4409, 281, 1920),
                 (1, 6016, 4096, 256), (0, 309, 205, 3712), (0, 196, 174, 6016), (1, 287, 279, 3712), (1, 481, 213, 12544)]

# Small tiles and the kernel of each, (outer mode, M, N, K, tile, K split, whether the waves split the reduction).  Split waves work in stages
# of 4 chunks of 64 (8 with outer blocks): whole and ragged outputs, in one piece and split, with a last split shorter than a
# stage, one that ends inside a stage, and whole ones; neighbours that stay with the other kernel.
SMALL_TILE_KERNELS = [
    (0, 130, 129, 640, (64, 64), 1, True), (0, 144, 5505, 2048, (64, 128), 1, True), (0, 181, 128, 5248, (64, 64), 9, True),
    (0, 128, 128, 5824, (64, 64), 10, True), (0, 145, 131, 1664, (64, 64), 3, True), (0, 128, 128, 2304, (64, 64), 3, True),
    (0, 129, 451, 11264, (64, 128), 15, True), (1, 263, 263, 896, (64, 64), 1, True), (1, 921, 802, 1664, (64, 64), 1, True),
    (1, 3303, 260, 1792, (64, 128), 1, True), (1, 258, 275, 1792, (64, 64), 3, True), (1, 256, 320, 2688, (64, 64), 4, True),
    (1, 257, 274, 8704, (64, 64), 9, True), (1, 256, 704, 4096, (64, 64), 4, True), (1, 321, 267, 13056, (64, 128), 13, True),
    (1, 332, 270, 12544, (64, 128), 13, True), (1, 512, 704, 5760, (64, 128), 5, True),
    (0, 222, 4901, 320, (64, 64), 1, False), (0, 204, 513, 5632, (64, 128), 11, False), (0, 726, 372, 3072, (64, 128), 6, False),
    (1, 2162, 513, 1152, (64, 64), 1, False), (1, 290, 838, 10240, (64, 128), 14, False), (1, 257, 260, 2048, (64, 64), 4, False)]

# Layers whose backward products share a launch, (outer mode, N, D, C, tile, whether the waves split the reduction): every tile that such
# launches take, with both reductions (N and C) multiples of 256 (paired scale fetch; 128 x 256 is not chosen for these), neither, and one of them - the launch then
# fetches chunk by chunk what the product alone fetches in pairs.
JOINT_LAYERS = [
    (0, 320, 128, 256, (64, 64), True), (0, 320, 128, 320, (64, 64), True), (0, 256, 128, 256, (64, 64), True),
    (0, 768, 640, 896, (64, 128), True), (0, 832, 640, 832, (64, 128), True), (0, 768, 704, 768, (64, 128), True),
    (0, 512, 2560, 320, (128, 128), True), (0, 320, 3328, 320, (128, 128), True), (0, 768, 1408, 768, (128, 128), True),
    (0, 320, 4160, 512, (128, 128), False), (0, 576, 6464, 576, (128, 128), False), (0, 256, 4160, 256, (128, 128), False),
    (0, 512, 5504, 256, (128, 192), False), (0, 320, 6592, 768, (128, 256), False), (0, 576, 6592, 320, (128, 256), False),
    (0, 320, 4672, 512, (256, 128), False), (0, 320, 5568, 320, (256, 128), False), (0, 512, 6272, 512, (256, 128), False),
    (0, 576, 6592, 768, (256, 256), False), (0, 576, 6720, 576, (256, 256), False), (0, 1024, 6720, 1024, (256, 256), False),
    (1, 896, 256, 768, (64, 64), True), (1, 896, 256, 896, (64, 64), True), (1, 768, 256, 768, (64, 64), True),
    (1, 384, 128, 256, (64, 64), False), (1, 384, 128, 384, (64, 64), False), (1, 256, 128, 256, (64, 64), False),
    (1, 768, 640, 896, (64, 128), True), (1, 896, 640, 896, (64, 128), True), (1, 768, 768, 768, (64, 128), True),
    (1, 256, 2176, 256, (64, 128), False), (1, 256, 128, 896, (128, 128), False), (1, 384, 128, 896, (128, 128), False),
    (1, 256, 128, 768, (128, 128), False), (1, 896, 3328, 3456, (128, 128), False), (1, 512, 5504, 256, (128, 192), False),
    (1, 768, 6656, 384, (128, 256), False), (1, 384, 6272, 640, (128, 256), False), (1, 384, 6656, 256, (256, 128), False),
    (1, 384, 5504, 384, (256, 128), False), (1, 512, 6272, 512, (256, 128), False)]
