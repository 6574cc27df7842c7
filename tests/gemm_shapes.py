"""Sizes (rows, columns, k, products) whose int8 GEMM takes each of the four
tile shapes, at tile edges and with fewer, as many and more k-stages than the
copy ring of the shape: shared by the host test of the plan and the GPU test."""

# shape -> sizes
SHAPES = {
    3: [(1, 1, 1, 32), (63, 65, 64, 32), (64, 64, 129, 32), (65, 130, 320, 32), (129, 63, 321, 32), (100, 70, 385, 32),
        (33, 47, 449, 74), (60, 60, 2100, 16)],
    2: [(67, 1036, 64, 16), (1085, 65, 100, 16), (400, 390, 128, 32), (1084, 65, 192, 16), (510, 250, 200, 32),
        (66, 1036, 320, 16), (640, 500, 190, 32), (545, 67, 448, 32), (66, 1046, 570, 16), (690, 655, 250, 16), (700, 650, 70, 32)],
    1: [(1044, 70, 192, 32), (520, 520, 250, 32), (1035, 79, 320, 32), (1082, 71, 384, 32), (500, 333, 300, 32),
        (900, 130, 600, 32)],
    0: [(783, 770, 64, 16), (772, 784, 128, 16), (387, 794, 256, 32), (389, 773, 320, 32), (719, 259, 448, 32),
        (1537, 130, 300, 32)],
}

# sizes of the 256 x 256 tile with several tiles per workgroup: from the fewest
# k-stages up, even and odd counts, with idle slots and without, a second tile
# for some workgroups only
CHAINED = [(201, 4141, 320, 14), (206, 4279, 380, 14), (4134, 202, 440, 14), (203, 4146, 512, 14), (1801, 390, 448, 32),
           (387, 645, 760, 74), (3497, 388, 570, 14), (273, 3885, 3050, 14)]
