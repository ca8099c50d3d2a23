"""Shapes that take every way of the route that holds rows on chip: what one workgroup holds, every size with
several workgroups per row, the ends of tiles, words and rows (d mod 4), and shapes that keep to
separate launches.  `tiles`: tiles that a workgroup holds (0: separate launches), `workgroups`: per row.  The GPU
tests run the shapes, the CPU test checks that they are launched as it stands here, so a change of the
rules that moves a shape to another way does not go unnoticed."""

# n, d, dtype, rms, tiles, workgroups
SIGN_WORKER = [
    (3, 2047, "f32", False, 1, 1), (2, 2049, "f32", True, 2, 1), (2, 4 * 2048 - 3, "bf16", False, 4, 1),
    (2, 5 * 2048 + 2, "f32", False, 8, 1), (2, 8 * 2048 - 1, "bf16", True, 8, 1),
    (2, 8 * 2048 + 1, "f32", False, 1, 9), (2, 14 * 2048 - 2, "f32", True, 1, 14), (2, 32 * 2048 - 1, "bf16", False, 1, 32),
    (2, 32 * 2048 + 1, "f32", False, 1, 33), (60, 30 * 2048 + 5, "f32", False, 2, 16), (1100, 12 * 2048 - 1, "bf16", False, 14, 1),
    (2, 14 * 2048, "bf16", True, 1, 14), (2, 24 * 2048 - 2, "f32", False, 1, 24), (2, 25 * 2048 + 3, "f32", False, 1, 26),
    (5, 300_001, "bf16", False, 2, 74), (8, 700_002, "f32", True, 4, 86), (9, 1_800_003, "f32", False, 8, 110),
    (9, 2_600_001, "bf16", False, 14, 91), (9, 2_600_003, "f32", True, 14, 91),
    (3, 9_000_005, "f32", False, 24, 184), (3, 9_000_006, "bf16", True, 24, 184), (2, 25_000_001, "f32", False, 24, 509),
    (2, 25_200_001, "f32", False, 0, 12305),
]

# n, d, momentum, rms, tiles, workgroups
SIGN_SERVER = [
    (1, 3, True, False, 1, 1), (3, 2047, False, False, 1, 1), (70, 2047, True, False, 1, 1), (9, 2 * 2048 - 1, True, False, 2, 1),
    (28, 2 * 2048 - 1, False, True, 2, 1), (8, 3 * 2048 + 2, True, False, 4, 1), (16, 4 * 2048, False, True, 1, 4),
    (70, 2 * 2048 - 1, True, False, 1, 2), (8, 4 * 2048 + 2, False, True, 1, 5), (16, 14 * 2048, True, False, 1, 14),
    (5, 24 * 2048 - 3, True, False, 1, 24), (12, 25 * 2048 + 1, False, False, 1, 26), (40, 700_002, True, False, 1, 342),
    (8, 700_002, True, False, 2, 171), (12, 700_003, False, False, 2, 171), (40, 3_000_001, False, True, 2, 733),
    (3, 3_000_001, True, False, 4, 367), (3, 5_000_003, False, True, 4, 611), (2, 9_000_002, True, False, 8, 550),
    (28, 9_000_003, False, False, 8, 550), (2, 17_000_001, True, False, 14, 593), (1, 23_000_003, False, False, 24, 468),
    (40, 5_000_003, True, False, 0, 2442), (70, 3_000_001, False, True, 0, 1465),
]

# n, d, dtype, tiles, workgroups
TERNARY = [
    (3, 2047, "f32", 1, 1), (2, 4 * 2048 - 3, "bf16", 4, 1), (2, 2 * 2048 - 1, "f32", 2, 1), (2, 5 * 2048 + 1, "f32", 1, 6), (2, 8 * 2048 - 2, "bf16", 1, 8),
    (2, 32 * 2048 - 3, "bf16", 1, 32), (2, 32 * 2048 + 1, "f32", 1, 33), (60, 30 * 2048 + 5, "f32", 2, 16),
    (2, 8 * 2048 + 1, "f32", 1, 9), (2, 14 * 2048, "bf16", 1, 14), (2, 24 * 2048 - 2, "f32", 1, 24), (2, 25 * 2048 + 3, "f32", 1, 26),
    (5, 300_001, "bf16", 2, 74), (1, 300_003, "f32", 2, 74), (8, 700_002, "f32", 4, 86), (1, 1_000_003, "bf16", 4, 123),
    (9, 1_800_003, "f32", 8, 110), (4, 8_000_002, "bf16", 8, 489), (9, 2_600_001, "bf16", 14, 91), (9, 2_600_002, "f32", 14, 91),
    (4, 9_000_005, "f32", 14, 314), (2, 11_173_962, "f32", 24, 228), (5, 11_173_963, "f32", 24, 228), (7, 7_826_509, "bf16", 8, 478),
    (3, 9_000_005, "f32", 14, 314), (5, 6_000_002, "bf16", 14, 210), (3, 7_826_508, "bf16", 8, 478),
    (1, 5_000_003, "f32", 0, 2442), (2, 13_000_001, "bf16", 14, 454),
    (1, 5_000_002, "bf16", 0, 2442), (2, 25_200_001, "f32", 0, 12305), (2, 25_200_003, "bf16", 0, 12305),
]

# tiles -> tiles in registers and in LDS, the last template arguments of the kernels
REGISTERS_AND_LDS = {1: (1, 0), 2: (2, 0), 4: (4, 0), 8: (4, 4), 14: (8, 6), 24: (15, 9)}
