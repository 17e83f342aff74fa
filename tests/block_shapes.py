"""Shapes at which the backward takes blocks of 128 rows, and the kernels it takes: (B, H, Hkv, T, d, lengths or
None, query-stationary route, key-stationary route).  test_gpu_blocks.py runs them against the oracle, test_routes.py
asks the library's rules for their routes.

    query-stationary   "blocks" bwd_dq_kernel, "strips" bwd_dq_small_kernel
    key-stationary     "strips" bwd_dkv_small_kernel; d <= 64: "one group", "two groups" bwd_dkv_kernel;
                       d = 128: "64 keys", "128 keys", "pairs" bwd_dkv_pair_kernel
"""


def strips(T):
    return (T + 31) // 32


def blocks(T):
    return (T + 127) // 128


def above(limit, per_head):
    """Heads of the smallest grid beyond `limit`."""
    return limit // per_head + 1


# d = 128: around the points where a key block's sweep gains its first steady-state interval, and where the last tile is
# complete, ragged by one row, or short by one row
LOOP_T = (319, 320, 321, 383, 384, 385, 447, 448, 449, 511, 512, 513, 577, 640, 705)
LOOPS = [(1, above(256, strips(T)), None, T, 128, None, "blocks", "64 keys") for T in LOOP_T] + \
        [(1, above(256, blocks(T)), None, T, 128, None, "blocks", "128 keys") for T in LOOP_T] + \
        [(8, 16, None, T, 128, None, "blocks", "pairs") for T in (447, 448, 449, 511, 512)]

# the search for a start begins at row 384: beyond that, all kernels, with and without groups
LONG = [(1, 24, None, 705, 64, None, "blocks", "two groups"), (1, 24, None, 705, 32, None, "blocks", "two groups"),
        (1, 30, None, 1300, 64, None, "blocks", "two groups"), (1, 40, None, 1025, 64, None, "blocks", "two groups"),
        (1, 46, None, 1300, 64, None, "blocks", "two groups"), (1, 18, None, 4097, 32, None, "blocks", "two groups"), (1, 42, None, 1409, 32, None, "blocks", "two groups"),
        (1, 48, None, 1300, 64, None, "blocks", "one group"), (1, 48, None, 1300, 32, None, "blocks", "one group"),
        (1, 66, None, 449, 64, None, "blocks", "one group"), (1, 8, None, 1300, 128, None, "blocks", "64 keys"),
        (1, 28, None, 1300, 128, None, "blocks", "128 keys")]

GROUPED = [(1, 24, 8, 1025, 64, None, "blocks", "strips"), (1, 24, 8, 1300, 32, None, "blocks", "strips"),
           (1, 9, 3, 1025, 128, None, "blocks", "strips"), (1, 48, 24, 1300, 64, None, "blocks", "two groups"),
           (1, 48, 24, 1025, 32, None, "blocks", "two groups"), (1, 96, 48, 1300, 64, None, "blocks", "one group"),
           (1, 20, 10, 1025, 128, None, "blocks", "64 keys"), (1, 58, 29, 1025, 128, None, "blocks", "128 keys")]

LENS, LONG_AND_SHORT = [1100, 40, 0, 1300, 513], [2, 700, 1025, 31, 129]
PACKED = [(5, 8, 8, 1300, 64, LENS, "blocks", "two groups"), (5, 24, 24, 1300, 64, LENS, "blocks", "one group"),
          (5, 16, 8, 1300, 32, LENS, "blocks", "two groups"), (5, 48, 24, 1300, 64, LENS, "blocks", "one group"),
          (5, 16, 4, 1300, 64, LENS, "blocks", "strips"), (5, 3, 3, 1300, 128, LENS, "blocks", "64 keys"),
          (5, 20, 10, 1300, 128, LENS, "blocks", "128 keys"), (5, 6, 2, 1300, 128, LENS, "blocks", "strips"),
          (5, 38, 38, 1887, 64, LONG_AND_SHORT, "blocks", "one group"), (5, 13, 13, 1887, 32, LONG_AND_SHORT, "blocks", "two groups"),
          (5, 5, 5, 1887, 128, LONG_AND_SHORT, "blocks", "64 keys")]

# packed sequences of much the same length, each of which gets as many workgroups as the longest may need; those above look
# their blocks up by length
ALIKE_LENS = [900, 1100, 1000, 1041]
ALIKE = [(4, H, Hkv, 1100, d, ALIKE_LENS, "blocks", keys) for H, Hkv, d, keys in
         ((8, 8, 64, "two groups"), (16, 16, 64, "one group"), (12, 6, 64, "two groups"), (48, 24, 64, "one group"), (16, 4, 64, "strips"),
          (8, 8, 32, "two groups"), (16, 16, 32, "one group"), (12, 6, 32, "two groups"),
          (5, 5, 128, "64 keys"), (12, 6, 128, "64 keys"), (8, 8, 128, "128 keys"), (16, 8, 128, "128 keys"), (16, 4, 128, "strips"))]

ALL = [s[:2] + (s[2] or s[1],) + s[3:] for s in LOOPS + LONG + GROUPED + PACKED + ALIKE]


def name(s):
    B, H, Hkv, T, d, lens, _, dkv = s
    return f"B{B}_H{H}_{Hkv}_T{T}_d{d}" + ("_packed" if lens else "") + "_" + dkv.replace(" ", "_")
