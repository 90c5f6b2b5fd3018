"""Attention shapes by the kernel that the library's plan rule gives them:
(n_q, n_kv, d, prefix tokens, suffix tokens).  The CPU tests ask the rule for
each one's plan, so a shape that drifts to another kernel fails there; the GPU
tests run them against the oracle."""

# (row tile, d, keys split over workgroups) -> shapes
BY_PLAN = {
    (32, 128, False): [
        # rows below, at and above one tile
        *[(4, 1, 128, 40, t) for t in (1, 7, 8, 9)], (5, 5, 128, 24, 33),
        # key counts around one unit of 32, one round of the 8 wavefronts and
        # two; an odd number of prefix pages puts prefix and suffix into one unit
        *[(8, 2, 128, tp, 3) for tp in (0, 8, 16, 24, 32, 240, 248, 256, 264, 520)],
        # many query heads on one KV head, and a count that is no power of two
        (64, 1, 128, 264, 9), (48, 3, 128, 488, 30), (40, 8, 128, 808, 201),
        # 15 groups of 8 tiles, each on one XCD
        (30, 15, 128, 261, 128),
    ],
    (32, 128, True): [(4, 1, 128, 4104, 2), (16, 2, 128, 6000, 20), (12, 6, 128, 4001, 30),
                      # 30 groups of 8 tiles, each on one XCD
                      (30, 15, 128, 4008, 128)],
    (32, 64, False): [
        *[(6, 2, 64, 40, t) for t in (1, 10, 11)], (3, 3, 64, 24, 31), (3, 3, 64, 24, 32),
        *[(8, 2, 64, tp, 5) for tp in (0, 8, 232, 256)], (16, 16, 64, 72, 50), (32, 4, 64, 3000, 200),
        (12, 4, 64, 104, 1003),
        # 15 groups of 18 tiles, each on one XCD
        (60, 15, 64, 128, 140),
    ],
    (32, 64, True): [(8, 2, 64, 1000, 5), (8, 8, 64, 8200, 1), (2, 1, 64, 20008, 1), (8, 8, 64, 30000, 100),
                     (24, 3, 64, 2005, 30)],
    # 64-row tiles: Q in LDS at d = 128, in registers at d = 64
    (64, 128, False): [(32, 8, 128, 104, 400), (64, 8, 128, 1000, 200), (64, 8, 128, 104, 197), (24, 3, 128, 2000, 700),
                       (20, 5, 128, 520, 500)],
    (64, 128, True): [(32, 8, 128, 16392, 64), (20, 5, 128, 16005, 70), (24, 3, 128, 4001, 200),
                      (32, 8, 128, 4001, 130)],
    (64, 64, False): [(20, 5, 64, 4000, 1500), (20, 5, 64, 1000, 500), (32, 8, 64, 2005, 300)],
    (64, 64, True): [(32, 4, 64, 8200, 200), (24, 3, 64, 8005, 130), (32, 8, 64, 8005, 130)],
    # 256-row tiles: (KV head, split) groups of a multiple of 8 and not
    (256, 128, False): [(24, 3, 128, 520, 2200), (32, 8, 128, 72, 2200)],
    (256, 128, True): [(8, 1, 128, 4000, 1200), (20, 5, 128, 8005, 300), (32, 8, 128, 8005, 200)],
    (256, 64, False): [(32, 8, 64, 72, 2200), (32, 8, 64, 301, 2200)],
    (256, 64, True): [(20, 5, 64, 4001, 500), (32, 8, 64, 8005, 300), (16, 16, 64, 8005, 700)],
}

# Prefixes that end inside a page, at several slots: what the page holds past
# them (NaN in the tests) must not reach the output.
RAGGED = {
    (32, 128): [(8, 2, 128, 16 * p + r, 5) for p, r in ((0, 1), (1, 5), (2, 8), (3, 15), (17, 1), (20, 15))],
    (32, 64): [(8, 2, 64, 16 * p + r, 7) for p, r in ((0, 15), (1, 8), (2, 5), (3, 1), (17, 5), (20, 8))],
    (64, 128): [(32, 8, 128, 16 * p + r, 300) for p, r in ((2, 1), (3, 5), (18, 8), (33, 15))],
    (64, 64): [(32, 8, 64, 16 * p + r, 300) for p, r in ((9, 15), (60, 8), (125, 5), (126, 1))],
    # the page in the first, a middle and the last key block of its range
    (256, 128): [(12, 6, 128, 3841, 700), (12, 6, 128, 3855, 700), (8, 1, 128, 5573, 700), (8, 1, 128, 5576, 700),
                 (12, 6, 128, 4129, 700), (8, 1, 128, 6879, 700)],
    (256, 64): [(12, 6, 64, 3845, 700), (12, 6, 64, 3848, 700), (8, 1, 64, 5473, 700), (8, 1, 64, 5487, 700),
                (12, 6, 64, 4136, 700), (8, 1, 64, 6865, 700)],
}

# Batched launches (256-row tiles): (n_q, n_kv, prefixes, suffixes, key blocks
# per range); prefixes that end inside a page in the only, first, middle and
# last block of a range.  At 5 or more blocks a range goes round the four tile
# buffers.
BATCHES = [
    (8, 2, (312, 389, 145, 95), (146, 185, 157, 195), {1}),
    (12, 6, (245, 376, 529, 399), (284, 147, 22, 316), {2}),
    (16, 4, (613, 401, 469, 517), (393, 32, 456, 24), {3}),
    (32, 8, (536, 385, 95, 549), (355, 437, 379, 397), {7, 8}),
]
