"""Which kernels a call takes (csrc/sb_share.h, csrc/sb_split.h), compiled for the host: the rules' edges, and the routes that the GPU
tests name for their shapes."""
import math
import os
import random
import shutil
import subprocess

import pytest

import block_shapes

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2410_17980_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

MAIN = r"""
#include <stdio.h>
#include "sb_share.h"
#include "sb_split.h"
using namespace sb;
int main()
{
    int B, H, Hkv, T, d, packed, Ttot;
    while (scanf("%d %d %d %d %d %d %d", &B, &H, &Hkv, &T, &d, &packed, &Ttot) == 7) {
        if (packed == 2) {                              // decode; Ttot: m wanted
            const Split s = split_of((long)B * Hkv * ((H / Hkv + 15) / 16), 4.0 * B * Hkv * T * d, T, d, Ttot);
            printf("%d %d %d %d\n", s.near, s.C, s.nfar, room(T));
            continue;
        }
        if (packed == 8 || packed == 9) {               // grouped heads' key-stationary pass where there is room for parts, of a batch or packed
            const KeyPlan p = key_plan(B, H, Hkv, T, d, packed == 9, Ttot);
            printf("%d %d %d\n", (int)p.keys, p.parts, p.beyond);
            continue;
        }
        const long strips = pieces(B, H, T, 32, packed, Ttot);
        if (packed == 3) {                              // waves of a strip's workgroup
            printf("%d %d\n", query_strips(B, H, T, d, false, 0) && four_waves(pieces(B, H, T, 32, false, 0), 1, T, d),
                   keys_of(B, H, Hkv, T, d, false, 0) == Keys::STRIPS && four_waves(pieces(B, Hkv, T, 32, false, 0), H / Hkv, T, d));
            continue;
        }
        if (packed == 4) {                              // packed batch: chunks a head of the remainder bias's gradient
            printf("%d\n", bias_chunks(B, T, true, Ttot));
            continue;
        }
        if (packed == 7) {                              // packed batch: its heads turn with every fourth block
            printf("%d\n", turn_with_every_fourth(H, H / Hkv));
            continue;
        }
        if (packed == 6) {                              // packed batch: its blocks are looked up by their length
            printf("%d\n", packed_as(B, T, Ttot) == Packed::BY_LENGTH);
            continue;
        }
        if (packed == 5) {                              // forward: waves that take a strip's subtiles; Ttot: without m, 2 where two strips share a workgroup
            const long n = pieces(B, H, T, 32, false, 0);
            printf("%d\n", !small_fwd_grid(n, T, d) ? 0 : Ttot && two_strips(n, T, d) ? 2 : d == 128 || (d == 32 && four_fwd_waves(n, T)) ? 4 : 8);
            continue;
        }
        printf("%d %d %ld %d\n", small_fwd_grid(strips, T, d), query_strips(B, H, T, d, packed, Ttot), strips,
               (int)keys_of(B, H, Hkv, T, d, packed, Ttot));
    }
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    if not shutil.which(HIPCC):
        pytest.skip("no hipcc")
    tmp = tmp_path_factory.mktemp("routes")
    (tmp / "main.hip").write_text(MAIN)
    subprocess.run([HIPCC, "-std=c++17", "-O1", "--offload-host-only", f"-I{CSRC}", "main.hip", "-o", "main"],
                   cwd=tmp, check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)

    def run(rows):
        text = "".join(" ".join(str(int(x)) for x in r) + "\n" for r in rows)
        out = subprocess.run([str(tmp / "main")], input=text, text=True, check=True, stdout=subprocess.PIPE).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return run


def packed(lens, H, d, max_T=None, Hkv=None):
    return (len(lens), H, Hkv or H, max_T or max(lens), d, 1, sum(lens))


KEYS = ("strips", "one group", "two groups", "64 keys", "128 keys", "pairs")


def strips(ask, row):
    """Whether the forward, the query-stationary and the key-stationary pass take a strip a workgroup."""
    fwd, dq, _, keys = ask([row])[0]
    return bool(fwd), bool(dq), KEYS[keys] == "strips"


def test_packed_strips_are_counted_and_launched_as_they_exist(ask):
    """However loose max_T is: no more workgroups than strips and one per sequence and head."""
    rng = random.Random(3)
    rows, least = [], []
    for _ in range(200):
        lens = [rng.choice((0, 1, 31, 32, 33, 64, 100, rng.randrange(1, 3000))) for _ in range(rng.randrange(1, 200))] + [5]
        H = rng.randrange(1, 9)
        for max_T in {max(lens), sum(lens)}:
            rows.append(packed(lens, H, 64, max_T))
            least.append(H * sum((n + 31) // 32 for n in lens))
    for row, strips, got in zip(rows, least, ask(rows)):
        assert strips <= got[2] <= strips + row[0] * row[1]


def test_chunks_of_the_bias_in_packed_batches(ask):
    """Every row once, however loose max_T is; no more than one chunk a sequence too many."""
    rng = random.Random(7)
    rows, least = [], []
    for _ in range(200):
        lens = [rng.choice((0, 1, 127, 128, 129, rng.randrange(1, 3000))) for _ in range(rng.randrange(1, 200))] + [5]
        for max_T in {max(lens), sum(lens)}:
            rows.append((len(lens), 1, 1, max_T, 64, 4, sum(lens)))
            least.append(sum((n + 127) // 128 for n in lens))
    for row, chunks, (got,) in zip(rows, least, ask(rows)):
        assert chunks <= got <= chunks + row[0]


def test_routes_of_the_bias_in_packed_batches(ask):
    """test_gpu_varlen.py, test_bias_gradient_of_many_sequences."""
    import test_gpu_varlen as t
    for (H, lens), want in zip(t.test_bias_gradient_of_many_sequences.pytestmark[1].args[1], (False, True)):
        assert all(strips(ask, packed(lens * 9, H, d, 1400))[1:] == (want, want) for d in (32, 64, 128))


def test_strips_of_packed_batches(ask):
    """By the strips that there are and by max_T, as in a batched call; one long sequence among short ones takes strips."""
    for lens, H, d, max_T in (([600] + [20] * 30, 2, 128, None), ([1000] + [20] * 30, 4, 32, None), ([500] + [60] * 40, 2, 32, None),
                              ([250] + [16] * 20, 4, 64, None), ([32] * 64, 4, 64, 2048), ([100] * 13, 4, 64, 1300)):
        assert strips(ask, packed(lens, H, d, max_T)) == (True, True, True), (H, d)
    for lens, H, d, max_T in (([32] * 64, 4, 64, 64), ([32] * 64, 8, 128, 512), ([32] * 200, 4, 64, 6400), ([4000] + [16] * 40, 4, 128, None)):
        assert not any(strips(ask, packed(lens, H, d, max_T))), (H, d, max_T)


def test_equal_lengths_take_the_route_of_the_batched_call(ask):
    rng = random.Random(4)
    shapes = [(rng.randrange(1, 9), rng.randrange(1, 25), rng.randrange(1, 4200), rng.choice((32, 64, 128))) for _ in range(400)]
    batched = ask([(B, H, H, T, d, 0, 0) for B, H, T, d in shapes])
    for shape, a, b in zip(shapes, batched, ask([(B, H, H, T, d, 1, B * T) for B, H, T, d in shapes])):
        assert a[:2] == b[:2] and (KEYS[a[3]] == "strips") == (KEYS[b[3]] == "strips"), shape


def test_shapes_of_the_gpu_tests(ask):
    """test_gpu_small_grids.py, test_packed_places: one strip a workgroup (the forward at d = 32 only beyond 320 rows)."""
    for lens, H, Hkv, max_T in (([0] * 3 + [1, 33] * 32 + [0, 300, 31], 2, 2, 300), ([2, 0, 34] * 21 + [1, 400] + [0] * 70, 1, 1, 400),
                                ([100] * 13, 4, 2, 1300)):
        for d in (32, 64, 128):
            assert strips(ask, packed(lens, H, d, max_T, Hkv)) == (d > 32 or max_T > 320, True, True), (lens, d)


def test_shapes_of_four_waves(ask):
    """test_gpu_small_grids.py, test_strips_of_four_waves."""
    for d in (32, 64):
        assert ask([(1, H, Hkv, T, d, 3, 0) for H, Hkv, T in ((21, 21, 993), (15, 15, 2200), (11, 11, 3105), (72, 24, 1750))]) == \
            [(1, 1)] * 3 + [(0, 1)], d
    assert ask([(1, 12, 12, 3200, 64, 3, 0)]) == [(1, 1)]               # test_sharp_and_far_rows_in_one_strip
    import test_gpu_small_grids as t
    for H, T in t.test_forward_strips_of_four_waves.pytestmark[0].args[1]:
        assert ask([(1, H, H, T, 32, 5, 0), (2, H, H, T, 32, 5, 0)]) == [(4,), (0,)], (H, T)
    for H, Hkv, T, d in t.test_forward_two_strips.pytestmark[0].args[1]:
        assert ask([(1, H, Hkv, T, d, 5, 1), (2, H, Hkv, T, d, 5, 1)]) == [(2,), (0,)], (H, T, d)
    for H, d in t.test_forward_two_strips_packed.pytestmark[0].args[1]:
        n = H * sum((x + 31) // 32 for x in t.TWO_STRIPS_LENS)
        got = ask([packed(t.TWO_STRIPS_LENS, H, d)])[0]
        assert got[0] and n <= got[2] and (384 < got[2] <= 512 if d == 128 else got[2] > 768), (H, d)


def test_shapes_of_the_longest_strips(ask):
    """test_gpu_small_grids.py, test_longest_strips: strips up to 8192 rows."""
    for d in (32, 64, 128):
        for T in (4096, 4097, 8192):
            assert strips(ask, (1, 1, 1, T, d, 0, 0)) == (True, True, True), (T, d)
        assert strips(ask, (1, 1, 1, 8193, d, 0, 0))[1:] == (False, False), d
    import test_gpu_small_grids as t
    for T in (65, 96, 97, 128, 129, 255, 257, 321, 500, 1000, 4096):
        for d in (32, 64, 128):
            once, often = ask([(B, 3, 3, T, d, 5, 0) for B in (1, t.beyond_small_grids(T))])
            assert (once > (0,) or (d == 32 and T <= 320)) and often == (0,), (T, d)


def test_limits_of_strips(ask):
    """The shapes that the limits were measured at, on the sides where the comments beside them list them."""
    backward = {True: [(16, 500, 32), (14, 2048, 32), (12, 4096, 32), (1, 8192, 64), (14, 2500, 64), (12, 2600, 64), (16, 500, 128), (8, 2000, 128), (5, 4096, 128),
                       (2, 8192, 128), (1, 8192, 128)],
                False: [(48, 500, 32), (16, 4096, 32), (32, 1000, 64), (32, 500, 128), (24, 1000, 128), (10, 3000, 128), (16, 3000, 64), (8, 3000, 128),
                        (24, 1000, 32), (26, 320, 32), (32, 500, 64), (24, 1000, 64)]}
    forward = {True: [(10, 3000, 32), (1, 8192, 32), (64, 100, 64), (24, 500, 64), (10, 3000, 64), (1, 8192, 64), (1, 16384, 64), (24, 500, 128), (12, 1000, 128),
                      (10, 2048, 128), (1, 8192, 128), (1, 16384, 128)],
               False: [(37, 200, 32), (18, 2048, 32), (96, 100, 64), (48, 500, 64), (16, 2000, 64), (12, 4096, 64), (48, 500, 128), (24, 1000, 128), (9, 4096, 128),
                       (32, 500, 32), (12, 2000, 64), (37, 200, 128)]}
    for side in (True, False):
        for H, T, d in backward[side]:
            assert strips(ask, (1, H, H, T, d, 0, 0))[1:] == (side, side), (H, T, d)
        for H, T, d in forward[side]:
            assert strips(ask, (1, H, H, T, d, 0, 0))[0] == side, (H, T, d)


def test_waves_of_strips(ask):
    """Four waves in place of eight where they are faster whatever the heads' reach, or nearly so: not where a lone far head's chain is long."""
    for d in (32, 64):
        for H, T, four in ((14, 2048, 1), (13, 1990, 1), (10, 2500, 1), (10, 2800, 1), (10, 3300, 1), (12, 2600, 1), (9, 4096, 1), (12, 4096, 1),
                           (8, 2000, 0), (12, 2048, 0), (9, 2900, 0), (8, 3100, 0), (9, 3400, 0), (8, 4096, 0)):
            assert ask([(1, H, H, T, d, 3, 0)]) == [(four, four)], (H, T, d)
    for H, T, waves in ((10, 2500, 4), (10, 3000, 4), (8, 3100, 8), (9, 2753, 8), (7, 3000, 8), (7, 4096, 8), (5, 6000, 8), (4, 7900, 8), (1, 16384, 8), (13, 1990, 0)):
        assert ask([(1, H, H, T, 32, 5, 0)]) == [(waves,)], (H, T)
    assert ask([(1, 10, 10, 3000, 64, 5, 0), (1, 10, 10, 2048, 128, 5, 0)]) == [(8,), (4,)]
    for H, T, d, two in ((12, 2080, 64, 1), (10, 2500, 64, 1), (9, 2752, 64, 1), (10, 3000, 64, 1), (9, 3500, 64, 1), (12, 1200, 128, 1), (8, 2000, 128, 1),
                         (6, 2500, 128, 1), (2, 8192, 128, 1), (1, 16384, 128, 1), (7, 3000, 64, 0), (7, 3500, 64, 0), (5, 6000, 64, 0), (9, 2000, 128, 0),
                         (12, 1000, 128, 0), (7, 3000, 32, 0), (10, 3000, 32, 0)):
        assert (ask([(1, H, H, T, d, 5, 1)]) == [(2,)]) == bool(two), (H, T, d)


def test_shapes_of_the_tests_of_carries(ask):
    """test_gpu_small_grids.py: strips in both passes."""
    import test_gpu_small_grids as t
    rows = [(1, p[0], p[0], p[1], p[2], 0, 0) for f in (t.test_weights_of_rows_that_are_nearly_exhausted, t.test_sharp_and_far_rows_in_one_strip)
            for p in f.pytestmark[0].args[1]]
    assert len(rows) == 12
    for row, (_, dq, _, keys) in zip(rows, ask(rows)):
        assert dq and KEYS[keys] == "strips", row


def test_block_shapes(ask):
    """test_gpu_blocks.py: every shape takes the kernels that it names."""
    rows = [packed(lens, H, d, T, Hkv) if lens else (B, H, Hkv, T, d, 0, 0) for B, H, Hkv, T, d, lens, _, _ in block_shapes.ALL]
    for shape, (_, dq, _, keys) in zip(block_shapes.ALL, ask(rows)):
        assert ("strips" if dq else "blocks", KEYS[keys]) == shape[6:], shape
    by_length = lambda shapes: [x for x, in ask([(s[0], 1, 1, s[3], s[4], 6, sum(s[5])) for s in shapes])]
    assert by_length(block_shapes.PACKED) == [1] * len(block_shapes.PACKED) and by_length(block_shapes.ALIKE) == [0] * len(block_shapes.ALIKE)
    import test_gpu_varlen as varlen
    assert all(x for x, in ask([(len(lens), 1, 1, max(lens), 64, 6, sum(lens)) for lens in varlen.BY_LENGTH.values()]))
    import test_gpu_blocks
    rest = [s[:5] + (0, 0) for s in test_gpu_blocks.random_shapes()] + \
           [(1, H, H, T, d, 0, 0) for H, T, d in ((19, 1300, 64), (48, 1300, 64), (19, 1300, 32), (7, 1300, 128), (28, 1300, 128),
                                                  (24, 333, 128), (66, 449, 64), (30, 1300, 32), (128, 449, 128))]
    for row, (_, dq, _, keys) in zip(rest, ask(rest)):
        assert not dq and KEYS[keys] != "strips", row
    import test_gpu_nonfinite as nonfinite
    rows = [(1, 2 * n, 2 * n, nonfinite.T, d, 0, 0) for d, n, _ in nonfinite.GRIDS]
    assert [(fwd, dq, KEYS[keys]) for fwd, dq, _, keys in ask(rows)] == [(0, 0, g[2]) for g in nonfinite.GRIDS]
    rows = [(1, H, H, T, d, 0, 0) for T in (257, 320, 353, 385, 449, 577, 641, 1283) for d in (32, 64, 128)
            for H in [block_shapes.above(512, block_shapes.strips(T))]]
    assert not any(fwd for fwd, _, _, _ in ask(rows))


def test_strips_of_queries_come_with_strips_of_keys(ask):
    """bwd_dq_small_kernel leaves starts for the strips that exist alone, which is what bwd_dkv_small_kernel reads;
    the block kernels read whole blocks of four."""
    rng = random.Random(6)
    rows = []
    for _ in range(4000):
        Hkv, T, B = rng.randrange(1, 25), round(2 ** rng.uniform(0, 13)), rng.randrange(1, 40)
        is_packed = rng.random() < 0.5
        rows.append((B, Hkv * rng.randrange(1, 9), Hkv, T, rng.choice((32, 64, 128)), is_packed, rng.randrange(1, 1 + B * T) if is_packed else 0))
    got = ask(rows)
    assert any(dq for _, dq, _, _ in got)
    for row, (_, dq, _, keys) in zip(rows, got):
        assert not dq or KEYS[keys] == "strips", row


def test_turns_of_packed_heads(ask):
    """Every fourth block only where all heads would keep to one XCD, and are not many."""
    assert [H for H in range(1, 65) if ask([(4, H, H, 2000, 64, 7, 8000)]) == [(1,)]] == [8, 16, 24]
    assert ask([(4, H, H // 2, 2000, 64, 7, 8000) for H in (8, 16, 24)]) == [(0,)] * 3


def test_two_wave_groups(ask):
    """Key-stationary pass at d <= 64: two groups only where neither near heads nor far ones lose more than a mix gains."""
    for B, H, Hkv, T, want in ((2, 24, 24, 1024, 2), (1, 16, 16, 4096, 2), (1, 32, 32, 2011, 2), (1, 36, 36, 2011, 2), (1, 24, 24, 4096, 2), (1, 32, 32, 4096, 2),
                               (1, 16, 16, 8000, 2), (8, 16, 16, 512, 1), (1, 40, 40, 2048, 1), (1, 48, 48, 1499, 1), (1, 43, 43, 3035, 1), (1, 33, 33, 4096, 1),
                               (8, 16, 16, 2048, 1), (1, 32, 8, 8000, 2), (12, 9, 3, 1500, 2), (12, 9, 3, 3256, 1)):
        assert KEYS[ask([(B, H, Hkv, T, 64, 0, 0)])[0][3]] == ("one group", "two groups")[want - 1], (B, H, Hkv, T)
    for lens, H, max_T, want in (([5000] + [300] * 10, 4, None, 2), ([4500] + [50] * 30, 8, None, 2), ([4000] * 2, 12, None, 2), ([5000] + [16] * 60, 2, None, 2),
                                 ([2000] * 4, 12, None, 1), ([1500] * 6, 9, None, 1), ([5000] + [16] * 300, 2, None, 1), ([32] * 64, 4, 511, 1), ([32] * 64, 4, 512, 1)):
        assert KEYS[ask([packed(lens, H, 64, max_T)])[0][3]] == ("one group", "two groups")[want - 1], (lens[0], H, max_T)


def decode(B, H, Hkv, T, d, want_m=False):
    return (B, H, Hkv, T, d, 2, want_m)


ONE, SPREAD, FAR_AND_NEAR = "one workgroup a head", "spread", "nearest keys first"


def kind(row, got):
    near, _, nfar, _ = got
    return SPREAD if near == 0 else ONE if nfar == 0 else FAR_AND_NEAR


def test_decode_routes(ask):
    """A small cache is spread over the chip only where heads that end within their nearest keys lose less by it than
    far ones gain; always with m, which takes every key."""
    want = {ONE: [(1, 12, 4, 333, 128), (5, 30, 10, 588, 64), (5, 30, 10, 1000, 64), (2, 8, 8, 1000, 64), (5, 30, 10, 1000, 32), (2, 8, 8, 1280, 32),
                  (8, 16, 16, 1000, 128), (5, 30, 10, 1000, 128), (1, 1, 1, 512, 128), (4, 8, 8, 1500, 64)],
            SPREAD: [(1, 12, 4, 600, 128), (4, 8, 8, 1000, 128), (4, 8, 8, 1200, 128), (1, 12, 4, 1500, 128), (2, 8, 8, 1280, 64), (2, 8, 8, 1500, 64),
                     (2, 8, 8, 1500, 32), (1, 4, 4, 1600, 32), (2, 16, 16, 2000, 128), (1, 8, 8, 6000, 128)],
            FAR_AND_NEAR: [(8, 16, 16, 16384, 128), (1, 32, 8, 65000, 128), (8, 8, 8, 3000, 64), (2, 16, 16, 4000, 128)]}
    for name, shapes in want.items():
        rows = [decode(*s) for s in shapes]
        assert [kind(r, g) for r, g in zip(rows, ask(rows))] == [name] * len(rows), name
    for T, d in ((513, 128), (1025, 64), (1281, 32)):                        # test_gpu_exhausted.py, test_decode
        rows = [decode(1, 34, 2, T - 1, d), decode(1, 34, 2, T, d)]
        assert [kind(r, g) for r, g in zip(rows, ask(rows))] == [ONE, SPREAD]
    rows = [decode(B, H, Hkv, T, d, True) for B, H, Hkv, T, d in ((5, 30, 10, 588, 64), (5, 30, 10, 1000, 64), (2, 8, 8, 1000, 32), (2, 16, 16, 4000, 128))]
    assert all(kind(r, g) == SPREAD for r, g in zip(rows, ask(rows)))


def test_decode_of_many_heads(ask):
    """Larger caches: one workgroup a head up to 2048 keys at d = 32, and at d = 64 where the heads are most of a round of the chip; spread
    up to 45 MB beyond.  With m every key is taken by the second launch from 1537 keys on."""
    want = {ONE: [(16, 16, 16, 2048, 32), (32, 16, 16, 2048, 32), (24, 24, 8, 1600, 32), (16, 16, 16, 2048, 64), (24, 24, 8, 2048, 64), (16, 16, 16, 1536, 128)],
            SPREAD: [(6, 20, 20, 2048, 32), (6, 20, 20, 2560, 32), (4, 16, 16, 2560, 64), (2, 16, 16, 2500, 128)],
            FAR_AND_NEAR: [(16, 16, 16, 2049, 32), (33, 16, 16, 2048, 32), (16, 16, 16, 2049, 64), (12, 12, 12, 2000, 64), (17, 16, 16, 2000, 64), (16, 16, 16, 1537, 128),
                           (4, 16, 16, 2800, 64)]}
    for name, shapes in want.items():
        rows = [decode(*s) for s in shapes]
        assert [kind(r, g) for r, g in zip(rows, ask(rows))] == [name] * len(rows), name
    rows = [decode(*s, True) for s in ((16, 16, 16, 1537, 32), (16, 16, 16, 2048, 64))]
    assert all(kind(r, g) == SPREAD for r, g in zip(rows, ask(rows)))


def test_decode_chunks_cover_the_keys_and_fit(ask):
    rng = random.Random(5)
    rows = []
    for _ in range(2000):
        Hkv, T = rng.randrange(1, 33), round(2 ** rng.uniform(0, 19))
        rows.append(decode(rng.randrange(1, 33), Hkv * rng.choice((1, 2, 3, 17)), Hkv, T, rng.choice((32, 64, 128)), rng.random() < 0.5))
    for row, (near, C, nfar, room) in zip(rows, ask(rows)):
        T = row[3]
        assert near + C * nfar >= T and near + C * (nfar - 1) < T and nfar <= 127, row
        assert nfar == 0 or nfar + (near > 0) <= room, row


def test_parts_of_grouped_heads(ask):
    """test_gpu_parts.py; and no parts without groups, a divisor of the group's heads, with sums that stay below 210 MB."""
    import test_gpu_parts as t
    rows = [(B, H, Hkv, T, d, 8 if lens is None else 9, 0 if lens is None else sum(lens)) for B, H, Hkv, T, d, lens, *_ in t.SHAPES]
    for shape, got in zip(t.SHAPES, ask(rows)):
        assert (KEYS[got[0]],) + got[1:] == shape[6:], shape
    rng = random.Random(11)
    rows = []
    for _ in range(3000):
        G, Hkv, B, T = rng.choice((1, 2, 3, 4, 5, 6, 8, 12, 16)), rng.randrange(1, 40), rng.randrange(1, 40), int(2 ** rng.uniform(0, 14))
        rows.append((B, G * Hkv, Hkv, T, rng.choice((32, 64, 128)), *((8, 0) if rng.random() < 0.5 else (9, max(T, rng.randrange(1, T * B + 1))))))
    for row, (keys, parts, beyond) in zip(rows, ask(rows)):
        B, H, Hkv, T, d, packed, Ttot = row
        assert parts == 1 or (H // Hkv) % parts == 0 and parts * Hkv * (Ttot or B * T) * d * 8 <= 211e6, row


def test_memory_of_parts_is_bounded(ask):
    """What sb_attn.h says of the larger workspace, 210 MB more at most with counts and rounding, for batches of many sequences and lengths that differ by far too."""
    from paper_2410_17980_amd import binding as sb
    rng = random.Random(21)
    log = lambda lo, hi: int(math.exp(rng.uniform(math.log(lo), math.log(hi))))
    rows = [(272, 16, 1, 8004, 32, 154768), (113, 8, 1, 8049, 64, 61811)]
    while len(rows) < 20000:
        G, Hkv, n, T = rng.choice((2, 3, 4, 6, 8, 16)), log(1, 33), log(1, 1001), log(32, 16385)
        rows.append((n, G * Hkv, Hkv, T, rng.choice((32, 64, 128)), max(T, int(n * T * math.exp(rng.uniform(-math.log(100), 0.0))))))
    for B, H, Hkv, T, d, Ttot in rows:
        for more in (sb.sb_attn_varlen_bwd_gqa_workspace_bytes(B, H, Hkv, Ttot, T, d) - sb.sb_attn_varlen_bwd_workspace_bytes(B, H, Ttot, T, d),
                     sb.sb_attn_bwd_gqa_workspace_bytes(B, H, Hkv, T, d) - sb.sb_attn_bwd_workspace_bytes(B, H, T, d)):
            assert 0 < more <= 210e6, (B, H, Hkv, T, d, Ttot, more)


def test_equal_lengths_take_the_plan_of_the_batched_call(ask):
    rng = random.Random(12)
    shapes = [(rng.randrange(1, 9), rng.randrange(2, 9), rng.randrange(1, 12), rng.randrange(1, 4200), rng.choice((32, 64, 128))) for _ in range(600)]
    batched = ask([(B, G * H, H, T, d, 8, 0) for B, G, H, T, d in shapes])
    for shape, a, b in zip(shapes, batched, ask([(B, G * H, H, T, d, 9, B * T) for B, G, H, T, d in shapes])):
        assert a[1:] == b[1:] and (KEYS[a[0]] == "strips") == (KEYS[b[0]] == "strips"), shape
