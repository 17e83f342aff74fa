"""Which kernels a call takes (csrc/sb_share.h, csrc/sb_split.h), compiled for the host: the rules' edges, and the routes that the GPU
tests name for their shapes."""
import os
import random
import shutil
import subprocess

import pytest

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
        const long mean = mean_length(B, T, packed, Ttot);
        printf("%d %d %d %ld %d %d\n", small_fwd_grid(pieces(B, H, T, 32, packed, Ttot), T, mean, d),
               small_grid(pieces(B, H, T, 32, packed, Ttot), T, mean, d),
               small_grid(pieces(B, Hkv, T, 32, packed, Ttot), T, mean, d),
               packed ? H * packed_places(B, Ttot) : (long)B * H * ((T + 31) / 32),
               take_in_turn(pieces(B, Hkv, T, 128, packed, Ttot), (T + 127) / 128, packed, mean, (long)B * Hkv * ((T + 127) / 128)),
               pieces(B, Hkv, T, 128, packed, Ttot) <= small_kv_grid((T + 127) / 128));
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
        assert strips <= got[3] <= strips + row[0] * row[1]


def test_short_sequences_keep_the_blocks(ask):
    """64 sequences of 32 rows: a strip a workgroup is slower, whatever max_T says."""
    for H, d, max_T in ((4, 64, 65), (4, 64, 512), (4, 64, 2048), (4, 32, 2048), (8, 128, 512)):
        assert ask([packed([32] * 64, H, d, max_T)])[0][:3] == (0, 0, 0), (H, d, max_T)
    assert ask([packed([70] * 100, 1, 64, 400)])[0][:3] == (0, 0, 0)
    # one of 600 rows among short ones, a place on the chip for every strip; and ordinary lengths, loose max_T
    assert ask([packed([600] + [20] * 30, 2, 128)])[0][:3] == (1, 1, 1)
    for max_T in (100, 300, 1300):
        assert ask([packed([100] * 13, 4, 64, max_T)])[0][:3] == (1, 1, 1)


def test_equal_lengths_take_the_route_of_the_batched_call(ask):
    rng = random.Random(4)
    shapes = [(rng.randrange(1, 9), rng.randrange(1, 25), rng.randrange(1, 4200), rng.choice((32, 64, 128))) for _ in range(400)]
    batched = ask([(B, H, H, T, d, 0, 0) for B, H, T, d in shapes])
    for shape, a, b in zip(shapes, batched, ask([(B, H, H, T, d, 1, B * T) for B, H, T, d in shapes])):
        assert a[:3] == b[:3], shape


def test_shapes_of_the_gpu_tests(ask):
    """test_gpu_small_grids.py, test_packed_places: one strip a workgroup (the forward at d = 32 only beyond 320 rows)."""
    for lens, H, Hkv, max_T in (([0] * 3 + [1, 33] * 32 + [0, 300, 31], 2, 2, 300), ([2, 0, 34] * 21 + [1, 400] + [0] * 70, 1, 1, 400),
                                ([100] * 13, 4, 2, 1300)):
        for d in (32, 64, 128):
            assert ask([packed(lens, H, d, max_T, Hkv)])[0][:3] == (d > 32 or max_T > 320, 1, 1), (lens, d)


def test_two_wave_groups(ask):
    """Key-stationary pass at d <= 64: two groups only where neither near heads nor far ones lose more than a mix gains."""
    for B, H, T, two in ((1, 8, 4096, 1), (2, 24, 1024, 1), (1, 16, 4096, 1), (1, 32, 2011, 1), (8, 16, 512, 0), (1, 40, 2048, 0), (1, 24, 4096, 0),
                         (1, 30, 3500, 0), (1, 32, 4096, 0), (8, 16, 2048, 0)):
        assert ask([(B, H, H, T, 64, 0, 0)])[0][4] == two, (B, H, T)
    for lens, H, max_T, two in (([5000] + [300] * 10, 4, None, 1), ([4200] + [800] * 3, 8, None, 0), ([32] * 64, 4, 2048, 0), ([32] * 64, 4, 512, 0)):
        assert ask([packed(lens, H, 64, max_T)])[0][4] == two, (H, max_T)


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
    rows = [decode(B, H, Hkv, T, d, True) for B, H, Hkv, T, d in ((5, 30, 10, 588, 64), (5, 30, 10, 1000, 64), (2, 8, 8, 1000, 32), (2, 16, 16, 4000, 128))]
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
