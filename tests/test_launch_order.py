"""The order in which a launch hands its blocks to workgroups (csrc/sb_share.h), compiled for the host:
every block once, neighbouring blocks of a head on one XCD, costly heads spread over the XCDs."""
import itertools
import os
import random
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2410_17980_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

MAIN = r"""
#include <stdio.h>
#include "sb_share.h"
int main(int argc, char** argv)
{
    int heads, nblk, pairs, d, backward;                         // d: of the forward and the query-stationary pass, or 0
    while (scanf("%d %d %d %d %d", &heads, &nblk, &pairs, &d, &backward) == 5) {
        if (pairs == 2) {                                        // fp32 forward
            const int run = sb::f32_run(heads, nblk, 16 * nblk, d), grid = run == sb::EIGHTHS ? (heads * nblk + 7) / 8 * 8 : heads * nblk;
            printf("%d %d\n", grid, run);
            for (int wg = 0; wg < grid; ++wg) {
                const sb::Share s = run == sb::EIGHTHS ? sb::share_in_eighths(wg, heads, nblk) : sb::share_of(wg, heads, run);
                printf("%d %d\n", s.bh, s.i);
            }
            continue;
        }
        const int grid = (int)sb::share_grid(heads, nblk, pairs), run = d ? sb::query_run(heads, nblk, d, backward) : sb::share_run(heads, nblk);
        printf("%d %d\n", grid, run);
        for (int wg = 0; wg < grid; ++wg) {
            const sb::Share s = pairs ? sb::share_in_pairs(wg, nblk) : sb::share_of(wg, heads, run);
            printf("%d %d\n", s.bh, s.i);
        }
    }
}
"""


@pytest.fixture(scope="module")
def order(tmp_path_factory):
    if not shutil.which(HIPCC):
        pytest.skip("no hipcc")
    tmp = tmp_path_factory.mktemp("order")
    (tmp / "main.hip").write_text(MAIN)
    subprocess.run([HIPCC, "-std=c++17", "-O1", "--offload-host-only", f"-I{CSRC}", "main.hip", "-o", "main"],
                   cwd=tmp, check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)

    def get(heads, nblk, pairs=False, d=0, backward=False):
        out = subprocess.run([str(tmp / "main")], input=f"{heads} {nblk} {int(pairs)} {d} {int(backward)}\n", text=True, check=True,
                             stdout=subprocess.PIPE).stdout.split()
        grid, run = int(out[0]), int(out[1])
        return np.array(out[2:], dtype=np.int64).reshape(grid, 2), 1 << run if run >= 0 else 0
    return get


SHAPES = [(h, n) for h, n in itertools.product((1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 24, 30, 32, 40, 63, 64, 65, 67, 72, 96, 128, 130, 512),
                                               (1, 2, 3, 4, 12, 16, 31, 32, 33, 64, 128)) if h * n <= 16384]


def test_every_block_once(order):
    for heads, nblk in SHAPES:
        got, _ = order(heads, nblk)
        assert sorted(map(tuple, got)) == [(h, i) for h in range(heads) for i in range(nblk)], (heads, nblk)
        assert np.all(np.diff(got[:, 1]) >= 0), "the longest blocks first"
        pairs, _ = order(heads, nblk, True)
        pairs = pairs[pairs[:, 0] < heads]
        assert sorted(map(tuple, pairs)) == [(h, i) for h in range(heads) for i in range((nblk + 1) // 2)], (heads, nblk)


def xcds(order, heads, nblk):
    got, run = order(heads, nblk)
    x = np.empty((heads, nblk), dtype=np.int64)
    x[got[:, 0], got[:, 1]] = np.arange(len(got)) % 8
    return x, run


@pytest.mark.parametrize("heads,nblk,run", [(128, 32, 2), (64, 32, 2), (256, 64, 2), (64, 128, 4), (32, 128, 4), (24, 128, 4), (40, 64, 2)])
def test_neighbouring_blocks_share_an_xcd(order, heads, nblk, run):
    """Launches several rounds deep: a head moves to another XCD after a run of blocks only."""
    x, got = xcds(order, heads, nblk)
    assert got == run
    assert (x[:, 1:] == x[:, :-1])[:, np.arange(1, nblk) % run != 0].all()


@pytest.mark.parametrize("heads,nblk", [(9, 83), (8, 128), (12, 128), (30, 64), (95, 25), (96, 31), (65, 64), (512, 8), (40, 63)])
def test_small_or_short_launches_turn_with_every_block(order, heads, nblk):
    x, got = xcds(order, heads, nblk)
    assert got == 0
    assert (x[:, 1:] != x[:, :-1]).mean() >= 0.8


def test_few_heads_meet_every_xcd(order):
    """Also one head alone keeps all XCDs busy."""
    for heads in range(1, 9):
        x, _ = xcds(order, heads, 128)
        for h in range(heads):
            assert np.bincount(x[h], minlength=8).max() <= 24, (heads, h)


def test_costly_heads_are_spread(order):
    """Half of the heads of a layer reach far, the same ones in every batch entry (as in a real model),
    the rest costs next to nothing: no XCD gets more than 1.35 times its share of the causal cost."""
    rng = random.Random(1)
    for B, H, nblk in ((8, 16, 32), (1, 32, 128), (8, 16, 16), (2, 32, 64), (4, 32, 32), (16, 32, 8)):
        worst = []
        for _ in range(40):
            far = np.array([rng.random() < 0.5 for _ in range(H)])
            if far.sum() < 8:
                continue
            x, _ = xcds(order, B * H, nblk)
            cost = np.repeat(np.tile(far, B)[:, None], nblk, 1) * np.arange(nblk, 0, -1)
            load = np.array([cost[x == c].sum() for c in range(8)])
            worst.append(load.max() / load.mean())
        assert np.mean(worst) <= 1.35, (B, H, nblk, np.mean(worst))


@pytest.mark.parametrize("heads,nblk,d,run", [(128, 16, 64, 2), (96, 8, 128, 2), (96, 7, 128, 0), (128, 16, 32, 0), (48, 32, 64, 4), (32, 32, 32, 4), (32, 32, 128, 2),
                                              (24, 47, 128, 4), (40, 20, 64, 2), (24, 31, 64, 0), (24, 32, 64, 4), (24, 64, 128, 2), (24, 64, 64, 4), (32, 128, 128, 4)])
def test_runs_of_the_forward(order, heads, nblk, d, run):
    """Every block once, the longest first, a head's blocks on one XCD for a run and on all eight over the launch."""
    got, r = order(heads, nblk, d=d)
    assert r == run
    assert sorted(map(tuple, got)) == [(h, i) for h in range(heads) for i in range(nblk)]
    assert np.all(np.diff(got[:, 1]) >= 0)
    x = np.empty((heads, nblk), dtype=np.int64)
    x[got[:, 0], got[:, 1]] = np.arange(len(got)) % 8
    for i in range(nblk - 1 if run else 0):
        assert np.array_equal(x[:, i] == x[:, i + 1], np.full(heads, (i + 1) % run != 0)), i
    if nblk >= 8 * max(run, 1):
        assert all(len(set(x[h])) == 8 for h in range(heads))


def test_runs_of_middling_head_counts(order):
    """d = 64, query-stationary pass: not from 64 heads on until there are 128; otherwise as the forward."""
    runs = lambda **k: [h for h in range(64, 200, 8) if order(h, 20, **k)[1] > 1]
    assert runs(d=64, backward=True) == list(range(128, 200, 8))
    assert runs(d=64) == runs(d=128) == runs(d=128, backward=True) == list(range(64, 200, 8))
    for d, nblk in ((32, 24), (64, 24), (128, 40)):
        assert all(order(h, nblk, d=d)[1] == order(h, nblk, d=d, backward=True)[1] > 1 for h in (32, 40, 48, 56))


@pytest.mark.parametrize("heads,nblk,d,eighths", [(1, 1, 32, True), (3, 5, 64, True), (28, 8, 128, True), (8, 33, 64, True), (12, 22, 128, True), (7, 30, 128, True),
                                                  (5, 53, 64, False), (8, 34, 128, False), (10, 120, 128, False), (16, 128, 128, False), (18, 76, 128, True), (28, 109, 64, True)])
def test_orders_of_the_fp32_forward(order, heads, nblk, d, eighths):
    """Every block once; in eighths an XCD's blocks lie side by side in the list of all heads' blocks, otherwise the longest come first."""
    got, _ = order(heads, nblk, pairs=2, d=d)
    there = got[:, 0] < heads
    assert sorted(map(tuple, got[there])) == [(h, i) for h in range(heads) for i in range(nblk)]
    if eighths:
        at, xcd = got[:, 0] * nblk + got[:, 1], np.arange(len(got)) % 8
        assert all(np.all(np.diff(at[there & (xcd == x)]) == 1) for x in range(8))
    else:
        assert there.all() and np.all(np.diff(got[:, 1]) >= 0)
