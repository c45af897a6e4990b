"""The block table of the layer-parallel column solves: every column once, in blocks
that fit, and an even share of every depth for each of the 8 parts that the kernel
gives to the XCDs."""

import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "column_blocks_table")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-fsanitize=address,undefined", "-I",
                    os.path.join(ROOT, "paper_2605_16082_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "column_blocks_table.cpp"), "-o", exe], check=True)
    return exe


def _table(program, n_cols, depth):
    out = subprocess.run([program], input=f"64 {n_cols}\n" + "\n".join(map(str, depth)), check=True,
                         capture_output=True, text=True).stdout.split()
    return int(out[0]), np.array(out[1:], dtype=int).reshape(-1, 3)


def _parts(n):
    """First block of each XCD's part (xcd_tile of the kernels), and the end."""
    return np.concatenate([[0], np.cumsum([n // 8 + (x < n % 8) for x in range(8)])])


def _depths(kind, n):
    rng = np.random.default_rng(n)
    x = np.linspace(0.0, 6.0, n)
    return {"one": np.full(n, 30), "smooth": np.rint(32.5 + 27.5 * np.sin(x)).astype(int),
            "noise": rng.integers(1, 65, n), "shallow": np.rint(2.5 + 1.5 * np.sin(x)).astype(int),
            "one deep": np.where(np.arange(n) == n // 2, 64, 3)}[kind]


KINDS = ["one", "smooth", "noise", "shallow", "one deep"]


@pytest.mark.parametrize("n", [1, 2, 7, 9, 64, 353, 1067])
@pytest.mark.parametrize("kind", KINDS)
def test_every_column_once(program, kind, n):
    depth = _depths(kind, n)
    n_cols = 64 * n - 23
    max_np, t = _table(program, n_cols, depth)
    cols = np.concatenate([c + np.arange(1 << g) for c, _, g in t])
    assert np.array_equal(np.sort(cols[cols < n_cols]), np.arange(n_cols))
    assert len(np.unique(cols)) == len(cols) and cols.max() < 64 * n
    assert np.array_equal(t[:, 1], depth[t[:, 0] // 64])
    prisms = t[:, 1] << t[:, 2]
    assert prisms.max() == max_np <= 256
    assert ((t[:, 2] == 6) | (2 * prisms > 256)).all() and (t[:, 2] >= 2).all()
    if kind == "one":
        assert np.array_equal(t[:, 0], np.sort(t[:, 0]))


@pytest.mark.parametrize("n", [353, 1067])
@pytest.mark.parametrize("kind", ["smooth", "noise", "shallow"])
def test_parts_get_an_even_share(program, kind, n):
    depth = _depths(kind, n)
    _, t = _table(program, 64 * n, depth)
    p = _parts(len(t))
    share = [(np.sum(b[:, 1] << b[:, 2]), b[:, 1].sum()) for b in (t[p[x]:p[x + 1]] for x in range(8))]
    for v in np.array(share).T:                   # prisms; layers of the serial chains
        assert v.max() <= 1.06 * v.min(), v       # dealt in cells: two of a part's 44 or more
    # a cell's groups stay together, but for those that even out the parts' lengths
    cell = t[:, 0] // 64
    part = np.searchsorted(p, np.arange(len(t)), side="right")
    assert sum(len(np.unique(part[cell == k])) > 1 for k in range(n)) <= 16
