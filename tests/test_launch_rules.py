"""The rules that choose a launch by sizes (lbm_plan.h), on the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not found")
    exe = str(tmp_path_factory.mktemp("rules") / "launch_rules")
    subprocess.run(["g++", "-std=c++20", "-O1", "-Wall", "-fsanitize=undefined",
                    "-fno-sanitize-recover=all", "-I",
                    os.path.join(ROOT, "paper_2212_07494_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "launch_rules.cpp"), "-o", exe], check=True)

    def run(queries):
        text = "\n".join(" ".join(str(v) for v in q) for q in queries) + "\n"
        r = subprocess.run([exe], input=text, capture_output=True, text=True, check=True)
        return [[int(v) for v in line.split()] for line in r.stdout.splitlines()]

    return run


# nwaves, groups, longest group, Q, nx, rows
@pytest.mark.parametrize("query,by_node", [
    ((1, 1, 1, 27, 1, 10 ** 6), 1), ((185, 1, 185, 27, 1, 10 ** 6), 1),
    ((9, 5, 4, 19, 16, 62500), 1), ((185, 9, 42, 27, 128, 16384), 0),
    ((185, 9, 42, 27, 32, 62500), 0), ((1, 1, 1, 27, 128, 16384), 1),
    ((0, 0, 0, 9, 64, 32), 1),
    # the rows' launch would pass 2^32 threads: 2^26 rows
    ((10 ** 4, 16, 700, 39, 31, 1 << 26), 1), ((10 ** 4, 16, 700, 39, 31, 1 << 25), 0)])
def test_waves_by_node(ask, query, by_node):
    assert ask([("waves_by_node", *query)]) == [[by_node]]


LDS, NCU = 160 * 1024, 256


def test_plan_covers_the_lattice_within_a_launch(ask):
    """Tiles cover every node once and none is empty, margins leave room in a tile's columns,
    the LDS holds it, and a launch stays below 2^32 threads (512 a tile)."""
    sizes = [1, 2, 3, 5, 11, 12, 14, 27, 28, 32, 33, 53, 57, 64, 65, 113, 200, 1000, 65535]
    cases = [(nx, ny, wy, elem) for nx in sizes + [1 << 20, 5 * 10 ** 8, 10 ** 9, 2 ** 31 - 1] for ny in sizes
             for wy in (0, 1) for elem in (2, 4, 8) if nx * ny < 2 ** 31]
    got = ask([("multi_plan", *c, LDS, LDS, NCU) for c in cases])
    assert len(got) == len(cases)
    for (nx, ny, wy, elem), (K, wx, ox, oy, ntx, nty, lds) in zip(cases, got):
        if not K:
            continue
        what = (nx, ny, wy, elem)
        assert K in (3, 5, 7) and (wy or ny >= 2 * K - 2 or K == 3 and ny >= 3), what
        assert (ntx - 1) * ox < nx <= ntx * ox and (nty - 1) * oy < ny <= nty * oy, what
        assert ntx == 1 and nx <= wx or ox + 2 * (K - 1) <= wx, what
        assert lds == (oy + 2 * (K - 1)) * wx * 9 * elem <= LDS, what
        assert ntx * nty * 512 < 2 ** 32, what


@pytest.mark.parametrize("query,grid", [
    ((8, 256, 10 ** 6), 2048), ((0, 256, 1), 8), ((0, 256, 17), 24),
    ((0, 256, 2 ** 24 - 9), 2 ** 24 - 8), ((0, 256, 2 ** 24), 2 ** 24 - 8),
    ((0, 256, 2 ** 31 - 1), 2 ** 24 - 8)])
def test_batch_grid(ask, query, grid):
    assert ask([("batch_grid", *query)]) == [[grid]]


@pytest.mark.parametrize("n", [0, 1, 255, 256, 257, 2 ** 31 - 257, 2 ** 31 - 256, 2 ** 31 - 255,
                               2 ** 31 - 1])
def test_pieces(ask, n):
    """Tiles of up to 256 nodes of the largest domains: no sum passes 2^31."""
    count = -(-n // 256)
    start = max(0, count - 1) * 256
    assert ask([("pieces", n, 256)]) == [[count, start, n - start, count]]


@pytest.mark.parametrize("cu,block,most", [(LDS, 64 * 1024, 64 * 1024), (64 * 1024, LDS, 64 * 1024),
                                           (LDS, 4000, 0), (LDS, 0, 0), (LDS, -1, 0)])
def test_tiles_fit_a_workgroup(ask, cu, block, most):
    """The LDS of a tile is what one workgroup may take, not what a compute unit has."""
    (K, *_, lds), = ask([("multi_plan", 1024, 1024, 0, 8, cu, block, NCU)])
    assert lds <= most and (K > 0) == (most > 0)


def test_rows_plain(ask):
    """Without walls and solid nodes always; with them, where the offsets cost more."""
    for Q in (9, 19, 27, 39):
        for elem in (2, 4, 8):
            got = [v for v, in ask([("rows_plain", Q, elem, x, w) for x in (0, 1) for w in (0, 1)])]
            assert got[0] == 1
            assert got[1:] == ([0, 0, 0] if elem == 2 else [1, 0, 0] if Q == 27 else [1, 1, 1])


def _default(ask, cases):
    """(Q, bytes of a value, nx, ny, nz, walls across x, walls elsewhere)"""
    return ask([("default_launch", Q, e, nx, ny, 2 * Q * e * nx * ny * nz, x, w)
                for Q, e, nx, ny, nz, x, w in cases])


def test_default_launch_is_valid(ask):
    """A shape and variant that lbm_set_tuning takes; consecutive nodes on ragged widths only."""
    cases = [(Q, e, nx, ny, nz, x, w) for Q in (9, 19, 27, 39) for e in (2, 4, 8)
             for nx in (1, 3, 50, 64, 65, 126, 127, 128, 192, 256, 257, 1000, 4097, 65536, 2 ** 31 - 1)
             for ny in (1, 2, 3, 40, 500) for nz in ((1,) if Q == 9 else (1, 60, 500))
             for x in (0, 1) for w in (0, 1)]
    for c, (bx, by, v, linear) in zip(cases, _default(ask, cases)):
        assert bx in (64, 128, 256) and by >= 1 and bx * by <= 256 and 0 <= v < 12, c
        assert linear == (by == 3) and not (linear and c[2] % 64 == 0), c


@pytest.mark.parametrize("case,variants", [
    # no XCD placement: binary16 rows, walls across x, walled FP32 rows well within the cache
    ((19, 2, 128, 128, 128, 0, 0), (3,)), ((19, 2, 256, 128, 96, 1, 1), (3,)),
    ((19, 4, 64, 128, 64, 1, 1), (0,)), ((19, 4, 64, 128, 64, 0, 1), (0,)),
    ((27, 4, 64, 128, 64, 0, 0), (3,)), ((9, 8, 1000, 1, 1, 0, 0), (3,)),
    # consecutive nodes, D2Q9 and periodic rows within the cache
    ((19, 4, 100, 100, 100, 0, 0), (9,)), ((19, 8, 64, 64, 64, 0, 0), (9,)),
    ((9, 8, 1024, 1024, 1, 0, 0), (9,)),
    # non-temporal stores beyond it
    ((27, 8, 128, 128, 128, 0, 0), (4,)), ((19, 4, 256, 256, 256, 0, 0), (4,))])
def test_default_variant(ask, case, variants):
    assert _default(ask, [case])[0][2] in variants


def test_multi_rows(ask):
    """The rows that the stages compute, counted one by one (but for walls within a margin of a
    tile between the first and the last)."""
    cases = [(ny, oy, K, w) for ny in (1, 2, 5, 12, 27, 28, 60, 131) for oy in (1, 3, 7, 22, 27)
             for K in (3, 5, 7) for w in (0, 1) if -(-ny // oy) <= 4 or (oy >= K - 1 and (ny - 1) % oy >= K - 2)]
    want = []
    for ny, oy, K, w in cases:
        n = 0
        for y0 in range(0, ny, oy):
            y1 = min(y0 + oy, ny)
            for m in range(K):
                n += (min(ny, y1 + m) - max(0, y0 - m)) if w else y1 - y0 + 2 * m
        want.append([n])
    assert ask([("multi_rows", *c) for c in cases]) == want


@pytest.mark.parametrize("lattice,several", [
    ((64, 32, 1, 8), 1), ((50, 200, 1, 8), 1), ((32, 32, 0, 8), 1), ((1024, 1024, 0, 4), 1),
    ((2048, 2048, 0, 4), 1), ((65536, 3, 1, 8), 1), ((1, 5, 1, 8), 1),
    # low or narrow, where the tiles' rows leave lanes and wavefronts idle
    ((1, 65535, 0, 8), 0), ((8, 16384, 1, 8), 0), ((12, 65535, 0, 4), 0),
    ((2097152, 1, 1, 4), 0), ((1048576, 1, 1, 8), 0), ((524288, 1, 1, 4), 0)])
def test_lattices_that_take_several_steps(ask, lattice, several):
    (K, *_), = ask([("multi_plan", *lattice, LDS, LDS, NCU)])
    assert (K > 0) == bool(several)


# bytes, steps, tiles, rows of a launch, blocks of 256 nodes, nodes
@pytest.mark.parametrize("batch,several", [
    ((8, 5, 2196, 340380, 11712, 2998272), 1),    # 732 domains of 64 x 64
    ((8, 5, 24000, 3480000, 9000, 1800000), 0),   # 3000 of 3 x 200
    ((8, 5, 3000, 300000, 3000, 768000), 0),      # 3000 of 16 x 16
    ((8, 3, 3000, 45000, 3000, 27000), 0),        # 3000 of 3 x 3
    ((4, 5, 117, 11700, 117, 29952), 1)])         # 117 of 16 x 16
def test_batches_that_take_several_steps(ask, batch, several):
    assert ask([("batch_pays", *batch, NCU)]) == [[several]]
