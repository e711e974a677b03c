"""Which tiles the grouped GEMMs run, in which order, and the launches of a routing (CPU only;
tile_order.cpp compiles the library's own functions for the host).

The 256 x 256 tiles cover every output row and column exactly once: two workgroups that store the
same rows race, and fprop's K rotation follows the XCD block, so the bits that stay would depend on
timing.  The choice between them and the small tiles is the faster one at measured sizes, and so is
the number of launches that a routing takes.
"""

import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2511_02302_amd import build as ff8_build

SRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "tile_order.cpp")


@pytest.fixture(scope="module")
def host_lib(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("order") / "order.so")
    cmd = [ff8_build.hipcc()] + ff8_build.COMMON + ["-x", "hip", "--cuda-host-only", "-shared", SRC, "-o", lib]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return ctypes.CDLL(lib)


@pytest.fixture(scope="module")
def walk(host_lib):
    fn = host_lib.tile_order_walk
    fn.restype = ctypes.c_long
    fn.argtypes = [ctypes.c_int, ctypes.c_void_p] + [ctypes.c_int] * 4 + [ctypes.c_void_p, ctypes.c_long]

    def tiles(rows, n_pt, n_qt=0, cus=256):
        off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
        cap = 4 * (sum(-(-r // 256) for r in rows) + len(rows) * n_qt + 8) * n_pt
        out = np.empty((cap, 6), np.int32)
        n = fn(len(rows), off.ctypes.data, int(off[-1]), n_pt, n_qt, cus, out.ctypes.data, cap)
        assert n >= 0
        return off, out[:n]

    return tiles


def _routing(rng):
    """Rows per expert as a routing gives them: even or skewed, padded to 16 or 128, empty ones."""
    E = int(rng.integers(1, 130))
    mean = float(np.exp(rng.uniform(np.log(8), np.log(1500))))
    p = rng.permutation(np.arange(1, E + 1) ** -1.2) if rng.random() < 0.4 else np.ones(E)
    rows = rng.poisson(np.minimum(mean * E * p / p.sum(), 8000))
    rows[rng.random(E) < 0.1] = 0
    align = int(rng.choice([16, 128]))
    return ((rows + align - 1) // align * align).tolist()


def _check_rows(walk, rows, n_pt, cus=256):
    off, t = walk(rows, n_pt, cus=cus)
    e, q0, q1, p0 = t[:, 0], t[:, 1], t[:, 2], t[:, 3]
    assert np.all((off[e] <= q0) & (q0 < q1) & (q1 <= off[e + 1])), "rows of another group"
    assert np.all((p0 % 256 == 0) & (p0 < 256 * n_pt))
    bands = off[-1] // 16  # groups are multiples of 16 rows
    writes = np.zeros((bands + 1, n_pt), np.int64)  # +1 where a tile begins, -1 past its end
    assert np.all(q0 % 16 == 0) and np.all(q1 % 16 == 0)
    np.add.at(writes, (q0 // 16, p0 // 256), 1)
    np.add.at(writes, (q1 // 16, p0 // 256), -1)
    count = np.cumsum(writes, axis=0)[:bands]
    assert np.all(count == 1), f"{int((count > 1).sum())} bands written twice, {int((count == 0).sum())} never"


@pytest.mark.parametrize("n_pt", [1, 2, 3, 4, 5, 6, 8, 11, 16, 28, 87])
def test_row_tiles_cover_every_output_once(walk, n_pt):
    rng = np.random.default_rng(n_pt)
    for _ in range(60):
        _check_rows(walk, _routing(rng), n_pt, cus=int(rng.choice([256, 256, 128, 304])))


@pytest.mark.parametrize("rows,n_pt", [
    ([384] * 64, 11),          # 44 chunks: four left for the last sweep
    ([1024, 784, 512], 79),    # 25 chunks: one left
    ([272, 0, 16, 528, 256], 11), ([4096], 3), ([512] * 19, 7)])
def test_split_last_sweep_covers_every_output_once(walk, rows, n_pt):
    _check_rows(walk, rows, n_pt)
    off, t = walk(rows, n_pt)
    chunks = -(-sum(-(-r // 256) for r in rows) * n_pt // 32)
    last = t[t[:, 4] >= chunks // 8 * 8]
    assert 1 <= chunks % 8 <= 4 and len(last)
    # the last sweep's tiles are halves: no workgroup of it stores more than 128 rows
    assert np.all(last[:, 2] - last[:, 1] <= 128)


@pytest.mark.parametrize("n_pt,n_qt", [(1, 1), (3, 5), (4, 8), (11, 16), (16, 28), (28, 16)])
def test_wgrad_blocks_cover_every_tile_once(walk, n_pt, n_qt):
    rows = [128, 0, 1024, 16, 528]
    _, t = walk(rows, n_pt, n_qt)
    got = sorted(map(tuple, t[:, [0, 1, 3]].tolist()))
    assert got == [(e, 256 * q, 256 * p) for e in range(len(rows)) for q in range(n_qt) for p in range(n_pt)]


# Measured on one MI355X, operands in no cache: us with 256 x 256 tiles, us with the small ones.
FPROP, DGRAD, WGRAD = 0, 1, 2


@pytest.mark.parametrize("mode,E,M_cap,N,K,small", [
    (FPROP, 16, 16 * 384, 2048, 2048, 0),      # 34 / 40
    (FPROP, 16, 16 * 192, 2048, 2048, 128),    # 37 / 31
    (FPROP, 16, 16 * 256, 2048, 2048, 128),    # 40 / 32
    (FPROP, 8, 8 * 192, 4096, 7168, 128),      # 96 / 84
    (FPROP, 8, 8 * 256, 1024, 1024, 64),       # 24 / 12
    (DGRAD, 16, 16 * 192, 6912, 1024, 64),     # 88 / 52
    # up to 256 rows per group: at least one tile per expert
    (DGRAD, 64, 64 * 128, 2048, 1408, 128),    # 61 / 50
    (DGRAD, 64, 64 * 160, 2048, 1408, 128),    # 61 / 50, skewed 29 / 21
    (DGRAD, 32, 32 * 128, 4096, 7168, 0),      # 221 / 237
    (FPROP, 32, 32 * 144, 7168, 2048, 0),      # 121 / 138
    (FPROP, 30, 30 * 128, 7040, 256, 128),     # a step with these: 376 us / 364
    (FPROP, 60, 60 * 128, 2048, 3072, 128),    # 2 tokens x 6: 40 / 28
    (FPROP, 49, 49 * 128, 1792, 3456, 128),    # 9 tokens: 39 / 26
    (FPROP, 63, 15872, 1024, 1024, 128),       # 47 / 38
    (FPROP, 27, 4864, 3328, 4096, 128),        # 100 / 90
    (DGRAD, 30, 30 * 128, 1024, 5120, 0),      # one token x 7: 21 / 25
    (DGRAD, 47, 6272, 1024, 5120, 0),          # 67 tokens x 3, skewed: 21 / 25
    # a few rows per group
    (DGRAD, 28, 28 * 18, 4096, 2048, 64),      # 58 tokens: 43 / 26
    (DGRAD, 48, 48 * 16, 2560, 1280, 64),      # 4 tokens x 7: 34 / 21
    (DGRAD, 32, 32 * 16, 7168, 2048, 0),       # 95 / 101
    (DGRAD, 64, 64 * 16, 2048, 1408, 64),      # 56 / 40
    (FPROP, 32, 32 * 16, 7168, 2048, 64),      # 106 / 90
    (FPROP, 8, 8 * 96, 4096, 7168, 128),       # 80 / 57
    (WGRAD, 32, 32 * 768, 7168, 2048, 0),      # 583 / 613
    (WGRAD, 32, 24064, 7168, 2048, 0),         # 10000 tokens x 2: 561 / 610
    (WGRAD, 64, 64 * 768, 7168, 2048, 0),      # 1158 / 1229
    (WGRAD, 32, 32 * 512, 7168, 2048, 128),    # 509 / 512
    (WGRAD, 32, 32 * 384, 7168, 2048, 128),    # 467 / 436
    (WGRAD, 32, 32 * 640, 4096, 2560, 128),    # 414 / 407
    (WGRAD, 6, 19328, 1024, 1536, 128),        # 6408 tokens x 3, skewed: 77 / 60
    (WGRAD, 8, 8 * 4096, 640, 1024, 128),      # 60 / 44
    (WGRAD, 18, 20864, 2048, 128, 128),        # 2309 tokens x 8, skewed: 40 / 26
    (WGRAD, 64, 64 * 384, 2816, 2048, 128),    # 383 / 344
    (WGRAD, 64, 64 * 768, 2048, 1408, 128),    # 262 / 246
    (WGRAD, 16, 16 * 768, 2816, 2048, 128),    # 131 / 122
    (WGRAD, 32, 32 * 768, 4096, 7168, 128),    # 1212 / 1050
    (WGRAD, 11, 11136, 3072, 5632, 0),         # 1374 tokens x 7, skewed: 273 / 326
])
def test_tile_shape_choice(host_lib, mode, E, M_cap, N, K, small):
    args = [ctypes.c_int64(v) for v in (M_cap, N, K, 256)]
    assert host_lib.tile_rule(mode, E, *args) == small


@pytest.mark.parametrize("E,M_cap,N,K,wide", [
    (32, 32 * 512, 4096, 7168, True),    # 128 x 128 tiles 1024 us, 256 x 128 ones 920
    (16, 16 * 640, 2048, 2048, True),    # 82, 69
    (43, 21760, 2816, 256, False),       # skewed: 93, 148
    (15, 10496, 512, 3840, False),       # skewed: 77, 112
    (8, 8 * 512, 1024, 1024, False),     # 17, 19
    (28, 18304, 768, 384, False),        # skewed: 31, 46
    (35, 35 * 128, 512, 1792, False)])   # 19 tokens: 28, 30
def test_wgrad_small_tile_choice(host_lib, E, M_cap, N, K, wide):
    args = [ctypes.c_int64(v) for v in (N, K, 256)]
    assert host_lib.tile_rule(WGRAD, E, ctypes.c_int64(M_cap), *args) == 128
    assert host_lib.tile_rule_wide(E, *args) == wide


@pytest.mark.parametrize("rows,n_pt,packs", [
    ([512] * 16, 6, False),        # six chunks, or eight blocks: one sweep either way (37 us packed, 34 in blocks)
    ([448] * 16, 6, False),        # the same with halves of tiles (60, 56)
    ([512] * 64, 11, True),        # 44 chunks, five and a half sweeps, or 48 blocks, six
    ([1024] * 64, 6, True),        # 48 chunks, or 64 blocks
    ([384] * 4 + [256] * 9, 10, True)])  # 17 q tiles: six chunks, or nine blocks
def test_row_tiles_are_packed_where_it_saves_a_sweep(walk, rows, n_pt, packs):
    _, t = walk(rows, n_pt)
    spans = [len(set((t[t[:, 4] == b][:, 3] // 1024).tolist())) for b in set(t[:, 4].tolist())]
    assert (max(spans) > 1) == packs  # a block's tiles lie in four columns of tiles


@pytest.mark.parametrize("E,n_pt,n_qt,packs", [(8, 3, 4, False), (8, 6, 8, False), (64, 6, 8, True), (8, 9, 8, False)])
def test_wgrad_tiles_are_packed_where_it_saves_a_sweep(walk, E, n_pt, n_qt, packs):
    _, t = walk([1152] * E, n_pt, n_qt)
    spans = [len(set((t[t[:, 4] == b][:, 3] // 1024).tolist())) for b in set(t[:, 4].tolist())]
    assert (max(spans) > 1) == packs


@pytest.mark.parametrize("E,tq,per_cu", [(1, 64, 3), (360, 64, 3), (362, 64, 2), (1024, 64, 2), (1024, 128, 2)])
def test_small_tile_workgroups_fit_a_cu(host_lib, E, tq, per_cu):
    """Two stages of 128 + tq rows x 128 bytes, two scale batches, two tables of E + 1 entries."""
    lds = 2 * (128 + tq) * 128 + 2 * (256 + 16 * tq) + 8 * (E + 1)
    got = host_lib.tile_per_cu(3 if tq == 64 else 2, lds)
    assert got == per_cu and got * lds <= 160 * 1024


@pytest.mark.parametrize("T,k,E,align,launches", [
    (7, 1, 1024, 16, 1), (4096, 1, 1024, 128, 1), (512, 8, 8, 128, 1),
    (513, 8, 8, 128, 2), (16384, 8, 64, 128, 2), (4096, 8, 512, 16, 2),
    (8192, 1, 1024, 128, 2),            # two launches 50 us, three 94
    (8192, 1, 1024, 16, 3),             # 48, 35
    (8192, 2, 768, 16, 3),              # 41, 34
    (8192, 2, 512, 16, 3), (16384, 8, 256, 128, 3)])
def test_routing_launch_count(host_lib, T, k, E, align, launches):
    assert host_lib.route_launch_count(ctypes.c_int64(T), k, E, align) == launches
