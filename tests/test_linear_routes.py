"""Which kernel takes a matrix-core linear, on the host: the dispatch over all
shapes that the entry points accept, and the launch plans' bounds."""
import random

import pytest

from routes import group_quad_wave, route, split_plan, stream_plan

LDS = 160 * 1024


def _shapes(n, seed):
    r = random.Random(seed)
    for _ in range(n):
        bits, M = r.choice([3, 4]), r.randint(2, 16)
        N = int(2 ** r.uniform(0, 24))
        if r.random() < 0.2:
            N = 16 * r.choice([255, 256, 257, 1023, 1024, 1025, 3071, 3072])
        yield bits, M, N, r.randint(1, 64) if r.random() < 0.5 else int(2 ** r.uniform(6, 10.5))


def test_routes_are_consistent():
    """Every route only where its kernel takes the shape."""
    seen = set()
    for bits, M, N, G in _shapes(40000, 1):
        tiles, nq = (N + 15) // 16, (G + 3) // 4
        MT = 4 if M <= 4 else 8 if M <= 8 else 16
        plain, ws = route(bits, M, N, 128 * G), route(bits, M, N, 128 * G, True)
        seen |= {plain, ws}
        assert plain not in ("split", "split_stream")
        sp = split_plan(M, N, G)
        if sp.S == 1:
            assert ws == plain
        for r in (plain, ws):
            case = (r, bits, M, N, G)
            if r == "stream":
                assert nq <= 16 and stream_plan(bits, M, N, G, 1).W > 0, case
            elif r == "share":
                assert nq <= 5 and M > 4 and nq * MT * 1024 * 2 <= LDS, case
            elif r.startswith("quad_wave"):
                unit = nq * (bits * 1024 + 512) if r == "quad_wave_codes" else 0
                assert nq <= 10 and nq * MT * 1024 + unit <= LDS, case
                assert r != "quad_wave_regs" or M <= 8, case
                assert r != "quad_wave_codes" or tiles <= 256 * (LDS // (nq * MT * 1024 + unit)), case
            elif r in ("walk4", "walk8"):
                assert tiles >= (3072 if r == "walk8" else 1024), case
            elif r in ("split", "split_stream"):
                assert sp.S > 1 and 1 <= sp.qs <= 5 and sp.S * sp.qs >= nq, case
                if r == "split_stream":
                    st = stream_plan(bits, M, N, G, (nq + 15) // 16)
                    assert st.W > 0 and st.ranges <= sp.S, case
            else:
                assert nq > 10 and tiles < 1024 and (r == "one_tile_codes" or tiles > 256), case
    assert len(seen) == 11, seen


def test_stream_plans_in_bounds():
    """Blocks, waves, ring stages and every LDS use of a plan: activation slabs,
    ring, partials and the reads of eight partials past the last quad."""
    n = 0
    for bits, M, N, G in _shapes(40000, 2):
        nq_all = (G + 3) // 4
        ranges = 1 if nq_all <= 16 else (nq_all + 15) // 16
        if ranges > 16:
            continue
        p = stream_plan(bits, M, N, G, ranges)
        if p.W == 0:
            continue
        n += 1
        case = (bits, M, N, G, ranges)
        unit, PB, W = bits * 1024 + 512, 16 * {4: 16, 8: 32, 16: 64}[p.MT], p.W
        groups = ((N + 15) // 16 + p.TS - 1) // p.TS
        assert p.MT >= M and W == p.TS * p.nq and 1 <= W <= 16, case
        assert p.nb in (1, 2) and 1 <= p.nblocks * p.ranges <= 256 and p.nblocks <= groups, case
        assert p.ranges * p.nq >= nq_all and (p.ranges - 1) * p.nq < nq_all and p.ranges <= ranges, case
        assert ranges == 1 or p.nq % 2 == 0, case
        iters = -(-groups // p.nblocks)
        assert 1 <= p.D <= 4 and p.D <= iters and (iters == 1 or p.D >= 2), case
        slabs = W * unit + p.nq * p.MT * p.PH * 256
        ring = p.D * W * unit + p.nb * W * PB
        reads = p.D * W * unit + (p.nb - 1) * W * PB + ((p.TS - 1) * p.nq + max(0, p.nq - 8) + 8) * PB
        assert max(slabs, ring, reads) <= p.lds <= LDS, case
        assert (p.TS == 1 or p.PH == 4) and (p.MT, p.PH) in {(16, 4), (16, 2), (16, 1), (8, 4), (8, 2), (4, 4)}, case
    assert n > 20000


# (bits, M, N, K, workspace) -> kernel: shapes next to the measured lines, on
# both sides.
LINES = [
    ((3, 8, 20480, 2560), "share"), ((3, 8, 49152, 2560), "stream"), ((4, 8, 20480, 2560), "quad_wave_regs"),
    ((3, 8, 20000, 3200), "quad_wave_regs"), ((4, 8, 30000, 3584), "stream"), ((3, 8, 10944, 4608), "quad_wave_regs"),
    ((3, 8, 24576, 4096), "stream"), ((3, 8, 12288, 4096), "quad_wave_regs"), ((3, 4, 21856, 4608), "quad_wave_regs"),
    ((3, 4, 24592, 4096), "stream"), ((3, 4, 37456, 3584), "quad_wave_regs"), ((4, 4, 37456, 3584), "stream"),
    ((3, 16, 16384, 3584), "walk4"), ((3, 16, 16368, 3584), "stream"), ((3, 16, 16384, 4096), "walk4"),
    ((4, 16, 16384, 4096), "stream"), ((3, 16, 16384, 8192), "stream"), ((4, 16, 49152, 2176), "share"),
    ((4, 16, 49152, 2560), "stream"), ((3, 8, 4096, 8192), "one_tile_codes"), ((3, 8, 4112, 8192), "stream"),
    ((3, 16, 656, 25600, True), "split"), ((3, 8, 656, 25600, True), "split_stream"),
    ((3, 16, 1120, 25600, True), "split"), ((3, 16, 5120, 25600, True), "split_stream"),
    ((3, 16, 5120, 25600), "two_tiles"), ((3, 9, 536, 768), "quad_wave"), ((4, 9, 536, 768), "quad_wave_codes"),
    ((4, 4, 1280, 512), "quad_wave"), ((4, 4, 1280, 640), "quad_wave_codes"),
    ((4, 3, 8192, 2304), "quad_wave_codes"), ((4, 3, 8208, 2304), "quad_wave"), ((4, 3, 12288, 3072), "quad_wave_codes"),
    ((3, 4, 2560, 4096), "quad_wave_codes"),
    ((3, 9, 32768, 4608), "walk4"), ((3, 9, 32784, 4608), "stream"), ((3, 8, 29600, 5632), "walk4"),
    ((3, 16, 28672, 6656), "stream"), ((3, 16, 28688, 6656), "walk4"), ((3, 16, 28688, 6528), "stream"),
    # codes in LDS, eight waves above M = 8: one block on a compute unit
    ((3, 9, 4096, 5376), "one_tile_codes"), ((3, 9, 4112, 5376), "two_tiles"),
    # 11 to 16 quads: up to 512 tiles, to 768, below 1024
    ((3, 10, 8192, 5376), "two_tiles"), ((3, 12, 5376, 7680), "two_tiles"), ((4, 9, 8192, 7680), "two_tiles"),
    ((3, 9, 8192, 8192), "stream"), ((3, 9, 8192, 7168), "two_tiles"), ((4, 9, 8192, 7168), "stream"),
    ((3, 8, 8192, 7680), "two_tiles"), ((4, 8, 8192, 7680), "stream"), ((3, 8, 8192, 7040), "stream"),
    ((3, 10, 8208, 5376), "stream"), ((3, 5, 12288, 5504), "stream"), ((3, 5, 12304, 5504), "two_tiles"),
    ((3, 3, 15104, 6528), "two_tiles"), ((3, 4, 15104, 7168), "stream"), ((3, 5, 15104, 7168), "two_tiles"),
    ((3, 5, 15104, 7680), "stream"), ((3, 10, 15104, 6528), "two_tiles"), ((3, 11, 15104, 6528), "stream"),
    ((4, 10, 15104, 5504), "two_tiles"), ((4, 11, 15104, 5504), "stream"), ((4, 8, 15104, 5504), "stream"),
]


@pytest.mark.parametrize("shape,kernel", LINES)
def test_measured_lines(shape, kernel):
    assert route(*shape) == kernel


# (M, tiles, quads of the longest row) -> form, on both sides of the lines.
GROUP_LINES = [
    ((4, 384, 5), 0), ((4, 1216, 5), 1), ((16, 1216, 5), 1), ((9, 1216, 5), -1), ((9, 512, 5), 0), ((9, 1216, 8), -1),
    ((9, 256, 8), 0), ((16, 1216, 8), 1), ((9, 320, 6), -1), ((14, 320, 6), 1), ((9, 1216, 2), -1), ((16, 1216, 2), 1),
    ((5, 1216, 8), -1), ((8, 1216, 8), 1), ((4, 256, 10), 0), ((4, 320, 10), 1), ((4, 3200, 10), -1), ((4, 4, 11), -1),
    ((9, 2400, 1), -1), ((16, 2400, 1), 1),
]


@pytest.mark.parametrize("shape,form", GROUP_LINES)
def test_group_lines(shape, form):
    assert group_quad_wave(*shape) == form
