"""GPU parity: the HIP kernels (through the C ABI) against the CPU oracle.

Quantize: packed words, scale bits and zero bytes bit-exact.
Linear:   each fp16 output is an fp16 rounding of a value within
          1e-3 x RMS of the oracle's exact fp64 result (oracle/compare.py).
Inputs are seeded (paper_2605_08755_amd.inputs); the linear is fed the
oracle's own quantization, so its parity does not depend on the quantize
kernel.
"""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from oracle.compare import linear_check
from paper_2605_08755_amd import inputs, laq
from routes import group_quad_wave, route, split_plan

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def say(*a):
    print("[gpu-case]", *a, flush=True)


def to_dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def gpu_quantize(w16, bits):
    q, s, z = laq.quantize(to_dev(w16), bits)
    torch.cuda.synchronize()
    return (q.cpu().numpy().view(np.uint32), s.cpu().numpy().view(np.uint16), z.cpu().numpy())


def oracle_packed(w16, bits):
    codes, s, z = oracle.quantize(w16, bits)
    return codes, oracle.pack(codes, bits), s, z


def gpu_linear(x16, qw, s, z, bits):
    y = laq.linear(to_dev(x16), to_dev(qw.view(np.int32)), to_dev(s.view(np.float16)), to_dev(z), bits)
    torch.cuda.synchronize()
    return y.cpu().numpy()


# ---------------------------------------------------------------------------
# quantize
# ---------------------------------------------------------------------------
QSHAPES = [(1, 128), (17, 384), (33, 2560), (5, 9728), (1024, 1024), (300, 4096), (2, 25600)]


@pytest.mark.parametrize("bits", [3, 4])
@pytest.mark.parametrize("N,K", QSHAPES)
def test_quantize_bitexact(bits, N, K):
    say("quantize", bits, N, K)
    w = inputs.weights(N, K, cfg=10, layer=N, proj=K % 97)
    codes, qw, s, z = oracle_packed(w, bits)
    gq, gs, gz = gpu_quantize(w, bits)
    assert np.array_equal(gs, s), "scales differ"
    assert np.array_equal(gz, z), "zeros differ"
    assert np.array_equal(gq, qw), "packed codes differ"


@pytest.mark.parametrize("bits", [3, 4])
def test_quantize_special_groups(bits):
    say("quantize special", bits)
    qmax = (1 << bits) - 1
    K = 384
    rows = []
    rows.append(np.zeros(K))                                   # all zero
    rows.append(np.full(K, 0.75))                              # constant positive
    rows.append(-np.linspace(0.01, 0.5, K))                    # all negative
    r = np.zeros(K); r[17] = -3.0; rows.append(r)              # single outlier
    r = np.zeros(K); r[:5] = [6e-8, -6e-8, 1.2e-7, 0, -1.8e-7]; rows.append(r)  # subnormal range
    r = np.zeros(K); r[0], r[1] = -3 / 64, 4 / 64
    r[2:12] = np.array([2.5, 1.5, -0.5, 0.5, 3.5, -2.5, -1.5, 4.0, -3.0, 0.0]) / 64
    rows.append(r)                                             # exact ties (W3 grid)
    rng = np.random.default_rng(3)
    for e in (-14, -3, 5):                                     # on-grid groups
        z0 = int(rng.integers(0, qmax + 1))
        j = rng.integers(0, qmax + 1, K); j[0], j[1] = 0, qmax
        rows.append(np.ldexp((j - z0).astype(np.float64), e))
    rows.append(np.full(K, 65504.0))                           # largest half
    r = np.full(K, -65504.0); r[::2] = 65504.0; rows.append(r)  # widest range
    rows.append(np.full(K, -0.0))                              # negative zeros
    w = np.array(rows).astype(np.float16)
    codes, qw, s, z = oracle_packed(w, bits)
    gq, gs, gz = gpu_quantize(w, bits)
    assert np.array_equal(gs, s) and np.array_equal(gz, z) and np.array_equal(gq, qw)


def test_quantize_canary():
    """Writes stay inside the outputs: sentinels around them are untouched."""
    say("quantize canary")
    N, K = 37, 640
    w = to_dev(inputs.weights(N, K, cfg=11))
    words = laq.packed_words(3, N, K)
    G = K // 128
    qbuf = torch.full((words + 64,), 0x5A5A5A5A, dtype=torch.int32, device=DEV)
    sbuf = torch.full((N * G + 64,), 7.0, dtype=torch.float16, device=DEV)
    zbuf = torch.full((N * G + 64,), 0xEE, dtype=torch.uint8, device=DEV)
    laq.quantize(w, 3, out=(qbuf[:words], sbuf[:N * G].view(N, G), zbuf[:N * G].view(N, G)))
    torch.cuda.synchronize()
    assert torch.all(qbuf[words:] == 0x5A5A5A5A)
    assert torch.all(sbuf[N * G:] == 7.0)
    assert torch.all(zbuf[N * G:] == 0xEE)


# ---------------------------------------------------------------------------
# pack with caller-supplied scales and zero points (Eq. 1, trained parameters)
# ---------------------------------------------------------------------------
def random_params(N, K, bits, seed):
    """Positive fp16 scales from the subnormal range to 2^7, zero points 0..qmax."""
    rng = np.random.default_rng(seed)
    G = K // 128
    e = rng.integers(-24, 8, (N, G))
    sv = np.ldexp(1.0 + rng.integers(0, 1024, (N, G)) / 1024.0, e).astype(np.float16)
    sv[sv == 0] = np.float16(2.0 ** -24)
    z = rng.integers(0, (1 << bits), (N, G)).astype(np.uint8)
    return sv.view(np.uint16), z


def gpu_pack(w16, s, z, bits):
    qw = laq.pack(to_dev(w16), to_dev(s.view(np.float16)), to_dev(z), bits)
    torch.cuda.synchronize()
    return qw.cpu().numpy().view(np.uint32)


@pytest.mark.parametrize("bits", [3, 4])
@pytest.mark.parametrize("N,K", QSHAPES)
def test_pack_bitexact(bits, N, K):
    say("pack", bits, N, K)
    w = inputs.weights(N, K, cfg=13, layer=N, proj=K % 89)
    s, z = random_params(N, K, bits, seed=N * 7 + K)
    ref = oracle.pack(oracle.codes_from_params(w, s, z, bits), bits)
    assert np.array_equal(gpu_pack(w, s, z, bits), ref)


@pytest.mark.parametrize("bits", [3, 4])
def test_pack_reproduces_quantize(bits):
    """Fed the parameters the min-max path wrote, pack gives its qweight."""
    say("pack vs quantize", bits)
    w = inputs.weights(129, 2560, cfg=14)
    gq, gs, gz = gpu_quantize(w, bits)
    assert np.array_equal(gpu_pack(w, gs, gz, bits), gq)


@pytest.mark.parametrize("bits", [3, 4])
def test_pack_special(bits):
    """Ties, clipping at both ends, extreme scales and weights."""
    say("pack special", bits)
    qmax = (1 << bits) - 1
    K = 256
    w = np.zeros((4, K))
    w[0, :12] = np.array([2.5, 1.5, -0.5, 0.5, 3.5, -2.5, -1.5, 4.0, -3.0, 0.0, 10.0, -10.0]) / 64
    w[1, :4] = [65504.0, -65504.0, 6e-8, -6e-8]
    w[2, :] = np.linspace(-8, 8, K)
    w[3, :] = -0.0
    w = w.astype(np.float16)
    s = np.array([[1 / 64, 0.5], [2.0 ** -24, 65504.0], [1.0, 2.0 ** -14], [0.25, 1.0]], np.float16).view(np.uint16)
    z = np.array([[3 % (qmax + 1), 0], [qmax, 0], [0, qmax], [1, qmax]], np.uint8)
    ref_codes = oracle.codes_from_params(w, s, z, bits)
    assert np.array_equal(gpu_pack(w, s, z, bits), oracle.pack(ref_codes, bits))


def test_pack_canary():
    """pack writes only qweight; scales and zeros are left as they were."""
    say("pack canary")
    N, K = 21, 768
    w = to_dev(inputs.weights(N, K, cfg=15))
    s, z = random_params(N, K, 3, seed=5)
    sd, zd = to_dev(s.view(np.float16)), to_dev(z)
    s0, z0 = sd.clone(), zd.clone()
    words = laq.packed_words(3, N, K)
    qbuf = torch.full((words + 64,), 0x3C3C3C3C, dtype=torch.int32, device=DEV)
    laq.pack(w, sd, zd, 3, out=qbuf[:words])
    torch.cuda.synchronize()
    assert torch.all(qbuf[words:] == 0x3C3C3C3C)
    assert torch.equal(sd, s0) and torch.equal(zd, z0)


# ---------------------------------------------------------------------------
# linear
# ---------------------------------------------------------------------------
LSHAPES = [(1, 128), (17, 384), (64, 128), (300, 2560), (1024, 1024), (4096, 1024), (257, 4096), (100, 9728), (3, 25600)]


@pytest.mark.parametrize("bits", [3, 4])
@pytest.mark.parametrize("M", [1, 2, 3, 4, 5, 8, 11, 16])
@pytest.mark.parametrize("N,K", LSHAPES)
def test_linear_parity(bits, M, N, K):
    say("linear", bits, M, N, K)
    w = inputs.weights(N, K, cfg=12, layer=M, proj=N % 89)
    x = inputs.activations(M, K, cfg=12, layer=N)
    codes, qw, s, z = oracle_packed(w, bits)
    y = gpu_linear(x, qw, s, z, bits)
    ref = oracle.linear(x, codes, s, z)
    r = linear_check(y, ref)
    assert r["ok"], r


@pytest.mark.parametrize("bits", [3, 4])
def test_linear_onehot_bitwise(bits):
    """x = e_k picks one exact term: y == fp16(w_hat[:, k]) bitwise."""
    say("linear onehot", bits)
    N, K = 200, 1280
    w = inputs.weights(N, K, cfg=13)
    codes, qw, s, z = oracle_packed(w, bits)
    wh = oracle.dequant(codes, s, z)
    for k in (0, 1, 29, 30, 31, 32, 127, 128, 555, K - 2, K - 1):
        x = np.zeros((1, K), np.float16)
        x[0, k] = 1.0
        y = gpu_linear(x, qw, s, z, bits)
        assert np.array_equal(y[0], wh[:, k].astype(np.float16)), k


@pytest.mark.parametrize("bits", [3, 4])
def test_linear_zero_codes_and_scaling(bits):
    say("linear zero/pow2", bits)
    M, N, K = 4, 130, 768
    w = inputs.weights(N, K, cfg=14)
    x = inputs.activations(M, K, cfg=14)
    codes, qw, s, z = oracle_packed(w, bits)
    # all-zero weights quantize to codes 0, zero point 0: y is exactly zero
    wz = np.zeros((N, K), np.float16)
    cz, qz, sz, zz = oracle_packed(wz, bits)
    assert np.all(gpu_linear(x, qz, sz, zz, bits) == 0)
    # codes equal to a nonzero zero point (a state quantize never produces):
    # the kernel forms sum x*q and z*sum x separately, so the result is the
    # fp32 rounding residue of that cancellation, bounded by a few fp32 ulps
    # of s*z*sum|x| per group (v_dot2_f32_f16 does not round each step to
    # nearest; see the design notes)
    c0 = np.repeat(z, 128, axis=1).astype(np.uint8)
    y0 = gpu_linear(x, oracle.pack(c0, bits), s, z, bits).astype(np.float64)
    sv = oracle.f16_to_f32(s).astype(np.float64)
    ax = np.abs(x.astype(np.float64)).reshape(M, K // 128, 128).sum(axis=2)      # [M][G]
    bound = (ax[:, None, :] * (sv * z)[None, :, :]).sum(axis=2) * 2.0 ** -16      # [M][N]
    assert np.all(np.abs(y0) <= bound + 2.0 ** -24), float(np.max(np.abs(y0) / (bound + 1e-30)))
    # y(4x) == 4 y(x) bitwise (power-of-two scaling is exact end to end)
    y1 = gpu_linear(x, qw, s, z, bits)
    y4 = gpu_linear((x.astype(np.float32) * 4).astype(np.float16), qw, s, z, bits)
    assert np.array_equal(y4, (y1.astype(np.float32) * 4).astype(np.float16))


@pytest.mark.parametrize("bits", [3, 4])
def test_linear_rows_consistent_and_deterministic(bits):
    say("linear rows/determinism", bits)
    N, K = 512, 2560
    w = inputs.weights(N, K, cfg=15)
    x = inputs.activations(16, K, cfg=15)
    codes, qw, s, z = oracle_packed(w, bits)
    y16 = gpu_linear(x, qw, s, z, bits)
    y16b = gpu_linear(x, qw, s, z, bits)
    assert np.array_equal(y16, y16b)
    ref = oracle.linear(x, codes, s, z)
    for m in (0, 7, 15):
        y1 = gpu_linear(x[m:m + 1], qw, s, z, bits)
        assert linear_check(y1[0], ref[m])["ok"]
        # both are within tolerance of the same exact value
        assert np.max(np.abs(y1[0].astype(np.float64) - y16[m])) <= 2e-3 * np.sqrt(np.mean(ref[m] ** 2)) + \
            np.max(np.abs(ref[m])) * 2 ** -10


def test_linear_canary():
    say("linear canary")
    M, N, K = 3, 77, 640
    w = inputs.weights(N, K, cfg=16)
    x = inputs.activations(M, K, cfg=16)
    codes, qw, s, z = oracle_packed(w, 3)
    ybuf = torch.full((M * N + 128,), 3.0, dtype=torch.float16, device=DEV)
    laq.linear(to_dev(x), to_dev(qw.view(np.int32)), to_dev(s.view(np.float16)), to_dev(z), 3,
               out=ybuf[:M * N].view(M, N))
    torch.cuda.synchronize()
    assert torch.all(ybuf[M * N:] == 3.0)
    r = linear_check(ybuf[:M * N].view(M, N).cpu().numpy(), oracle.linear(x, codes, s, z))
    assert r["ok"], r


def test_two_streams():
    say("two streams")
    M, N, K = 2, 2048, 2560
    w = inputs.weights(N, K, cfg=17)
    x = inputs.activations(M, K, cfg=17)
    codes, qw, s, z = oracle_packed(w, 3)
    ref = gpu_linear(x, qw, s, z, 3)
    xd, qd, sd, zd = to_dev(x), to_dev(qw.view(np.int32)), to_dev(s.view(np.float16)), to_dev(z)
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    outs = []
    for st in (s1, s2, s1, s2):
        with torch.cuda.stream(st):
            outs.append(laq.linear(xd, qd, sd, zd, 3))
    torch.cuda.synchronize()
    for o in outs:
        assert np.array_equal(o.cpu().numpy(), ref)


# ---------------------------------------------------------------------------
# full-size shapes (the Qwen3-4B layer; Qwen3-32B projections on sampled rows)
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("bits", [3, 4])
def test_layer4b_full(bits):
    """All seven Qwen3-4B projections at full size: GPU quantize bit-exact,
    GPU linear (M = 1 and 16) on the GPU-quantized weights vs the oracle."""
    for pi, (name, N, K) in enumerate(inputs.QWEN3_4B):
        say("layer4b", bits, name, N, K)
        w = inputs.weights(N, K, cfg=2, layer=0, proj=pi)
        codes, qw, s, z = oracle_packed(w, bits)
        gq, gs, gz = gpu_quantize(w, bits)
        assert np.array_equal(gs, s) and np.array_equal(gz, z) and np.array_equal(gq, qw), name
        for M in (1, 16):
            x = inputs.activations(M, K, cfg=2, layer=0, slot=inputs.X_SLOT[name])
            y = gpu_linear(x, gq, gs, gz, bits)
            r = linear_check(y, oracle.linear(x, codes, s, z))
            assert r["ok"], (name, M, r)


def test_stack32b_sampled():
    """Qwen3-32B projection shapes at full size on the GPU; the oracle checks
    every output of sampled rows (quantize is per row, so sampling rows of
    the weight matrix gives the same codes)."""
    rng = np.random.default_rng(32)
    for pi, (name, N, K) in enumerate(inputs.QWEN3_32B):
        if name in ("k", "v", "up"):
            continue
        say("stack32b", name, N, K)
        w = inputs.weights(N, K, cfg=5, layer=0, proj=pi)
        rows = np.sort(rng.choice(N, 96, replace=False))
        codes, qw, s, z = oracle_packed(np.ascontiguousarray(w[rows]), 3)
        wd = to_dev(w)
        q, sd, zd = laq.quantize(wd, 3)
        del wd
        torch.cuda.synchronize()
        assert np.array_equal(sd[rows].cpu().numpy().view(np.uint16), s)
        assert np.array_equal(zd[rows].cpu().numpy(), z)
        assert np.array_equal(q[rows].cpu().numpy().view(np.uint32), qw)
        for M in (1, 16):
            x = inputs.activations(M, K, cfg=5, layer=0, slot=inputs.X_SLOT[name])
            y = laq.linear(to_dev(x), q, sd, zd, 3)
            torch.cuda.synchronize()
            r = linear_check(y.cpu().numpy()[:, rows], oracle.linear(x, codes, s, z))
            assert r["ok"], (name, M, r)
        del q, sd, zd
        torch.cuda.empty_cache()


@pytest.mark.parametrize("bits", [3, 4])
def test_max_k(bits):
    """The largest K the ABI accepts (2^24): quantize and pack bit-exact, and
    the linear at M = 1 (K-tiled kernel: the activation row exceeds LDS), 2
    and 16 (matrix cores, many quad batches per wave) against the oracle."""
    K = 1 << 24
    N = 3
    say("max K", bits, N, K)
    rng = np.random.default_rng(77)
    w = (rng.standard_normal((N, K), dtype=np.float32) * 0.02).astype(np.float16)
    codes, qw, s, z = oracle_packed(w, bits)
    gq, gs, gz = gpu_quantize(w, bits)
    assert np.array_equal(gs, s) and np.array_equal(gz, z) and np.array_equal(gq, qw)
    assert np.array_equal(gpu_pack(w, s, z, bits), qw)
    for M in (1, 2, 16):
        x = rng.standard_normal((M, K), dtype=np.float32).astype(np.float16)
        y = gpu_linear(x, qw, s, z, bits)
        r = linear_check(y, oracle.linear(x, codes, s, z))
        assert r["ok"], (M, r)


QUAD_WAVE_SHAPES = [(17, 128), (300, 640), (1030, 2560), (257, 4992), (4100, 5120), (16400, 1152), (10256, 4992),
                    (257, 5248)]


@pytest.mark.parametrize("bits", [3, 4])
@pytest.mark.parametrize("N,K", QUAD_WAVE_SHAPES)
def test_matrix_core_quad_wave(bits, N, K):
    """Rows of at most 10 quads: one 16-row tile per block, one wave per quad, with
    the codes through LDS or in registers.  A single group (K = 128), a partial
    last quad (K = 640, five groups; K = 4992, 39 groups, ten quads), ten full
    quads (K = 5120), a ragged last tile (N = 17, 300, 1030, 257, 4100), at least
    1024 tiles (N = 16400; above M = 8, in W3 above 4, three tiles per block
    instead), more waves than stay resident with the fragments read up front
    (N = 10256, K = 4992: 641 tiles x 10 waves, the 64-register form up to M = 8,
    the streaming kernel above), and K = 5248 (eleven quads: just past the
    kernel's limit).  M from 3 (four-row slab) to 16 (sixteen-row slab)."""
    assert {route(3, 4, 257, 4992), route(4, 4, 300, 640)} == {"quad_wave_codes"}
    assert {route(3, 4, 1030, 2560), route(4, 16, 257, 4992)} == {"quad_wave"}
    assert {route(bits, M, 10256, 4992) for M in (3, 8)} == {"quad_wave_regs"}
    say("mfma quad wave", bits, N, K)
    w = inputs.weights(N, K, cfg=22, layer=bits, proj=K % 97)
    codes, qw, s, z = oracle_packed(w, bits)
    for M in (3, 4, 5, 8, 9, 16):
        x = inputs.activations(M, K, cfg=22, layer=M)
        y = gpu_linear(x, qw, s, z, bits)
        r = linear_check(y, oracle.linear(x, codes, s, z))
        assert r["ok"], (M, r)


SHARE_SHAPES = [(16437, 2176), (16400, 128), (19456, 2560), (16389, 1664)]


@pytest.mark.parametrize("bits", [3, 4])
@pytest.mark.parametrize("N,K", SHARE_SHAPES)
def test_matrix_core_quad_share(bits, N, K):
    """At least 1024 tiles, rows of at most five quads, M > 4 (W4: M > 8, the
    one-tile blocks below that): three tiles per block sharing the quads'
    activation slabs (8 rows up to M = 8, 16 above).
    A last block with two real tiles and an idle one, the last tile ragged
    (N = 16437 = 1027 * 16 + 5, 1028 tiles) and a last quad of one group
    (K = 2176, 17 groups); a single group (K = 128); the Qwen3-4B gate|up
    shape; a last block with one real tile (N = 16389: 1025 tiles, ragged) and
    four quads (K = 1664, 13 groups).  Repeated calls are bit-identical."""
    say("mfma quad share", bits, N, K)
    w = inputs.weights(N, K, cfg=23, layer=bits, proj=K % 89)
    codes, qw, s, z = oracle_packed(w, bits)
    for M in (5, 8, 9, 16):
        x = inputs.activations(M, K, cfg=23, layer=M)
        y = gpu_linear(x, qw, s, z, bits)
        r = linear_check(y, oracle.linear(x, codes, s, z))
        assert r["ok"], (M, r)
        assert np.array_equal(gpu_linear(x, qw, s, z, bits).view(np.uint16), y.view(np.uint16)), M


@pytest.mark.parametrize("bits", [3, 4])
def test_matrix_core_two_tiles_ragged(bits):
    """Rows longer than 10 quads, enough 16-row tiles (>= 256) and long
    enough rows for each wave to take two tiles, with a last block holding a
    partial tile (N = 4100 = 256 * 16 + 4) and a partial last quad (K = 9728,
    76 groups: 19 quads)."""
    N, K = 4100, 9728
    say("mfma two tiles", bits, N, K)
    w = inputs.weights(N, K, cfg=16, layer=bits)
    codes, qw, s, z = oracle_packed(w, bits)
    for M in (3, 5, 8, 16):
        assert route(bits, M, N, K) == ("one_tile_codes" if M == 3 else "two_tiles")
        x = inputs.activations(M, K, cfg=16, layer=M)
        y = gpu_linear(x, qw, s, z, bits)
        r = linear_check(y, oracle.linear(x, codes, s, z))
        assert r["ok"], (M, r)


@pytest.mark.parametrize("bits", [3, 4])
@pytest.mark.parametrize("N,K", [(16404, 640), (16400, 128), (16448, 2560)])
def test_matrix_core_shared_slab(bits, N, K):
    """Enough 16-row tiles (>= 1024) for blocks of three tiles sharing the
    activation slabs (M > 8; in W3 M > 4): a last block with idle waves and a
    partial tile (N = 16404 = 1025 * 16 + 4), a partial last 4-group quad (K =
    640, five groups) and a single group (K = 128).  M = 2, 3 and, in W4, 8 take
    the other kernels on the same weights."""
    assert route(bits, 9, N, K) == "share" and (route(bits, 8, N, K) == "share") == (bits == 3)
    say("mfma shared slab", bits, N, K)
    w = inputs.weights(N, K, cfg=17, layer=bits, proj=K % 97)
    codes, qw, s, z = oracle_packed(w, bits)
    for M in (2, 3, 8, 9, 12, 16):
        x = inputs.activations(M, K, cfg=17, layer=M)
        y = gpu_linear(x, qw, s, z, bits)
        r = linear_check(y, oracle.linear(x, codes, s, z))
        assert r["ok"], (M, r)


def _check_walk(bits, N, K):
    """Repeated weight rows against the oracle, equal rows bit for bit wherever
    they lie, repeated calls bit for bit, nothing written past the output."""
    codes, s, z, rows, w = _repeated_rows(bits, N, K)
    for M in (3, 8, 16):
        x = inputs.activations(M, K, cfg=19, layer=M)
        ybuf = torch.full((M * N + 64,), 3.0, dtype=torch.float16, device=DEV)
        y = laq.linear(to_dev(x), *w, bits, out=ybuf[:M * N].view(M, N))
        assert torch.equal(y, laq.linear(to_dev(x), *w, bits)) and torch.all(ybuf[M * N:] == 3.0), M
        y = y.cpu().numpy()
        assert np.array_equal(y, y[:, rows]), M
        r = linear_check(y[:, :len(codes)], oracle.linear(x, codes, s, z))
        assert r["ok"], (M, r)


# 17, 18 and 19 quads (every remainder of the loop over three register sets);
# 73 and 71 groups: a partial last quad.
WALK_K = [8704, 9088, 9344]


@pytest.mark.parametrize("bits", [3, 4])
@pytest.mark.parametrize("K", WALK_K)
def test_matrix_core_walk_four_tiles(bits, K):
    """1024..3071 row tiles of more than 16 quads walk K in blocks of four tiles,
    the quad weights in three register sets in turn.  N = 16400 = 1025 * 16: a
    last block with one tile."""
    N = 16400
    say("mfma walk four tiles", bits, N, K)
    assert {route(bits, M, N, K) for M in (3, 8, 16)} == {"walk4"}
    _check_walk(bits, N, K)


@pytest.mark.parametrize("M", [3, 5])
def test_matrix_core_two_tiles_per_wave_small_m(M):
    """More than 512 tiles (at M = 5 more than 256) and rows of more than 10
    quads: each wave takes two tiles, and its two KiB of partials reuse an
    activation slab of only M rows.  N = 8212 (ragged), K = 8704 (17 quads); rows
    with the same weights give the same bits wherever they lie."""
    N, K = 8212, 8704
    say("mfma two tiles per wave", M, N, K)
    assert route(3, M, N, K) == "two_tiles"
    codes, s, z, rows, w = _repeated_rows(3, N, K)
    x = inputs.activations(M, K, cfg=20, layer=M)
    y = laq.linear(to_dev(x), *w, 3).cpu().numpy()
    assert np.array_equal(y, y[:, rows])
    r = linear_check(y[:, :len(codes)], oracle.linear(x, codes, s, z))
    assert r["ok"], r


@pytest.mark.parametrize("bits", [3, 4])
@pytest.mark.parametrize("K", WALK_K)
def test_matrix_core_walk_ragged(bits, K):
    """From 3072 row tiles, blocks of eight tiles: N = 49173 = 3073 * 16 + 5, a
    last block with one whole and one partial tile."""
    N = 49173
    say("mfma walk ragged", bits, N, K)
    assert {route(bits, M, N, K) for M in (3, 8, 16)} == {"walk8"}
    _check_walk(bits, N, K)


STREAM_SHAPES = [(8200, 8192, (3, 8, 16)), (9003, 6528, (4, 9)), (80003, 2176, (3, 8, 16)), (65541, 2560, (3, 16)),
                 (33013, 3968, (8, 12)), (24581, 4096, (4, 5)), (10241, 5120, (8, 13))]


@pytest.mark.parametrize("bits", [3, 4])
@pytest.mark.parametrize("N,K,Ms", STREAM_SHAPES)
def test_matrix_core_stream(bits, N, K, Ms):
    """Activations in registers over many tiles: 16 quads (K = 8192: the
    activations staged in one, two or four phases by M; W4 at M = 16 with one
    buffer of partials), 13 and 8 quads with partial last ones (51 and 31
    groups), an odd count of quads whose last one has a single group (K =
    2176), three tiles per step (K = 2560), whole lines (G % 8 == 0: K = 4096,
    5120, 8192) and part lines, ragged last tiles and last steps with idle
    tiles.  Sampled rows and the last rows against the oracle; repeated calls
    bit-identical; nothing written past the output."""
    say("mfma stream", bits, N, K)
    assert {route(bits, M, N, K) for M in Ms} == {"stream"}
    rng = np.random.default_rng(N + bits)
    w = inputs.weights(N, K, cfg=24, layer=bits, proj=K % 97)
    rows = np.concatenate([np.arange(16), np.sort(rng.choice(N - 64, 48, replace=False)) + 16, np.arange(N - 40, N)])
    codes, qw, s, z = oracle_packed(np.ascontiguousarray(w[rows]), bits)
    q, sd, zd = laq.quantize(to_dev(w), bits)
    for M in Ms:
        x = inputs.activations(M, K, cfg=24, layer=M)
        ybuf = torch.full((M * N + 64,), 3.0, dtype=torch.float16, device=DEV)
        y = laq.linear(to_dev(x), q, sd, zd, bits, out=ybuf[:M * N].view(M, N))
        y2 = laq.linear(to_dev(x), q, sd, zd, bits)
        torch.cuda.synchronize()
        r = linear_check(y.cpu().numpy()[:, rows], oracle.linear(x, codes, s, z))
        assert r["ok"], (M, r)
        assert torch.equal(y, y2) and torch.all(ybuf[M * N:] == 3.0), M


# Shapes of the streaming kernel: every count of staged rows and staging phase,
# split into K ranges, whole and partial lines.
STREAM_ROUND_SHAPES = [(8200, 8192), (10241, 5120), (80003, 2176), (24581, 4096), (1600, 25216)]


def _repeated_rows(bits, N, K, period=251):
    """Quantized weights whose N rows repeat `period` base rows: (codes, scales,
    zeros) of the base rows, the base row of each row, and the device tensors."""
    codes, qw, s, z = oracle_packed(inputs.weights(period, K, cfg=25, layer=bits, proj=K % 97), bits)
    rows = np.arange(N) % period
    take = torch.from_numpy(rows).to(DEV)
    return codes, s, z, rows, [to_dev(a)[take].contiguous() for a in (qw.view(np.int32), s.view(np.float16), z)]


@pytest.mark.parametrize("bits", [3, 4])
@pytest.mark.parametrize("N,K", STREAM_ROUND_SHAPES)
def test_matrix_core_stream_rounding(bits, N, K):
    """Almost every output is the fp16 rounding of the exact sum itself: what
    comes before that rounding is a 32-bit accumulation of exact (q - z) x
    products.  At most K / 32 + K / 128 additions on the way to an output, each
    off by up to 2^-25 of the sum so far, in random directions: about 1e-6 of
    the output's RMS for the longest row, and an error e moves a value across a
    rounding boundary with probability 2 |e| / ulp, where the ulp is 7e-4 of a
    typical value: 0.2 %.  Bound: 0.5 %.  (5120-wide rows below M = 8 take the
    one-wave-per-quad kernel.)  Activations of both signs, one-signed,
    subnormal and up to the largest halves.  Rows with the same weights give
    the same bits wherever they lie."""
    say("mfma stream rounding", bits, N, K)
    assert {route(bits, M, N, K, True) for M in (8, 16)} <= {"stream", "split_stream"}
    codes, s, z, rows, (qd, sd, zd) = _repeated_rows(bits, N, K)
    P = len(codes)
    for kind, xscale, sscale in (("both signs", 1.0, 1.0), ("one sign", 1.0, 1.0), ("subnormal", 2.0**-17, 2.0**6),
                                 ("large", 2.0**14, 2.0**-8)):
        sh = (s.view(np.float16).astype(np.float64) * sscale).astype(np.float16)
        sk = to_dev(sh)[torch.from_numpy(rows).to(DEV)].contiguous()
        wrong = total = 0
        for M in (3, 8, 16):
            x = inputs.activations(M, K, cfg=25, layer=M).astype(np.float64)
            x = np.clip((np.abs(x) if kind == "one sign" else x) * xscale, -65504, 65504).astype(np.float16)
            y = laq.linear(to_dev(x), qd, sk, zd, bits)
            torch.cuda.synchronize()
            y = y.cpu().numpy()
            assert np.array_equal(y, y[:, rows]), (kind, M)
            ref = oracle.linear(x, codes, sh.view(np.uint16), z)
            assert np.abs(ref).max() < 60000
            r = linear_check(y[:, :P], ref)
            assert r["ok"], (kind, M, r)
            wrong += int((y[:, :P] != ref.astype(np.float16)).sum())
            total += ref.size
        assert wrong <= 0.005 * total, (kind, wrong, total)


@pytest.mark.parametrize("bits", [3, 4])
@pytest.mark.parametrize("N,K", [(200, 640), (100, 16384), (16437, 2176), (16400, 8704), (4100, 9728), (731, 22272)] +
                         STREAM_ROUND_SHAPES)
def test_matrix_core_infinite_activation(bits, N, K):
    """One infinite activation: its row's outputs are infinite with the sign of
    (q - z) x, or NaN where q = z, on every matrix-core path alike; the other
    rows' outputs do not change."""
    say("infinite activation", bits, N, K)
    codes, s, z, rows, w = _repeated_rows(bits, N, K)
    d = codes.astype(np.int64) - np.repeat(z.astype(np.int64), 128, axis=1)
    for M in (3, 8, 16):
        x = inputs.activations(M, K, cfg=25, layer=M)
        plain = laq.linear(to_dev(x), *w, bits).cpu().numpy()
        for row, col, v in ((0, 0, np.inf), (M - 1, K - 1, -np.inf), (1, K // 2 + 5, np.inf)):
            xi = x.copy()
            xi[row, col] = v
            got = laq.linear(to_dev(xi), *w, bits).cpu().numpy()
            ref = plain.copy()
            dc = d[rows, col]
            ref[row] = np.where(dc == 0, np.nan, np.where(dc > 0, v, -v))
            assert np.array_equal(got, ref, equal_nan=True), (M, row, col)


SPLIT_SHAPES = [(5120, 25600), (100, 25088), (3, 20608), (1030, 20480), (1030, 20608), (1600, 25216), (731, 22272),
                (190, 131840), (250, 131840), (380, 131840)]


@pytest.mark.parametrize("bits", [3, 4])
@pytest.mark.parametrize("N,K", SPLIT_SHAPES)
def test_split_k(bits, N, K):
    """K split across workgroups (rows of >= 40 quads, fewer than 1024 tiles).
    With many (tile, quad) units the ranges run in the streaming kernel: the
    Qwen3-32B down projection, 1030 rows (at M = 16 in W4 only), and odd group
    counts (K = 20608: 161, 25216: 197) with part lines, a partial last quad and
    quads past the row in the last range.  Otherwise blocks of four tiles over
    ranges of one (N = 100, 3), two (731), three, four and five (K = 131840) quads,
    with idle tiles in the last block and a partial tile; against the oracle,
    deterministic, and the plain entry point also within tolerance."""
    ranges = {100: 1, 3: 1, 731: 2, 190: 3, 250: 4, 380: 5}.get(N)
    if ranges:
        assert split_plan(16, N, K // 128).qs == ranges and route(bits, 16, N, K, True) == "split"
    else:
        assert route(bits, 8, N, K, True) == "split_stream"
    say("split K", bits, N, K)
    assert laq.workspace_bytes(16, N, K) > 0
    w = inputs.weights(N, K, cfg=19, layer=bits, proj=K % 83)
    codes, qw, s, z = oracle_packed(w, bits)
    qd, sd, zd = to_dev(qw.view(np.int32)), to_dev(s.view(np.float16)), to_dev(z)
    for M in (2, 3, 5, 8, 16):
        x = inputs.activations(M, K, cfg=19, layer=M)
        xd = to_dev(x)
        y1 = laq.linear(xd, qd, sd, zd, bits)
        y2 = laq.linear(xd, qd, sd, zd, bits)
        yp = laq.linear(xd, qd, sd, zd, bits, split_k=False)
        torch.cuda.synchronize()
        ref = oracle.linear(x, codes, s, z)
        assert torch.equal(y1, y2), M
        r = linear_check(y1.cpu().numpy(), ref)
        assert r["ok"], (M, r)
        r = linear_check(yp.cpu().numpy(), ref)
        assert r["ok"], (M, "plain", r)


def test_split_k_small_workspace():
    """A workspace smaller than laq_linear_workspace_bytes: the _ws call is
    the plain call, bit for bit."""
    N, K, M = 1030, 20480, 16
    say("split K small workspace", N, K, M)
    w = inputs.weights(N, K, cfg=20, layer=1)
    codes, qw, s, z = oracle_packed(w, 3)
    qd, sd, zd = to_dev(qw.view(np.int32)), to_dev(s.view(np.float16)), to_dev(z)
    xd = to_dev(inputs.activations(M, K, cfg=20, layer=2))
    need = laq.workspace_bytes(M, N, K)
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    y = torch.empty((M, N), dtype=torch.float16, device=DEV)
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    st = laq.lib().laq_linear_ws_w3g128(ctypes.c_void_p(xd.data_ptr()), ctypes.c_void_p(qd.data_ptr()),
                                        ctypes.c_void_p(sd.data_ptr()), ctypes.c_void_p(zd.data_ptr()),
                                        ctypes.c_void_p(y.data_ptr()), M, N, K, ctypes.c_void_p(ws.data_ptr()),
                                        need - 16, stream)
    assert st == laq.LAQ_OK
    yp = laq.linear(xd, qd, sd, zd, 3, split_k=False)
    torch.cuda.synchronize()
    assert torch.equal(y, yp)


# ---------------------------------------------------------------------------
# grouped calls: several independent linears in one launch
# ---------------------------------------------------------------------------
def _group_case(bits, specs, M, cfg):
    """specs: list of (N, K, x_slot); calls sharing a slot share x."""
    xs = {}
    calls, refs = [], []
    for i, (N, K, slot) in enumerate(specs):
        if slot not in xs:
            xs[slot] = inputs.activations(M, K, cfg=cfg, layer=slot)
        x = xs[slot]
        w = inputs.weights(N, K, cfg=cfg, layer=i, proj=bits)
        codes, qw, s, z = oracle_packed(w, bits)
        calls.append((to_dev(x), to_dev(qw.view(np.int32)), to_dev(s.view(np.float16)), to_dev(z)))
        refs.append(oracle.linear(x, codes, s, z))
    ys = laq.linear_group(calls, bits)
    singles = [laq.linear(*c, bits) for c in calls]
    torch.cuda.synchronize()
    return [y.cpu().numpy() for y in ys], [y.cpu().numpy() for y in singles], refs


@pytest.mark.parametrize("bits", [3, 4])
@pytest.mark.parametrize("M", [1, 2, 3, 4, 8, 16])
def test_group_qkv(bits, M):
    """q, k, v of a Qwen3-4B layer (same activations) as one launch.  Up to
    M = 2 the grouped and the single calls run the same VALU kernel body and
    agree bit for bit; from M = 3 both take the matrix cores, one wave per
    quad."""
    say("group qkv", bits, M)
    ys, singles, refs = _group_case(bits, [(4096, 2560, 0), (1024, 2560, 0), (1024, 2560, 0)], M, cfg=40)
    for y, y1, ref in zip(ys, singles, refs):
        r = linear_check(y, ref)
        assert r["ok"], r
        if M <= 2:  # the same kernel body, bit for bit
            assert np.array_equal(y.view(np.uint16), y1.view(np.uint16))


@pytest.mark.parametrize("bits", [3, 4])
@pytest.mark.parametrize("M", [1, 2, 16])
def test_group_mixed(bits, M):
    """Eight calls of different shapes (the most a group takes): several K,
    ragged N, a single row, separate activations."""
    say("group mixed", bits, M)
    specs = [(2560, 4096, 0), (257, 9728, 1), (1, 128, 2), (300, 2560, 3), (17, 384, 4),
             (1024, 1024, 5), (96, 9728, 1), (64, 128, 6)]
    ys, singles, refs = _group_case(bits, specs, M, cfg=41)
    for y, y1, ref in zip(ys, singles, refs):
        r = linear_check(y, ref)
        assert r["ok"], r
        if M <= 2:
            assert np.array_equal(y.view(np.uint16), y1.view(np.uint16))


@pytest.mark.parametrize("bits", [3, 4])
@pytest.mark.parametrize("M", [3, 4, 8, 9, 16])
def test_group_row_lengths(bits, M):
    """Rows of 1, 2, 5 and 10 quads in one launch of the one-wave-per-quad
    kernel (waves past a shorter row's quads only join the barrier), ragged N,
    partial last quads, separate activations."""
    say("group row lengths", bits, M)
    specs = [(300, 4992, 0), (17, 128, 1), (257, 640, 2), (1, 2560, 3), (130, 2176, 4)]
    assert group_quad_wave(M, sum(-(-N // 16) for N, _, _ in specs), 10) == 0
    ys, _, refs = _group_case(bits, specs, M, cfg=43)
    for y, ref in zip(ys, refs):
        r = linear_check(y, ref)
        assert r["ok"], r


@pytest.mark.parametrize("bits", [3, 4])
@pytest.mark.parametrize("M,form", [(3, 1), (8, 1), (9, -1), (16, 1)])
def test_group_many_tiles(bits, M, form):
    """More tiles than are resident in the up-front form: the 64-register form,
    or at M = 9 the kernel whose waves walk several quads; one call with shorter
    rows and a ragged last tile.  Repeated weight rows give the same bits,
    repeated calls too, and nothing is written past the outputs."""
    say("group many tiles", bits, M)
    shapes = [(9728, 2560), (9731, 640), (9728, 2560)]
    assert group_quad_wave(M, sum(-(-N // 16) for N, _ in shapes), 5) == form
    cases = [_repeated_rows(bits, N, K) for N, K in shapes]
    xs = [inputs.activations(M, K, cfg=44, layer=i) for i, (_, K) in enumerate(shapes)]
    calls = [(to_dev(x), *c[4]) for x, c in zip(xs, cases)]
    bufs = [torch.full((M * N + 64,), 3.0, dtype=torch.float16, device=DEV) for N, _ in shapes]
    ys = laq.linear_group(calls, bits, outs=[b[:M * N].view(M, N) for b, (N, _) in zip(bufs, shapes)])
    again = laq.linear_group(calls, bits)
    torch.cuda.synchronize()
    for x, (codes, s, z, rows, _), y, y2, buf in zip(xs, cases, ys, again, bufs):
        assert torch.equal(y, y2) and torch.all(buf[y.numel():] == 3.0)
        y = y.cpu().numpy()
        assert np.array_equal(y, y[:, rows])
        r = linear_check(y[:, :len(codes)], oracle.linear(x, codes, s, z))
        assert r["ok"], r


@pytest.mark.parametrize("bits", [3, 4])
def test_group_long_rows_one_row(bits):
    """M = 1 with a row longer than LDS holds: one launch per call, same results."""
    say("group long rows", bits)
    ys, singles, refs = _group_case(bits, [(5, 32768, 0), (3, 32768, 0)], 1, cfg=42)
    for y, y1, ref in zip(ys, singles, refs):
        assert linear_check(y, ref)["ok"]
        assert np.array_equal(y.view(np.uint16), y1.view(np.uint16))


# ---------------------------------------------------------------------------
# graph capture: every kernel path replayed several times, each replay equal
# (bitwise) to the eager call, with eager work of the same kernels between
# ---------------------------------------------------------------------------
GRAPH_CASES = [
    ("flat M=2 two rows per lane", 2, 300, 9728, 3),
    ("matrix cores one wave per quad M=5", 5, 1030, 4096, 4),
    ("matrix cores one wave per quad M=16", 16, 300, 5120, 3),
    ("matrix cores one wave per quad, 64 registers M=4", 4, 10256, 4992, 3),
    ("matrix cores one tile M=5", 5, 1030, 9728, 4),
    ("matrix cores three tiles M=16", 16, 16400, 2560, 3),
    ("streaming M=12", 12, 16400, 4096, 3),
    ("matrix cores walk M=12", 12, 16400, 8704, 3),
    ("split K with workspace M=16", 16, 1030, 25600, 3),
    ("split K, streaming ranges M=16", 16, 1600, 25216, 3),
]


@pytest.mark.parametrize("name,M,N,K,bits", GRAPH_CASES)
def test_graph_replay(name, M, N, K, bits):
    say("graph replay", name, M, N, K, bits)
    w = to_dev(inputs.weights(N, K, cfg=21, layer=M))
    x = to_dev(inputs.activations(M, K, cfg=21, layer=M))
    q, s, z = laq.quantize(w, bits)
    y_eager = laq.linear(x, q, s, z, bits)
    torch.cuda.synchronize()
    qg, sg, zg = torch.empty_like(q), torch.empty_like(s), torch.empty_like(z)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=torch.cuda.Stream()):
        laq.quantize(w, bits, out=(qg, sg, zg))
        y_graph = laq.linear(x, qg, sg, zg, bits)
    for _ in range(3):
        for t in (qg, sg, zg, y_graph):
            t.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(qg, q) and torch.equal(sg, s) and torch.equal(zg, z), name
        assert torch.equal(y_graph.view(torch.int16), y_eager.view(torch.int16)), name
        # eager work of the same kernels between replays
        y2 = laq.linear(x, q, s, z, bits)
        torch.cuda.synchronize()
        assert torch.equal(y2.view(torch.int16), y_eager.view(torch.int16)), name
    del g
