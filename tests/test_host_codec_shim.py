"""The per-block codec that the GPU lanes run (csrc/zc_codec.h) is also compiled
for the host and compared, block by block and bit for bit, with the reference
codec.  This checks the kernels' logic (tables, bit transposition, stream
windowing) without a GPU; the GPU parity tests check the kernels themselves."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2409_02423_amd import workloads

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "shim", "zc_codec_host.cpp")
LIB = os.path.join(HERE, "shim", "libzc_codec_host.so")
HDR = os.path.join(HERE, "..", "paper_2409_02423_amd", "csrc", "zc_codec.h")
RATES = (4, 8, 12, 16, 20, 24, 28, 32)


@pytest.fixture(scope="module")
def shim():
    newest = max(os.path.getmtime(SRC), os.path.getmtime(HDR))
    if not os.path.exists(LIB) or os.path.getmtime(LIB) < newest:
        subprocess.check_call(["g++", "-std=c++17", "-O2", "-fwrapv", "-ffp-contract=off", "-shared", "-fPIC",
                               "-fconstexpr-ops-limit=200000000", "-pthread", SRC, "-o", LIB])
    L = ctypes.CDLL(LIB)
    L.zc_host_encode_blocks.argtypes = [ctypes.c_int, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p]
    L.zc_host_decode_blocks.argtypes = [ctypes.c_int, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p]
    L.zc_host_add_blocks.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p]
    L.zc_host_encode_wave.argtypes = [ctypes.c_int, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p, ctypes.c_int]
    L.zc_host_decode_wave.argtypes = [ctypes.c_int, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p, ctypes.c_int]
    L.zc_host_region_order.argtypes = [ctypes.c_size_t, ctypes.c_size_t, ctypes.c_int]
    L.zc_host_region_order.restype = ctypes.c_size_t
    L.zc_host_accumulate4_all.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p]
    L.zc_host_accumulate4_all.restype = None
    return L


def _enc(L, x, rate):
    x = np.ascontiguousarray(x, dtype=np.float32)
    out = np.zeros(x.size // 4 * (rate // 2), dtype=np.uint8)
    assert L.zc_host_encode_blocks(rate, x.ctypes.data, x.size // 4, out.ctypes.data) == 0
    return out


def _dec(L, s, nblocks, rate):
    s = np.ascontiguousarray(s, dtype=np.uint8)
    out = np.zeros(4 * nblocks, dtype=np.float32)
    assert L.zc_host_decode_blocks(rate, s.ctypes.data, nblocks, out.ctypes.data) == 0
    return out


def _inputs():
    smooth = np.cumsum(workloads.gradient_iid(4096, std=1e-4)).astype(np.float32)  # small high-order coefficients
    ramp = (np.arange(4096, dtype=np.float32) * np.float32(0.37) - 700).astype(np.float32)
    return [workloads.edge_values(11), workloads.gradient_iid(1 << 14), workloads.activation_gelu(1 << 14),
            workloads.adam_second_moments(1 << 13), workloads.gradient_lowrank(64, 128), smooth, ramp]


@pytest.mark.parametrize("rate", RATES)
def test_encode_matches_reference(oracle, shim, rate):
    for x in _inputs():
        want = oracle.compress(x, rate)
        got = _enc(shim, x, rate)
        bad = np.flatnonzero((got != want).reshape(-1, rate // 2).any(axis=1))
        assert bad.size == 0, (rate, bad[:5], x.reshape(-1, 4)[bad[:1]])


@pytest.mark.parametrize("rate", RATES)
def test_decode_matches_reference(oracle, shim, rate):
    rng = np.random.default_rng(rate)
    for x in _inputs():
        s = oracle.compress(x, rate)
        want = oracle.decompress(s, x.size, rate)
        got = _dec(shim, s, x.size // 4, rate)
        bad = np.flatnonzero((got.view(np.uint32) != want.view(np.uint32)).reshape(-1, 4).any(axis=1))
        assert bad.size == 0, (rate, bad[:5])
    # arbitrary bytes: every string decodes, and to the same values
    for trial in range(3):
        s = rng.integers(0, 256, size=8192 * (rate // 2), dtype=np.uint8)
        if trial == 1:  # long runs of zero bits, short streams
            s &= rng.integers(0, 256, size=s.size, dtype=np.uint8) & rng.integers(0, 256, size=s.size, dtype=np.uint8)
        if trial == 2:
            s |= rng.integers(0, 256, size=s.size, dtype=np.uint8)
        with np.errstate(all="ignore"):
            want = oracle.decompress(s, 4 * 8192, rate)
        got = _dec(shim, s, 8192, rate)
        bad = np.flatnonzero((got.view(np.uint32) != want.view(np.uint32)).reshape(-1, 4).any(axis=1))
        assert bad.size == 0, (rate, trial, bad[:5])


def _mixed_blocks():
    """Blocks that need very different numbers of coder steps side by side: edge values, constants
    (one significant coefficient through all planes), zero blocks, ramps, noise, single spikes."""
    rng = np.random.default_rng(77)
    parts = [workloads.edge_values(12)[:2048], np.repeat(workloads.gradient_iid(256), 4), np.zeros(256, np.float32),
             workloads.gradient_iid(2048), (np.arange(1024, dtype=np.float32) * np.float32(1e-3)),
             workloads.activation_gelu(2048), np.where(rng.random(1024) < 0.1, 1.0, 0.0).astype(np.float32)]
    blocks = np.concatenate(parts).astype(np.float32).reshape(-1, 4)
    return blocks[rng.permutation(len(blocks))].reshape(-1)


@pytest.mark.parametrize("rate", RATES)
def test_lockstep_lanes_match_reference(oracle, shim, rate):
    """The per-lane codec with its wavefront-wide loop decisions taken by a vote among lanes that run
    in lockstep (16 and 5 lanes): what one lane does must not depend on its neighbours' blocks."""
    x = _mixed_blocks()[: 4 * 1500]
    nb = x.size // 4
    want_c = oracle.compress(x, rate)
    want_d = oracle.decompress(want_c, x.size, rate)
    rng = np.random.default_rng(500 + rate)
    junk = rng.integers(0, 256, size=nb * (rate // 2), dtype=np.uint8)
    junk[::3] &= rng.integers(0, 256, size=junk[::3].size, dtype=np.uint8)
    with np.errstate(all="ignore"):
        want_j = oracle.decompress(junk, x.size, rate)
    for lanes in (16, 5):
        got_c = np.zeros_like(want_c)
        assert shim.zc_host_encode_wave(rate, x.ctypes.data, nb, got_c.ctypes.data, lanes) == 0
        assert np.array_equal(got_c, want_c), (rate, lanes)
        for stream, want in ((want_c, want_d), (junk, want_j)):
            got = np.zeros(x.size, dtype=np.float32)
            assert shim.zc_host_decode_wave(rate, stream.ctypes.data, nb, got.ctypes.data, lanes) == 0
            bad = np.flatnonzero((got.view(np.uint32) != want.view(np.uint32)).reshape(-1, 4).any(axis=1))
            assert bad.size == 0, (rate, lanes, bad[:5])


def test_region_order_is_a_permutation_of_the_tiles(shim):
    """The tile order of the decompress kernels: every tile exactly once, whatever the tile count and
    region size; whole groups of eight regions are reordered (indices with the same value mod 8 walk
    through regions x, x + 8, ...), the rest stays in place."""
    for lg in (0, 2, 5, 6, 8):
        for tiles in (0, 1, 7, 8 << lg, (8 << lg) - 1, (8 << lg) + 1, 3 * (8 << lg) + 5, 12288, 65536, 36621):
            got = [shim.zc_host_region_order(v, tiles, lg) for v in range(tiles)]
            assert sorted(got) == list(range(tiles)), (lg, tiles)
            bulk = (tiles >> (lg + 3)) << (lg + 3)
            assert got[bulk:] == list(range(bulk, tiles))
            if bulk:
                mine = [got[v] for v in range(3, bulk, 8)]          # what XCD 3 walks through
                assert mine == sorted(mine) and all((t >> lg) % 8 == 3 for t in mine)


def test_rate4_accumulate_forms_on_every_block(oracle, shim):
    """The fused reduce at rate 4 adds a block to the running sum through a table and a fused
    multiply-add (plain form) unless unusual4 flags the block, in which case the tile is summed
    again in the careful form.  All 65536 two-byte blocks, against decode-then-add with the
    reference decoder, for running sums of either sign, tiny, huge and infinite; the flagged blocks
    are exactly those with exponent byte 250 and more or exponent byte 0 over a nonzero payload, and
    the plain form is wrong on some of them (so the flag is needed)."""
    W0 = np.arange(65536, dtype=np.uint16)
    stream = W0.view(np.uint8)
    decoded = oracle.decompress(stream, 4 * 65536, 4).reshape(-1, 4)
    E, payload = W0 & 0xFF, W0 >> 8
    expect_flag = (E >= 250) | ((E == 0) & (payload != 0))
    flags = np.zeros(65536, dtype=np.uint8)
    got = np.zeros((65536, 4), dtype=np.float32)
    shim.zc_host_accumulate4_all(1, 0, got.ctypes.data, flags.ctypes.data)
    assert np.array_equal(flags.astype(bool), expect_flag)
    assert np.array_equal(got.view(np.uint32), decoded.view(np.uint32))
    rng = np.random.default_rng(5)
    plain_differs = 0
    with np.errstate(over="ignore", invalid="ignore"):
        for base in (0.0, -0.0, 1e-3, -1e-3, 1e-42, -3e38, 3e38, np.inf, -np.inf):
            start = (np.float32(base) * (1 + rng.random((65536, 4), dtype=np.float32))).astype(np.float32)
            want = (start + decoded).astype(np.float32)
            for form in (0, 1):
                got = start.copy()
                shim.zc_host_accumulate4_all(0, form, got.ctypes.data, flags.ctypes.data)
                same = (got.view(np.uint32) == want.view(np.uint32)) | (np.isnan(got) & np.isnan(want))
                if form == 0:
                    assert same.all(), (base, np.flatnonzero(~same.all(axis=1))[:5])
                else:
                    assert same[~expect_flag].all()
                    plain_differs += int((~same[expect_flag]).any())
    assert plain_differs > 0


@pytest.mark.parametrize("rate", RATES)
@pytest.mark.parametrize("branches", (0, 1))
def test_decoded_blocks_are_added_with_one_rounding(oracle, shim, rate, branches):
    """The decoder that adds to a sum, with its rare cases branched around and not, against the reference's decoded
    values added in fp32: exponent bytes where the scaling's form changes (28 and 29, 251 and 252), zero blocks, empty
    first words and arbitrary bytes, onto ordinary sums, zeros of both signs and subnormals."""
    rng = np.random.default_rng(50 * rate + branches)
    n = 6000
    s = rng.integers(0, 256, size=(n, rate // 2), dtype=np.uint8)
    s[:, 0] = np.where(rng.random(n) < 0.7, rng.choice([0, 1, 2, 27, 28, 29, 30, 127, 250, 251, 252, 253, 255], size=n), s[:, 0])
    s[::5, 1:4] = 0
    s[::7, 1:] = 0
    s[1::7, 1:] &= rng.integers(0, 256, size=s[1::7, 1:].shape, dtype=np.uint8) & rng.integers(0, 256, size=s[1::7, 1:].shape, dtype=np.uint8)
    with np.errstate(all="ignore"):
        y = np.concatenate([oracle.decode_block(b, rate) for b in s])
        start = (rng.standard_normal(4 * n) * np.ldexp(1.0, rng.integers(-140, 120, size=4 * n))).astype(np.float32)
        start[::9], start[4::9] = 0.0, -0.0
        start[1::3] = (y[1::3] * rng.uniform(-2, 2, size=y[1::3].size)).astype(np.float32)
        want = start + y
    got = start.copy()
    assert shim.zc_host_add_blocks(rate, branches, s.ctypes.data, n, got.ctypes.data) == 0
    ok = (got.view(np.uint32) == want.view(np.uint32)) | (np.isnan(got) & np.isnan(want))
    assert ok.all(), (rate, branches, np.flatnonzero(~ok)[:5])


@pytest.mark.parametrize("rate", RATES)
@pytest.mark.parametrize("share", (0.5, 0.95, 1.0))
def test_zero_blocks_side_by_side_with_others(oracle, shim, rate, share):
    """Lockstep lanes most of which hold zero blocks, with and without a payload (which is ignored), beside blocks with
    common and uncommon exponent bytes, an empty first word and no payload at all."""
    rng = np.random.default_rng(60 * rate + int(100 * share))
    n = 1600
    s = rng.integers(0, 256, size=(n, rate // 2), dtype=np.uint8)
    s[:, 0] = np.where((rng.random(n // 80) < 0.4).repeat(80), rng.choice([1, 28, 29, 251, 252, 255], size=n), rng.integers(100, 140, size=n))
    s[::5, 1:4] = 0
    s[::11, 1:] = 0
    zero = rng.random(n) < share
    s[zero, 0] = 0
    s[zero & (rng.random(n) < 0.5), 1:] = 0
    s = np.ascontiguousarray(s.reshape(-1))
    with np.errstate(all="ignore"):
        want = oracle.decompress(s, 4 * n, rate)
    for lanes in (16, 5):
        got = np.zeros(4 * n, dtype=np.float32)
        assert shim.zc_host_decode_wave(rate, s.ctypes.data, n, got.ctypes.data, lanes) == 0
        bad = np.flatnonzero((got.view(np.uint32) != want.view(np.uint32)).reshape(-1, 4).any(axis=1))
        assert bad.size == 0, (rate, share, lanes, bad[:5])


def _rate8_blocks(rng):
    """Arbitrary blocks by the number of empty planes (the first plane crowded or not), dense and sparse, under exponent
    bytes of every kind, and what the encoder makes of ordinary values."""
    bits = rng.integers(0, 2, size=(24 * 1500, 24), dtype=np.uint8)
    for k in range(3):
        bits[k::4] &= rng.integers(0, 2, size=bits[k::4].shape, dtype=np.uint8)
    for lead in range(24):
        part = bits[1500 * lead:1500 * (lead + 1)]
        part[:, :lead] = 0
        part[:, lead] = 1
    s = np.zeros((len(bits), 4), dtype=np.uint8)
    s[:, 1:] = np.packbits(bits, axis=1, bitorder="little")
    s[:, 0] = np.where(rng.random(len(s)) < 0.3, rng.choice([0, 1, 28, 29, 30, 239, 240, 241, 251, 252, 255], size=len(s)), rng.integers(29, 241, size=len(s)))
    return s


@pytest.mark.parametrize("stream", (0, 1))
def test_rate8_matrix_matches_reference(oracle, shim, stream):
    """The decoder's inverse transform as a matrix product at rate 8, alone and added to sums (zeros of both signs among
    them, whose sign a stream does not keep), against the reference decoder and an addition in fp32; and that the matrix covers
    what it is for: nearly all of the encoder's blocks, and none without an empty plane."""
    shim.zc_host_matrix8.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p, ctypes.c_void_p]
    rng = np.random.default_rng(88 + stream)
    s = _rate8_blocks(rng)
    ordinary = oracle.compress(workloads.gradient_lowrank(64, 1024).reshape(-1), 8).reshape(-1, 4)
    rows = np.ascontiguousarray(np.concatenate([s, ordinary]))
    n = len(rows)
    with np.errstate(all="ignore"):
        y = oracle.decompress(rows.reshape(-1), 4 * n, 8)
        start = (rng.standard_normal(4 * n) * np.ldexp(1.0, rng.integers(-140, 120, size=4 * n))).astype(np.float32)
        start[::9], start[4::9] = 0.0, -0.0
        start[1::3] = (y[1::3] * rng.uniform(-2, 2, size=y[1::3].size)).astype(np.float32)
        want = start + y
    covered = np.zeros(n, dtype=np.uint8)
    got = np.zeros(4 * n, dtype=np.float32)
    assert shim.zc_host_matrix8(1, 0, rows.ctypes.data, n, got.ctypes.data, covered.ctypes.data) == 0
    bad = np.flatnonzero(got.view(np.uint32) != y.view(np.uint32))
    assert bad.size == 0, (bad[:5], rows[bad[:1] // 4])
    got = start.copy()
    assert shim.zc_host_matrix8(0, stream, rows.ctypes.data, n, got.ctypes.data, covered.ctypes.data) == 0
    ok = (got.view(np.uint32) == want.view(np.uint32)) | (np.isnan(got) & np.isnan(want)) | ((stream != 0) & (got == 0) & (want == 0))
    assert ok.all(), np.flatnonzero(~ok)[:5]
    by_lead = covered[:24 * 1500].reshape(24, 1500).mean(axis=1)
    assert by_lead[0] == 0 and 0 < by_lead[1] < by_lead[3] and (by_lead[15:] == 0).all(), by_lead
    assert covered[len(s):].mean() > 0.98


@pytest.mark.parametrize("lanes", (4, 16))
def test_rate8_matrix_in_lockstep(oracle, shim, lanes):
    """The same with lanes that vote: whether the matrix is taken, whether all are zero blocks, whether some lane is near its
    budget and whether some goes on past four steps is decided for all of them.  Wavefronts of blocks that the matrix covers, alone
    and with zero blocks, with one other block (an uncommon exponent byte, no empty plane, a crowded first plane after
    one, many empty planes), with constant blocks, whose steps are many, of zero blocks only and of any blocks."""
    shim.zc_host_matrix8.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p, ctypes.c_void_p]
    shim.zc_host_matrix8_wave.argtypes = shim.zc_host_matrix8.argtypes + [ctypes.c_int]
    rng = np.random.default_rng(800 + lanes)
    ordinary = oracle.compress(workloads.gradient_lowrank(64, 1024).reshape(-1), 8).reshape(-1, 4)
    alone = np.zeros(len(ordinary), dtype=np.uint8)
    assert shim.zc_host_matrix8(1, 0, ordinary.ctypes.data, len(ordinary), np.zeros(4 * len(ordinary), np.float32).ctypes.data,
                                alone.ctypes.data) == 0
    ordinary = ordinary[alone == 1]
    constant = oracle.compress(np.repeat(rng.standard_normal(256).astype(np.float32), 4), 8).reshape(-1, 4)
    any_block = _rate8_blocks(rng)
    def planes(first, *rest):   # a payload of 24 bits from its first ones
        bits = np.array(list(first) + list(rest) + [0] * 24, dtype=np.uint8)[:24]
        return np.packbits(bits, bitorder="little")
    other = np.concatenate([np.concatenate([[e], p])[None] for e, p in (
        (252, planes([0, 0, 1, 0, 0, 0])), (28, planes([0, 0, 1, 0, 0, 0])), (127, planes([1, 0, 0, 0])), (127, planes([0] + [1] * 12)),
        (127, planes([0] * 15 + [1])), (127, planes([0] * 24)), (255, planes([1] * 24)))]).astype(np.uint8)
    def wave(kind):
        w = ordinary[rng.integers(0, len(ordinary), size=lanes)].copy()
        at = rng.permutation(lanes)
        if kind == "zeros":     # with and without a payload
            zero = at[:rng.integers(1, lanes)]
            w[zero, 0] = 0
            w[zero[::2], 1:] = 0
        elif kind == "other":
            w[at[0]] = other[rng.integers(0, len(other))]
        elif kind == "constant":
            n = rng.integers(1, lanes + 1)
            w[at[:n]] = constant[rng.integers(0, len(constant), size=n)]
        elif kind == "none":
            w[:, 0] = 0
        elif kind == "any":
            w = any_block[rng.integers(0, len(any_block), size=lanes)].copy()
            w[rng.random(lanes) < 0.3, 0] = 0
        return w
    kinds = ["ordinary", "zeros", "other", "constant", "none", "any"] * 24
    rows = np.ascontiguousarray(np.concatenate([wave(k) for k in kinds]))
    n = len(rows)
    with np.errstate(all="ignore"):
        y = oracle.decompress(rows.reshape(-1), 4 * n, 8)
        start = (rng.standard_normal(4 * n) * np.ldexp(1.0, rng.integers(-140, 120, size=4 * n))).astype(np.float32)
        start[::9], start[4::9] = 0.0, -0.0
        want = start + y
    covered = np.zeros(n, dtype=np.uint8)
    for first, stream in ((1, 0), (0, 0), (0, 1)):
        got = start.copy()
        assert shim.zc_host_matrix8_wave(first, stream, rows.ctypes.data, n, got.ctypes.data, covered.ctypes.data, lanes) == 0
        expect = y if first else want
        ok = (got.view(np.uint32) == expect.view(np.uint32)) | (np.isnan(got) & np.isnan(expect)) | ((stream != 0) & (got == 0) & (expect == 0))
        assert ok.all(), (first, stream, np.flatnonzero(~ok)[:5], kinds[np.flatnonzero(~ok)[0] // 4 // lanes])
    by_wave = covered.reshape(-1, lanes)
    assert (by_wave == by_wave[:, :1]).all()
    share = {k: by_wave[[j for j, kind in enumerate(kinds) if kind == k], 0].mean() for k in set(kinds)}
    assert share["ordinary"] > 0.75 and share["zeros"] > 0.75, share
    assert share["other"] < 0.2 and share["none"] == 0 and 0 <= share["constant"] < 0.75, share
