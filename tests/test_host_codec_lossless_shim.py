"""The per-lane pieces of the lossless codec that the GPU runs (csrc/zl_codec.h), compiled
for the host and compared group by group with the reference's stage functions."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2409_02423_amd import workloads

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "shim", "zl_codec_host.cpp")
LIB = os.path.join(HERE, "shim", "libzl_codec_host.so")
HDR = os.path.join(HERE, "..", "paper_2409_02423_amd", "csrc", "zl_codec.h")


@pytest.fixture(scope="module")
def shim():
    newest = max(os.path.getmtime(f) for f in (SRC, HDR))
    if not os.path.exists(LIB) or os.path.getmtime(LIB) < newest:
        subprocess.check_call(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", SRC, "-o", LIB])
    L = ctypes.CDLL(LIB)
    L.zl_host_to_planes.argtypes = [ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p]
    L.zl_host_halves_to_planes.argtypes = L.zl_host_to_planes.argtypes
    L.zl_host_planes_of_groups.argtypes = [ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p]
    L.zl_host_from_planes.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p]
    return L


def _groups():
    rng = np.random.default_rng(11)
    parts = [workloads.edge_values(3).view(np.uint32), workloads.gradient_iid(4096).view(np.uint32),
             rng.integers(0, 1 << 32, size=4096, dtype=np.uint64).astype(np.uint32),
             (rng.integers(0, 1 << 32, size=2048, dtype=np.uint64).astype(np.uint32) & np.uint32(0xFFFF0000)),
             np.zeros(64, dtype=np.uint32), np.full(64, 0xC0490FDB, dtype=np.uint32)]
    w = np.concatenate(parts)
    return w[: w.size // 32 * 32].reshape(-1, 32).copy()


def test_planes_of_16_bit_words_match_reference(shim):
    """A group of 16-bit words v as two words to a register, against the reference on the words v << 16:
    either sign, the largest patterns in either half, equal words, zeros."""
    from oracle import zl_ref
    rng = np.random.default_rng(13)
    same = np.repeat(np.array([0x7FFF, 0xFFFF, 0x8000, 0x0000, 0xC049], dtype=np.uint16), 32)
    parts = [(workloads.activation_gelu(4096).view(np.uint32) >> np.uint32(16)).astype(np.uint16), same,
             rng.integers(0, 65536, size=4096).astype(np.uint16), rng.integers(0, 4, size=1024).astype(np.uint16)]
    for at in (0, 15, 16, 31):     # one word that stands out, in each register half's first and last place
        g = np.full(32, 0x3F80, dtype=np.uint16)
        g[at] = 0xFFFF
        parts.append(g)
    h = np.concatenate(parts).reshape(-1, 32)
    groups = len(h)
    refs, maps = np.zeros(groups, dtype=np.uint32), np.zeros(groups, dtype=np.uint32)
    planes = np.zeros((groups, 16), dtype=np.uint32)
    shim.zl_host_halves_to_planes(h.ctypes.data, groups, refs.ctypes.data, maps.ctypes.data, planes.ctypes.data)
    for g in range(groups):
        m, r = zl_ref.residuals(h[g].astype(np.uint32) << np.uint32(16))
        p = zl_ref.planes(r)
        assert refs[g] == m and not any(p[:16]) and np.array_equal(planes[g], p[16:]), g
        assert maps[g] == sum(1 << k for k in range(32) if p[k]), g


def test_plane_counts_match_reference(shim):
    """The count from which a workgroup works out the size of a chunk that it has not coded."""
    from oracle import zl_ref
    w = _groups()
    counts = np.zeros(len(w), dtype=np.uint32)
    shim.zl_host_planes_of_groups(w.ctypes.data, len(w), counts.ctypes.data)
    for g in range(len(w)):
        assert counts[g] == sum(1 for p in zl_ref.planes(zl_ref.residuals(w[g])[1]) if p), g


def test_planes_and_words_match_reference(shim):
    from oracle import zl_ref
    rng = np.random.default_rng(12)
    w = _groups()
    groups = len(w)
    refs = np.zeros(groups, dtype=np.uint32)
    maps = np.zeros(groups, dtype=np.uint32)
    planes = np.zeros_like(w)
    shim.zl_host_to_planes(w.ctypes.data, groups, refs.ctypes.data, maps.ctypes.data, planes.ctypes.data)
    for g in range(groups):
        m, r = zl_ref.residuals(w[g])
        p = zl_ref.planes(r)
        assert refs[g] == m and np.array_equal(planes[g], p), g
        assert maps[g] == sum(1 << k for k in range(32) if p[k]), g
    back = np.zeros_like(w)
    shim.zl_host_from_planes(planes.ctypes.data, refs.ctypes.data, groups, back.ctypes.data)
    assert np.array_equal(back, w)
    # planes and references that no encoder produces: same words as the reference computes
    odd = rng.integers(0, 1 << 32, size=(200, 32), dtype=np.uint64).astype(np.uint32)
    oref = rng.integers(0, 1 << 31, size=200, dtype=np.uint64).astype(np.uint32)
    shim.zl_host_from_planes(odd.ctypes.data, oref.ctypes.data, 200, back[:200].ctypes.data)
    for g in range(200):
        assert np.array_equal(back[g], zl_ref.words(int(oref[g]), zl_ref.unplanes(odd[g]))), g


@pytest.mark.parametrize("grid", [1024, 1792, 128, 8])
def test_chunk_counters_are_asked_evenly_whichever_dies_are_busy(shim, grid):
    """Workgroup b runs on die b mod 8.  As many workgroups ask each counter as any other (the last
    request is found by counting), with every die and with any one die held by another kernel, up
    to the rounding of its share, and also in the first workgroup of each die alone."""
    counters, dies = shim.zl_host_counters(), 8
    asked = np.array([shim.zl_host_counter_of(b) for b in range(grid)])
    die = np.arange(grid) % dies
    assert asked.min() >= 0 and asked.max() < counters
    assert (np.bincount(asked, minlength=counters) == grid // counters).all()
    for busy in range(dies):
        on_it = np.bincount(asked[die == busy], minlength=counters)
        assert on_it.max() - on_it.min() <= 1, busy
    assert sorted(asked[:dies]) == list(range(counters))
