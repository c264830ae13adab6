"""The split planner, checked on the CPU: its items, packed fragments, masks,
clamps and item orders replayed in 64 bits against direct dot products
(split_replay.cpp), in the tiled and the series-lane layout, over the forms
that univariate plans accept: every length, centred and other paddings, one to
33 kernels of a dilation, O down to 1, and generated sets."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

import paper_2601_17091_amd as rk
from paper_2601_17091_amd import rocket
from _util import full_dilations_set, kernel_set, many_widths_set

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2601_17091_amd", "csrc")


@pytest.fixture(scope="module")
def replay_lib(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("g++ is needed to build the replay")
    so = str(tmp_path_factory.mktemp("replay") / "split_replay.so")
    subprocess.run([gxx, "-std=c++17", "-O2", "-g", "-shared", "-fPIC", "-ffp-contract=off", "-D_GLIBCXX_ASSERTIONS",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(HERE, "split_replay.cpp"),
                    os.path.join(CSRC, "plan_split.cpp"), os.path.join(CSRC, "plan.cpp"),
                    os.path.join(CSRC, "generate.cpp"), os.path.join(CSRC, "minirocket.cpp"), "-o", so], check=True)
    return ctypes.CDLL(so)


@pytest.fixture(scope="module")
def replay(replay_lib):
    lib = replay_lib

    def run(ks, L, series, seed=0, may_refuse=False, with_forms=False):
        x = np.random.default_rng(seed).standard_normal(L).astype(np.float32)
        c, keep = rocket.as_c_kernels(ks)
        where, items, forms = ctypes.c_int32(), ctypes.c_int32(), ctypes.c_int32()
        rc = lib.split_replay(ctypes.byref(c), L, x.ctypes.data_as(ctypes.POINTER(ctypes.c_float)), int(series),
                              ctypes.byref(where), ctypes.byref(items), ctypes.byref(forms))
        if may_refuse and rc == 1:
            return 0
        assert rc == 0, "check %d failed at kernel %d" % (rc, where.value)
        return (items.value, forms.value) if with_forms else items.value

    return run


@pytest.mark.parametrize("L", [11, 16, 63, 64, 65, 127, 128])
def test_generated_short(replay, L):
    ks = rk.generate_kernels(4000 + L, 1500, L)
    for series in (False, True):
        assert replay(ks, L, series) > 0


@pytest.mark.parametrize("L", [129, 193, 257, 1021, 6465, 20255])
def test_generated(replay, L):
    assert replay(rk.generate_kernels(3000 + L, 400 if L < 4000 else 1500, L), L, False) > 0


@pytest.mark.parametrize("L", [41, 131, 321])
def test_lengths_and_paddings(replay, L):
    """Items of several lengths, even ones among them, of three and four
    widths, and of kernels with one output."""
    ks = many_widths_set(L, L)
    for series in ((False, True) if L <= 128 else (False,)):
        items, forms = replay(ks, L, series, with_forms=True)
        assert items > 0 and forms == 15


@pytest.mark.parametrize("count", [1, 2, 15, 31, 32, 33, 65])
def test_kernels_per_dilation(replay, count):
    for L, dilations in ((100, range(1, 9)), (400, range(1, 13))):
        items = replay(full_dilations_set(L, count, count, dilations), L, L == 100)
        # a handful of kernels a dilation is left to fp32 items
        assert items >= 2 * len(dilations) * (3 * count // 64) and (items > 0) == (count >= 15)


@pytest.mark.parametrize("L,d,series", [(100, 1 << 16, True), (100, 1 << 22, True), (128, 1 << 24, True),
                                        (200, 1 << 16, False), (200, 1 << 28, False), (500, 1 << 30, False)])
def test_far_taps(replay, L, d, series):
    """Dilations far beyond the series, with paddings to match: an outer tap
    reads padding at every output, never the series (a kernel's byte addresses
    have 32 bits).  Such sets either have right items or run in fp32."""
    rng = np.random.default_rng(d % 1000003 + L)
    ln = [3] * 40 + [9 if d < 1 << 28 else 3] * 40
    pad = [(n - 1) * d // 2 for n in ln]
    ks = kernel_set(ln, [d] * len(ln), pad, rng.uniform(-1, 1, len(ln)), [rng.standard_normal(n) for n in ln])
    replay(ks, L, series, may_refuse=d > 1 << 16)


@pytest.mark.parametrize("L,series", [(100, True), (400, False)])
def test_tiny_biases(replay, L, series):
    """Kernels with zero or tiny biases are left to fp32 items (short series:
    then all are); the others keep theirs."""
    ks = rk.generate_kernels(11, 1500, L)
    assert replay(ks, L, series) > 0
    ks["bias"][::7] = np.array([0.0, -0.0, 1e-40, -1e-31, 2.0 ** -101], np.float32)[np.arange(215) % 5]
    assert (replay(ks, L, series) > 0) == (L > 128)
    ks["bias"][:] = 0.0
    assert replay(ks, L, series) == 0


@pytest.mark.parametrize("L", [100, 400])
def test_places_do_not_depend_on_the_order_of_the_set(replay_lib, L):
    """Kernels that agree in their bias and their first weights (one length a
    prefix of another), or in all but their padding: each keeps its slot,
    whatever the order of the set."""
    rng = np.random.default_rng(L)
    first = rng.standard_normal(7)
    ln, pad, w = [], [], []
    for length in (7, 9, 11):
        for i in range(60):
            ln.append(length)
            pad.append(int(rng.integers(0, 3)) * (length - 1) // 2)
            w.append(np.concatenate([first, (i // 2) * 0.25 + np.arange(length - 7)]))
    ks = kernel_set(ln, [1] * len(ln), pad, np.full(len(ln), 0.5), w)

    def places(order):
        sub = {f: np.ascontiguousarray(ks[f][order]) for f in ("length", "dilation", "padding", "bias", "weights")}
        c, keep = rocket.as_c_kernels(sub)
        place = np.empty(len(order), np.int32)
        assert replay_lib.split_places(ctypes.byref(c), L, place.ctypes.data_as(ctypes.POINTER(ctypes.c_int32))) == 0
        return place

    # equal kernels may trade places: compare what sits in each slot
    key = [(ks["length"][i], ks["padding"][i], ks["weights"][i].tobytes()) for i in range(len(ln))]
    want = {p: key[i] for i, p in enumerate(places(np.arange(len(ln))))}
    assert len(want) > 32 and -1 not in want
    for _ in range(5):
        order = rng.permutation(len(ln))
        assert {p: key[order[i]] for i, p in enumerate(places(order))} == want
