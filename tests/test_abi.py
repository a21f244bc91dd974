"""CPU-side checks of the C ABI: the library builds for gfx950, loads, exports
every entry point include/pft.h declares, and its host-only logic (contour
plan, argument validation) behaves without touching a GPU."""
import ctypes
import os
import re

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def pft():
    from paper_1204_5434_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_1204_5434_amd import build
        build.build()
    return binding


def declared_functions():
    text = open(os.path.join(ROOT, "include", "pft.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(pft_[a-z0-9_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported(pft):
    lib = pft.load()
    names = declared_functions()
    assert len(names) >= 15
    for name in names:
        assert hasattr(lib, name), name
    assert set(names) == set(pft.EXPORTS)


@pytest.mark.parametrize("ns,f", [(50, 0.5), (128, 0.3), (100, 0.4), (40, 0.33), (7, 0.05), (9, 0.95),
                                  (200, 0.35), (61, 0.4731)])
def test_contour_plan_matches_oracle(pft, orc, ns, f):
    h, blk, J = pft.pft_contour_plan(ns, f)
    ho, bo, Jo = orc.contour(ns, f)
    assert J == Jo and np.array_equal(blk, bo)
    assert np.array_equal(h, ho)


def test_create_rejects_bad_parameters(pft):
    lib = pft.load()
    h = ctypes.c_void_p()
    bad = [dict(f=0.0), dict(f=1.0), dict(ns=1), dict(lx=0.0), dict(C=-1.0), dict(chiN=0.0),
           dict(precision=7), dict(scheme=3)]
    for kw in bad:
        p = pft.Params(16, 16, 16, 4.0, 4.0, 4.0, 50, 0.5, 15.0)
        for k, v in kw.items():
            setattr(p, k, v)
        assert lib.pft_create(ctypes.byref(p.c()), None, ctypes.byref(h)) == pft.PFT_E_INVALID, kw
        assert not h.value
    for n in (14, 28, 100, 7):
        p = pft.Params(16, 16, n, 4.0, 4.0, 4.0, 50, 0.5, 15.0)
        assert lib.pft_create(ctypes.byref(p.c()), None, ctypes.byref(h)) == pft.PFT_E_UNSUPPORTED
    assert lib.pft_create(None, None, ctypes.byref(h)) == pft.PFT_E_INVALID


def test_null_context_and_plan_errors(pft):
    lib = pft.load()
    assert lib.pft_propagate(None, None, None) == pft.PFT_E_INVALID
    assert lib.pft_densities(None, None, None, None) == pft.PFT_E_INVALID
    assert lib.pft_num_steps(None) == -1
    assert lib.pft_status_string(pft.PFT_E_STATE) == b"PFT_E_STATE"
    h = np.zeros(4)
    b = np.zeros(4, np.int32)
    J = np.zeros(1, np.int32)
    assert lib.pft_contour_plan(1, 0.5, h.ctypes.data, b.ctypes.data, J.ctypes.data) == -1
    assert lib.pft_contour_plan(3, 1.5, h.ctypes.data, b.ctypes.data, J.ctypes.data) == -1
    assert lib.pft_noise_words(0, 0, 0, 0, 0, None, None) == pft.PFT_E_INVALID


def test_tuning_file_leaves_untuned_lengths_untuned(pft, tmp_path):
    """A saved table says what was tuned and what was not, so that a process that
    loads it chooses the same kernels as the one that saved it."""
    def saved(name):
        pft.pft_tune_save(str(tmp_path / name))
        lines = [l.split() for l in open(tmp_path / name)]
        return lines[0][0], {tuple(map(int, l[1:4])): int(l[4]) for l in lines}

    def load(entries):
        path = tmp_path / "entries"
        path.write_text("".join(f"{arch} {p} {n} {k} {v}\n" for (p, n, k), v in entries.items()))
        pft.pft_tune_load(str(path))

    arch, before = saved("before")
    every = {(p, n, k) for p in (0, 1) for n in pft.SUPPORTED_AXES for k in range(3)}
    assert set(before) == every
    load(dict.fromkeys(every, -1))
    assert set(saved("none")[1].values()) == {-1}
    tuned = {(0, 24, 0): 1, (1, 128, 2): 0}
    load(tuned)
    _, table = saved("some")
    assert {k: v for k, v in table.items() if v != -1} == tuned
    load({(0, 24, 0): 3, (1, 100, 0): -1, (0, 32, 0): -2})  # no such variant, length or variant
    assert saved("same")[1] == table
    load(dict.fromkeys(every, -1))
    pft.pft_tune_load(str(tmp_path / "some"))
    assert saved("again")[1] == table
    pft.pft_tune_load(str(tmp_path / "before"))
    assert saved("end")[1] == before
