"""LBSystem.import_state and export_state on the CPU: what the binding hands to
the library, which is a stand-in here."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest

import lbinputs
import paper_0903_5067_amd as lbm

BOXES = [lbinputs.box_params("plain16", L=3, N=4), lbinputs.box_params("plain16", L=2, N=0),
         lbinputs.box_params("plain16", L=4, N=2)]


class Library:
    """Keeps imported state and gives it back on export."""

    def __init__(self):
        self.step, self.packed = None, None

    def lb_state_host_bytes(self, h):
        return 8 * (1 + sum(19 * int(b["L"]) ** 3 + 12 * int(b["N"]) for b in BOXES))

    def lb_export_state(self, h, buf, nbytes):
        a = np.ctypeslib.as_array(ctypes.cast(buf, ctypes.POINTER(ctypes.c_double)), (nbytes // 8,))
        a[:1].view(np.uint64)[0], a[1:] = self.step, self.packed
        return lbm.LB_OK

    def lb_export_arrays(self, h, step, ptrs, n):
        ctypes.cast(step, ctypes.POINTER(ctypes.c_uint64))[0] = self.step
        o = 0
        for p, s in zip(ptrs, self._sizes(n)):
            if s:
                np.ctypeslib.as_array(ctypes.cast(p, ctypes.POINTER(ctypes.c_double)), (s,))[:] = self.packed[o:o + s]
            o += s
        return lbm.LB_OK

    def _sizes(self, n):
        sizes = [s for b in BOXES for s in [19 * int(b["L"]) ** 3] + 4 * [3 * int(b["N"])]]
        assert n == len(sizes)
        return sizes

    def lb_import_state(self, h, buf, nbytes):
        a = np.ctypeslib.as_array(ctypes.cast(buf, ctypes.POINTER(ctypes.c_double)), (nbytes // 8,))
        self.step, self.packed = int(a[:1].view(np.uint64)[0]), a[1:].copy()
        return lbm.LB_OK

    def lb_import_arrays(self, h, step, ptrs, n):
        parts = [np.ctypeslib.as_array(ctypes.cast(p, ctypes.POINTER(ctypes.c_double)), (s,))
                 for p, s in zip(ptrs, self._sizes(n)) if s]
        self.step, self.packed = ctypes.c_uint64(step).value, np.concatenate(parts)
        return lbm.LB_OK


@pytest.fixture
def system(monkeypatch):
    s = lbm.LBSystem.__new__(lbm.LBSystem)
    s.boxes, s.h = [dict(b) for b in BOXES], None
    s.L = Library()
    monkeypatch.setattr(lbm, "lib", lambda: s.L)
    return s


def _state(step=7):
    rng = np.random.default_rng(3)
    return {"step": step, "boxes": [{"n": rng.normal(size=(19,) + 3 * (int(b["L"]),)),
                                     **{k: rng.normal(size=(int(b["N"]), 3)) for k in ("x", "v", "f", "fc")}} for b in BOXES]}


def _packed(state):
    return np.concatenate([b[k].reshape(-1) for b in state["boxes"] for k in ("n", "x", "v", "f", "fc")])


@pytest.mark.parametrize("step", [0, 7, np.int64(12), np.uint64(2 ** 64 - 1), 3.0, np.array(9)])
def test_import_takes_step_counts(system, step):
    st = _state(step)
    system.import_state(st)
    assert system.L.step == int(step) and np.array_equal(system.L.packed, _packed(st))


@pytest.mark.parametrize("step", [-1, 2 ** 64, np.array([5]), "five", None])
def test_import_refuses_what_is_no_step_count(system, step):
    with pytest.raises((OverflowError, ValueError, TypeError)):
        system.import_state(_state(step))
    assert system.L.packed is None


def test_import_of_other_layouts(system):
    """Strides, types and shapes of the right size are taken; a list of other
    sizes goes to the library as one buffer, which it checks."""
    st = _state()
    want = _packed(st)
    b = st["boxes"][0]
    b["n"] = np.asfortranarray(b["n"])
    b["x"] = b["x"].reshape(-1)
    b["v"] = np.repeat(b["v"], 2, axis=0)[::2]
    b["f"] = b["f"].tolist()
    system.import_state(st)
    assert np.array_equal(system.L.packed, want)
    st["boxes"][2]["fc"] = np.zeros((9, 3))
    system.import_state(st)
    assert system.L.packed.size == want.size + 21


def test_exported_arrays_are_independent(system):
    """Each array owns its memory: one that is kept does not keep the others."""
    st = _state(41)
    system.import_state(st)
    got = system.export_state()
    assert got["step"] == 41
    for b, w in zip(got["boxes"], st["boxes"]):
        assert list(b) == ["n", "x", "v", "f", "fc"]
        for k, a in b.items():
            assert np.array_equal(a, w[k]) and a.shape == w[k].shape and a.dtype == np.float64
            assert a.base is None and a.flags.c_contiguous and a.flags.writeable, k
