"""What the library launches, seen on the CPU: the host side on a HIP runtime that only takes notes (launch_notes.cpp)."""
import ctypes as C
import re

import pytest

import launch_notes_build
from paper_2310_18313_amd import binding as B

CUS = 256
FREE = 1 << 30                      # single_pass_min_chunks: the library chooses
LISTS = {
    "one small": [4095],
    "ragged": [(37 * i) % 9001 for i in range(400)],
    "mixed": [70001, 1, 4096, 333, 0, 16385, 3000000, 17],
    "large": [1 << 28, 5, 123456789],
}


class Library:
    """The library on the noting runtime, with calls on pointers that nothing follows."""
    P = 1 << 20

    def __init__(self, L):
        self.L = L
        L.notes_kernel.restype = C.c_char_p
        self.cfg, self.metas = B.autoscale_cfg(), [self.P + 4096 * i for i in range(1, 6)]

    def context(self, numels, tuning=None):
        arr, at = (B.Tensor * max(1, len(numels)))(), 0
        for a, n in zip(arr, numels):
            a.offset, a.numel = at, n
            at += (n + 15) // 16 * 16
        self.arr, self.n = arr, len(numels)
        h = C.c_void_p()
        assert self.L.fp8lm_create(C.byref(h), C.cast(arr, C.c_void_p), len(numels), 0) == 0
        if tuning:
            assert self.L.fp8lm_set_tuning(h, *tuning) == 0
        return h

    def hp(self, **kw):
        return B.adam_hparams(1e-3, 1, **kw)

    def calls(self, h):
        """Every entry point that walks the tensors: name -> the call."""
        L, P, cfg = self.L, self.P, C.addressof(self.cfg)
        g, m, v, w, q = self.metas
        far = 1 << 40
        ptrs = (C.c_void_p * 12)(*[P] * 12)
        out = {}
        for s in (B.SRC_BF16, B.SRC_F32):
            out[f"amax {s}"] = lambda s=s: L.fp8lm_amax_scale(h, P, s, B.E5M2, g, cfg, None)
            out[f"cast {s}"] = lambda s=s: L.fp8lm_cast_fp8(h, P, s, P, B.E5M2, g, cfg, None)
            out[f"delayed {s}"] = lambda s=s: L.fp8lm_cast_fp8_delayed(h, P, s, P, B.E5M2, g, cfg, None)
            out[f"quantize {s}"] = lambda s=s: L.fp8lm_quantize_fp8(h, P, s, P, B.E5M2, g, cfg, None)
            out[f"quantize for adam {s}"] = lambda s=s: L.fp8lm_quantize_fp8_for_adam(h, P, s, P, B.E5M2, g, cfg, P, m, 0.9, None)
            out[f"error stats {s}"] = lambda s=s: L.fp8lm_quant_error_stats(h, P, s, P, B.E5M2, g, P, None)
        out["requantize"] = lambda: L.fp8lm_requantize_fp8(h, P, B.E4M3, g, P, P, m, None)
        for r in (1, 3, 8, 12):
            out[f"sum {r}"] = lambda r=r: L.fp8lm_sum_fp8(h, C.cast(ptrs, C.c_void_p), r, B.E4M3, P, P, g, cfg, None)
        for name, hp in (("adam", self.hp()), ("adam stats", self.hp(stats=1)), ("adam fp32", self.hp(master_fmt=B.STATE_F32)),
                         ("adam predicted", self.hp(m_scale_mode=B.MSCALE_PREDICTED))):
            out[name] = lambda hp=hp: L.fp8lm_adam_step_fp8(h, P, B.E5M2, g, P, m, P, v, P, w, P, q, C.addressof(hp), None)
        hp0 = self.hp()
        out["adam pair"] = lambda: L.fp8lm_adam_step_fp8_m2(h, P, B.E5M2, g, P, P + far, m, P, v, P, w, 2 * P, q, C.addressof(hp0), None)
        out["init"] = lambda: L.fp8lm_init_master(h, P, P, w, None)
        return out

    def notes(self, call):
        """The launches of a call: (kernel, grid, tables or None)."""
        self.L.notes_clear()
        assert call() == 0
        out = []
        for i in range(self.L.notes_count()):
            v = (C.c_int64 * 7)()
            self.L.notes_launch(i, C.byref(v))
            name = re.sub(r"^_ZN5fp8lm\d+([a-z0-9_]+?)_kernel.*$", r"\1", self.L.notes_kernel(i).decode())
            out.append((name, v[0], dict(zip(("unit_elems", "unit_shift", "one_unit", "deferred", "n_chunks"), v[2:])) if v[1] else None))
        return out


@pytest.fixture()
def lib(monkeypatch):
    monkeypatch.setattr(B, "LIB_PATH", launch_notes_build.build())
    monkeypatch.setattr(B, "_lib", None)
    return Library(B.lib())


# kernels whose grid follows the tensors' elements (the others are a thread, a wavefront or a workgroup per tensor)
WALKS = {"amax", "cast", "cast_marked", "requantize", "sum_fp8", "adam_amax", "adam_update", "adam_update_var", "adam_moment_redo",
         "init_master_cast", "quant_stats", "skeleton"}


@pytest.mark.parametrize("sizes", LISTS)
@pytest.mark.parametrize("limit", [1, 3, 15])
def test_a_limit_on_workgroups_holds_for_every_launch(lib, sizes, limit):
    h = lib.context(LISTS[sizes], (16384, limit, FREE))
    seen = set()
    for what, call in lib.calls(h).items():
        for name, grid, _ in lib.notes(call):
            seen.add(name)
            if name in WALKS:
                assert 1 <= grid <= limit * CUS, (what, name, grid)
    bufs = (C.c_void_p * 5)(*[lib.P] * 5)
    for shape in range(B.SKEL_UPDATE_RANGES + 1):
        for name, grid, _ in lib.notes(lambda: lib.L.fp8lm_memory_skeleton(h, shape, C.cast(bufs, C.c_void_p), 4096 * 12345, None)):
            seen.add(name)
            assert 1 <= grid <= limit * CUS, (shape, name, grid)
    assert seen >= WALKS
    lib.L.fp8lm_destroy(h)


@pytest.mark.parametrize("sizes", LISTS)
def test_a_caller_chooses_how_statistics_are_combined(lib, sizes):
    """single_pass_min_chunks = 0: never a second launch, not in the second round of a speculation either, and no more
    tickets than a persistent grid has workgroups.  More than a workgroup ever has: always a second launch.  In between: the
    chunks per workgroup of the grid that is launched decide."""
    chunks = sum((n + 16383) // 16384 for n in LISTS[sizes])
    for per_cu in (16, 7, 1):
        for least in (0, 2, 5, FREE - 1):
            h = lib.context(LISTS[sizes], (16384, per_cu, least))
            for what, call in lib.calls(h).items():
                if "error stats" in what:                          # sums in a fixed order: always a second launch
                    continue
                notes = lib.notes(call)
                combining = [n for n in notes if n[0] in WALKS and n[0] != "adam_moment_redo"]    # that one finds nothing out
                for name, grid, tables in combining:
                    if name != "cast_marked":                      # decides as the cast before it
                        deferred = least > 0 and chunks // grid < least
                    assert tables["deferred"] == deferred, (what, name, grid, tables)
                    assert least > 0 or grid <= min(16 * CUS, max(256, chunks)), (what, name, grid)
                assert [n[0] for n in notes].count("epilogue") == sum(t["deferred"] for _, _, t in combining), (what, notes)
            lib.L.fp8lm_destroy(h)


def test_the_library_takes_tickets_for_the_smallest_launches_only(lib):
    for numel, tickets in ((64 * 4096, True), (64 * 4096 + 1, False), (1 << 28, False)):
        h = lib.context([numel])
        (name, grid, tables), *rest = lib.notes(lib.calls(h)["requantize"])
        assert name == "requantize" and grid == tables["n_chunks"] << tables["unit_shift"]
        assert tables["one_unit"] and bool(tables["deferred"]) is not tickets and len(rest) == (0 if tickets else 1)
        lib.L.fp8lm_destroy(h)


@pytest.mark.parametrize("sizes", LISTS)
def test_both_rounds_of_a_speculation_cut_the_tensors_alike(lib, sizes):
    """The first round marks a tensor with the number of its units, the second deals these units out."""
    for tuning in (None, (4096, 16, FREE), (12288, 16, 0), (1 << 20, 5, FREE)):
        h = lib.context(LISTS[sizes], tuning)
        for what, call in lib.calls(h).items():
            if what.split()[0] not in ("quantize",) and what != "adam pair":
                continue
            walks = [t for name, _, t in lib.notes(call) if name in WALKS]
            assert len(walks) == 2, what
            assert [(t["unit_elems"], t["unit_shift"]) for t in walks[1:]] == [(walks[0]["unit_elems"], walks[0]["unit_shift"])], (what, walks)
        lib.L.fp8lm_destroy(h)


@pytest.mark.parametrize("src,size", [(B.SRC_F32, 4), (B.SRC_BF16, 2)])
def test_amax_passes_of_a_gibibyte_walk_ranges(lib, src, size):
    """(A workgroup per unit is the faster form below, a persistent grid from there on; both leave the same results.)"""
    for numel, ranges in (((1 << 30) // size - 16384, False), ((1 << 30) // size, True)):
        h = lib.context([numel])
        (name, grid, tables), _ = lib.notes(lib.calls(h)[f"amax {src}"])
        assert name == "amax" and bool(tables["one_unit"]) is not ranges
        assert grid == (16 * CUS if ranges else tables["n_chunks"] << tables["unit_shift"])
        lib.L.fp8lm_destroy(h)
