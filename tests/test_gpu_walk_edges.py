"""The walk of the kernels and the short arithmetic of the update pass at the places where they can go wrong: sizes around groups,
tiles, units and chunks, launches small enough to finish by tickets and tensors large enough for several epilogue
workgroups, scales around the ends of the range in which the update takes its short root and division.  Everything is held to the
CPU oracle bit for bit."""
import numpy as np
import pytest
import torch

import oracle as O
import parity as P
import tame_cases
from conftest import say
from paper_2310_18313_amd import binding as B
from paper_2310_18313_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

SIZES = {
    "one small": [4095],                                               # tickets, a single unit
    "small": [1, 15, 16, 17, 0, 240, 241, 4096, 4097, 33],             # tickets, several tensors
    "edges": [4095, 8191, 8192, 8193, 12289, 16383, 16384, 16385, 20481, 32783, 0, 1],
    "many": [(37 * i) % 601 for i in range(300)],                      # chunks of one tile
    "large": [512 * 16384 + 4097, 5, 2 * 512 * 16384 - 1],             # two and three workgroups combine the records
}


@pytest.mark.parametrize("sizes", SIZES)
@pytest.mark.parametrize("dtype,own", [(torch.bfloat16, False), (torch.float32, True), (torch.float32, False)])
def test_sizes_around_groups_tiles_units_and_chunks(sizes, dtype, own):
    lay = synth.Layout([f"t{i}" for i in range(len(SIZES[sizes]))], SIZES[sizes])
    wl = synth.Workload(sizes, lay, lr=1e-3, sigma=None)
    st, w0 = P.make_state(wl, 11)
    ids = list(range(lay.n_tensors))
    P.check_init_master(st, w0, ids)
    grad = torch.zeros(max(lay.total, 16), dtype=dtype, device=DEV)
    for step in (1, 2, 3):
        synth.fill_gradients(grad, wl, 11, step)
        hp = B.adam_hparams(1e-3, step)
        snaps = [P.Snapshot(st, grad, t) for t in ids]
        say(f"sizes {sizes} {dtype} own_moment_pass={own} step={step}")
        st.step(grad, hp, speculative=step > 1, own_moment_pass=own)
        torch.cuda.synchronize()
        P.check_step(st, snaps, hp, what=f"{sizes} step {step}")


@pytest.mark.parametrize("hp", tame_cases.HPS)
@pytest.mark.parametrize("gfmt,master,vfmt", [(B.E5M2, B.STATE_F16, B.STATE_F16), (B.E4M3, B.STATE_F32, B.STATE_F16),
                                              (B.E5M2, B.STATE_BF16, B.STATE_E4M3)])
def test_update_around_the_ends_of_the_short_arithmetic(hp, gfmt, master, vfmt):
    """700 tensors of 4112 random codes, zeros of both signs among them, a tile and a group each, with scales drawn from ordinary
    ones to well past every bound of the range in which the short root and division are taken (which tensors are inside, and
    that every bound is met from both sides, is checked without a GPU)."""
    rng = np.random.default_rng(5)
    nt, n = tame_cases.N_TENSORS, 4112
    lay = synth.Layout([f"t{i}" for i in range(nt)], [n] * nt)
    st, _ = P.make_state(synth.Workload("scales", lay, lr=1e-3), 0, gfmt, master_fmt=master, v_fmt=vfmt)
    total = lay.total
    top = 0x7B if gfmt == B.E5M2 else 0x7E

    def codes8(hi, signed=True):
        c = rng.integers(0, hi + 1, total).astype(np.uint8)
        c[rng.random(total) < 0.1] = 0
        return c | (rng.integers(0, 2, total).astype(np.uint8) << 7 if signed else 0)

    def halves(signed):
        c = rng.integers(0, 0x7C00, total).astype(np.uint16)
        c[rng.random(total) < 0.1] = 0
        return c | (rng.integers(0, 2, total).astype(np.uint16) << 15 if signed else 0)

    host = dict(g8=codes8(top), m=codes8(0x7E), v=halves(False) if vfmt == B.STATE_F16 else codes8(0x7E, False))
    if master == B.STATE_F16:
        host["w"] = halves(True)
    else:
        w = (rng.standard_normal(total) * 10.0 ** rng.uniform(-6, 1, total)).astype(np.float32)
        host["w"] = w.view(np.uint32) if master == B.STATE_F32 else (w.view(np.uint32) >> 16).astype(np.uint16)
    ints = {1: np.uint8, 2: np.int16, 4: np.int32}
    for k in ("g8", "m", "v", "w"):
        t = getattr(st, k)
        t.view({1: torch.uint8, 2: torch.int16, 4: torch.int32}[t.element_size()])[:total].copy_(
            torch.from_numpy(host[k].view(ints[t.element_size()])))
    metas = {k: B.meta_to_numpy(getattr(st, k), nt) for k in ("g_meta", "m_meta", "v_meta", "w_meta", "q_meta")}
    payload = {"g_meta": 57344.0 if gfmt == B.E5M2 else 448.0, "m_meta": 448.0, "v_meta": 65504.0 if vfmt == B.STATE_F16 else 448.0,
               "w_meta": 65504.0 if master == B.STATE_F16 else 100.0}
    for k, scale in tame_cases.scales(hp, master).items():
        metas[k]["scale"], metas[k]["inv_scale"] = scale, np.float32(1.0) / scale
        metas[k]["amax_deq"] = np.float32(payload[k]) * metas[k]["inv_scale"]
    for k, mt in metas.items():
        setattr(st, k, B.meta_from_numpy(mt, DEV))
    h = B.adam_hparams(**tame_cases.HPS[hp], master_fmt=master, v_fmt=vfmt)
    say(f"scales at the ends: {hp} gfmt={gfmt} master={master} v={vfmt}")
    st.adam(h)
    torch.cuda.synchronize()
    wq = np.zeros(total, np.uint8)
    O.adam_step_fp8(O.tensors_array(lay.tensors()), host["g8"], gfmt, metas["g_meta"], host["m"], metas["m_meta"], host["v"],
                    metas["v_meta"], host["w"], metas["w_meta"], wq, metas["q_meta"], P.oracle_hp(h))
    inside = np.zeros(total, bool)
    for off, k in lay.tensors():
        inside[off:off + k] = True
    for name, ref in (("m", host["m"]), ("v", host["v"]), ("w", host["w"]), ("wq", wq)):
        got = P._host_bits(getattr(st, name), 0, total)
        bad = np.flatnonzero((got != ref) & inside)
        assert bad.size == 0, f"{name}: {bad.size} differ, first in tensor {bad[0] // 4352}"
    for k in ("m_meta", "v_meta", "w_meta", "q_meta"):
        got = B.meta_to_numpy(getattr(st, k), nt)
        for t in range(nt):
            diff = P.meta_equal(got[t], metas[k][t], ["scale", "inv_scale", "amax", "amax_deq", "flags"])
            assert not diff, (k, t, diff, got[t], metas[k][t])


def test_static_step_with_more_chunks_than_its_table_holds():
    """The step without a context enlarges its chunks when the list has more than 65 536 of the usual size: the same bytes as
    a context, whose chunks stay small."""
    n = 65536 * 16384 + 4097
    lay = synth.Layout(["big", "tail"], [n, 70001])
    gen = torch.Generator(device=DEV)
    gen.manual_seed(3)
    code = lambda: torch.randint(0, 256, (lay.total,), dtype=torch.uint8, device=DEV, generator=gen) & 0xF7
    half = lambda lo: torch.randint(lo, 0x7000, (lay.total,), dtype=torch.int16, device=DEV, generator=gen).view(torch.float16)
    g, m, v, w = code(), code(), half(0), half(0)
    ctx, cfg = B.Context(lay.tensors()), B.autoscale_cfg()
    metas = []
    for s, top in ((2.0 ** 20, 57344.0), (2.0 ** 16, 448.0), (2.0 ** 40, 65504.0), (2.0 ** 12, 65504.0), (1.0, 0.0)):
        a = B.meta_to_numpy(ctx.new_meta(cfg), 2)
        a["scale"], a["inv_scale"], a["amax_deq"] = s, 1.0 / s, top / s
        metas.append(a)
    out = []
    hp = B.adam_hparams(3e-4, 10)
    for static in (False, True):
        b = [g, m.clone(), v.clone(), w.clone(), torch.zeros(lay.total, dtype=torch.uint8, device=DEV)]
        mt = [B.meta_from_numpy(a, DEV) for a in metas]
        args = (b[0], B.E5M2, mt[0], b[1], mt[1], b[2], mt[2], b[3], mt[3], b[4], mt[4], hp)
        say(f"1.07e9 parameters, static={static}")
        if static:
            B.adam_step_fp8_static(lay.tensors(), *args)
        else:
            ctx.adam_step_fp8(*args)
        torch.cuda.synchronize()
        out.append((b, mt))
    for x, y in zip(out[0][0], out[1][0]):
        assert torch.equal(x.view(torch.uint8), y.view(torch.uint8))
    for x, y in zip(out[0][1], out[1][1]):
        assert torch.equal(x, y)
