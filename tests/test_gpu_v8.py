"""GPU parity of the PW -> DW (-> PW) kernels (k_ir8, NHWC and NCHW), forced through explicit
plans.

Every compiled variant that implements a case runs over tiles that leave ragged pixel
blocks, window tiles and image borders, with one and several groups of waves sharing a
tile's chunks and (PW -> DW) the intermediate channels split over workgroups, against the
CPU oracle. Cases cover both strides, filters, even and uneven chunks, input rows that are
not 16-byte multiples, output channels in a partial tile, padding other than half the
filter, and requantisation scales on both sides of the single-precision rule.
"""
import numpy as np
import pytest

from paper_2404_19331_amd import fcm
from paper_2404_19331_amd.workloads import Case, make_inputs

from gpu_util import assert_close, dev_inputs, oracle_ref, run_fused, to_np

pytestmark = pytest.mark.gpu

ELT = {"f32": 4, "bf16": 2, "i8": 1}
# (multiplier, shift, range): a power of two, a 15-bit and a 31-bit multiplier (the last not
# a single-precision value), about the same scales
RQ = ((1, 7, -127, 127), (20011, 22, -128, 127), (1342177283, 38, -127, 127))


def _cases():
    out = []
    shapes = {  # c_in, c_mid, c_out, k, stride, pad
        "f32": [(24, 144, 24, 3, 1, 1), (23, 36, 20, 5, 2, 1), (90, 64, 96, 3, 2, 2)],
        "bf16": [(24, 144, 24, 3, 1, 1), (40, 72, 20, 3, 2, 1), (24, 96, 20, 5, 1, 2), (70, 136, 68, 5, 2, 2),
                 (50, 64, 36, 3, 1, 0), (160, 200, 160, 3, 2, 2), (8, 16, 4, 3, 1, 1), (96, 576, 96, 3, 1, 1)],
        "i8": [(24, 144, 24, 3, 1, 1), (36, 64, 20, 3, 2, 1), (160, 208, 160, 5, 1, 2), (64, 384, 64, 3, 1, 0),
               (16, 48, 4, 5, 2, 4), (100, 320, 96, 3, 2, 2)],
    }
    nchw = {
        "f32": [(24, 144, 24, 3, 1, 1), (23, 36, 30, 3, 2, 1), (96, 64, 17, 3, 1, 0), (50, 100, 64, 5, 1, 2),
                (16, 20, 7, 5, 2, 4)],
        "bf16": [(24, 144, 24, 3, 1, 1), (150, 200, 37, 3, 2, 2)],
        "i8": [(24, 144, 24, 3, 1, 1), (100, 320, 33, 3, 2, 1)],
    }
    every = [(dt, "nhwc", sh) for dt, shp in shapes.items() for sh in shp]
    every += [(dt, "nchw", sh) for dt, shp in nchw.items() for sh in shp]
    for dt, layout, (ci, cm, co, k, s, pad) in every:
        for op in ("pw_dw", "pw_dw_pw"):
            act = [("relu6", "relu", "none"), ("none", "relu6", "relu")][len(out) // 2 % 2]
            out.append(Case(op, 2, 13, 11, ci, cm, co if op == "pw_dw_pw" else cm, k, s, pad, dt, layout, act,
                            RQ[len(out) % 3:] + RQ[:len(out) % 3], dist_x="i8small" if dt == "i8" else "n01",
                            dist_w="i8small", bias=True, seed=4100 + len(out),
                            name="v8-%s-%s-%s-%d-%d-%d-k%ds%dp%d" % (op, dt, layout, ci, cm, co, k, s, pad)))
    return out


CASES = _cases()


def _plans(case):
    desc = fcm.desc_from_case(case)
    mc = 64 // ELT[case.dtype]
    nch = -(-case.c_mid // mc)
    plans = []
    for v in range(fcm.lib().fcm_variant_count()):
        kernel = "k_ir8" if case.layout == "nhwc" else "k_pwdw8" if case.op == "pw_dw" else "k_pwdwpw8"
        if not fcm.variant_name(v).startswith("%s<%s,%d,%d," % (kernel, case.dtype, case.k, case.stride)):
            continue
        for th, tw in ((7, 7), (8, 16), (3, 5), (1, 11), (4, 4), (13, 2)):
            for groups in (1, 2, 8):
                blocks = sorted({nch, -(-nch // 2), 1}) if case.op == "pw_dw" else [0]
                for b in blocks:
                    cob = b * mc if b else -(-case.c_out // 16) * 16
                    try:
                        plans.append(fcm.plan_evaluate(case.op, desc, th, tw, mc, cob, v, splits=groups))
                    except fcm.FcmError:
                        pass
    return plans


@pytest.mark.parametrize("case", CASES, ids=lambda c: c.name)
def test_every_variant_tile_and_group(case):
    inp = make_inputs(case)
    ref = oracle_ref(case, inp)
    d = dev_inputs(inp, case.dtype)
    plans = _plans(case)
    assert plans and (any(p.splits > 1 for p in plans) or case.c_mid <= 64)
    for p in plans:
        print(case.name, fcm.variant_name(p.variant), p.tile_h, p.tile_w, p.co_block, p.splits, flush=True)
        got = to_np(run_fused(case, d, plan=p))
        assert_close(got, ref, case.dtype, "%s %s %dx%d block %d groups %d" % (
            case.name, fcm.variant_name(p.variant), p.tile_h, p.tile_w, p.co_block, p.splits))


def test_planner_takes_them_and_leaves_the_rest():
    case = next(c for c in CASES if c.dtype == "bf16")
    assert fcm.variant_name(fcm.plan("pw_dw", fcm.desc_from_case(case)).variant).startswith("k_ir8")
    for other in (case.with_(layout="nchw"), case.with_(c_mid=143, c_out=143), case.with_(c_in=25)):
        assert not fcm.variant_name(fcm.plan("pw_dw", fcm.desc_from_case(other)).variant).startswith("k_ir8")


@pytest.mark.parametrize("op", ["pw_dw", "pw_dw_pw"])
@pytest.mark.parametrize("act", ["none", "relu", "relu6"])
def test_non_finite_values_stay_in_their_channel(op, act):
    """bf16: an intermediate channel that overflows to infinity, or holds NaN, leaves the
    depthwise results of the others alone (NaN passes without an activation, becomes 0 with
    one, as in the other kernels of these modules)."""
    import torch

    ci, cm, co, h = 16, 64, 16, 9
    g = torch.Generator().manual_seed(5)
    x = torch.randn(1, h, h, ci, generator=g).bfloat16().cuda()
    w1 = torch.randn(cm, ci, generator=g).bfloat16().cuda()
    wd = torch.randn(cm, 3, 3, generator=g).bfloat16().cuda()
    w2 = torch.randn(co, cm, generator=g).bfloat16().cuda()
    b1 = torch.zeros(cm, device="cuda")
    b1[5], b1[41] = float("inf"), float("nan")
    if op == "pw_dw":
        desc = fcm.make_desc(1, h, h, ci, cm, cm, 3, 1, 1, "bf16", "nhwc", (act, "none"))
        run = lambda plan: fcm.pw_dw(x, w1, wd, b1, None, act=(act, "none"), layout="nhwc", plan=plan)  # noqa: E731
    else:
        desc = fcm.make_desc(1, h, h, ci, cm, co, 3, 1, 1, "bf16", "nhwc", (act, "none", "none"))
        run = lambda plan: fcm.pw_dw_pw(x, w1, wd, w2, b1, None, None, act=(act, "none", "none"),  # noqa: E731
                                        layout="nhwc", plan=plan)
    plans = fcm.plan_candidates(op, desc, max_count=400)
    names = [fcm.variant_name(p.variant) for p in plans]
    new = next(p for p, s in zip(plans, names) if s.startswith("k_ir8"))
    old = next(p for p, s in zip(plans, names) if not s.startswith("k_ir8"))
    a, b = run(new).float().cpu().numpy(), run(old).float().cpu().numpy()
    assert (np.isnan(a) == np.isnan(b)).all() and (np.isinf(a) == np.isinf(b)).all()
    fin = np.isfinite(b)
    assert np.abs(a[fin] - b[fin]).max(initial=0) <= 2e-2 * max(1.0, np.abs(b[fin]).max(initial=0))
