"""GPU parity of the NCHW DW -> PW kernels (k_dwpw9), forced through explicit plans: every
compiled variant that implements a case over tiles that leave ragged pixel blocks, windows
and borders and one, two or four groups of waves, against the CPU oracle. Cases cover every
element type, both strides and filters, channel counts that leave partial chunks and weight
rows of 16 bytes, words and single elements, partial output tiles and several output blocks,
and padding other than half the filter."""
import pytest

from paper_2404_19331_amd import fcm
from paper_2404_19331_amd.workloads import Case, make_inputs

from gpu_util import assert_close, dev_inputs, oracle_ref, run_fused, to_np

pytestmark = pytest.mark.gpu

ELT = {"f32": 4, "bf16": 2, "i8": 1}
RQ = ((20011, 22, -128, 127), (1342177283, 38, -127, 127), (1, 7, -127, 127))


def _cases():
    out = []
    for dt in ELT:
        for ci, co, k, s, pad in [(64, 64, 3, 1, 1), (182, 91, 3, 2, 1), (37, 130, 5, 1, 2), (130, 5, 3, 1, 0),
                                  (18, 33, 5, 2, 4), (400, 24, 3, 2, 2)]:
            out.append(Case("dw_pw", 2, 13, 11, ci, ci, co, k, s, pad, dt, "nchw",
                            [("relu6", "none", "none"), ("none", "relu", "none")][len(out) % 2], RQ,
                            dist_x="i8small" if dt == "i8" else "n01", dist_w="i8small", bias=True,
                            seed=5200 + len(out), name="v9-%s-%d-%d-k%ds%dp%d" % (dt, ci, co, k, s, pad)))
    return out


CASES = _cases()


@pytest.mark.parametrize("case", CASES, ids=lambda c: c.name)
def test_every_variant_tile_and_group(case):
    inp = make_inputs(case)
    ref = oracle_ref(case, inp)
    d = dev_inputs(inp, case.dtype)
    desc = fcm.desc_from_case(case)
    plans = []
    for v in range(fcm.lib().fcm_variant_count()):
        name = fcm.variant_name(v)
        if not name.startswith("k_dwpw9<%s,%d,%d," % (case.dtype, case.k, case.stride)):
            continue
        ct = int(name.split(",")[3])
        for th, tw in ((7, 7), (8, 8), (3, 5), (1, 11), (4, 4), (2, 11), (13, 2), (8, 16), (6, 7), (4, 9), (2, 4)):
            try:
                plans.append(fcm.plan_evaluate("dw_pw", desc, th, tw, 64 // ELT[case.dtype], 16 * ct, v))
            except fcm.FcmError:
                pass
    # (int8 holds at most 128 window positions: no stride-2 tile here fits)
    assert plans or (case.dtype == "i8" and case.stride == 2)
    for p in plans:
        print(case.name, fcm.variant_name(p.variant), p.tile_h, p.tile_w, p.splits, flush=True)
        got = to_np(run_fused(case, d, plan=p))
        assert_close(got, ref, case.dtype, "%s %s %dx%d groups %d" % (
            case.name, fcm.variant_name(p.variant), p.tile_h, p.tile_w, p.splits))


def test_planner_takes_them_for_nchw():
    for case in CASES:
        if case.dtype == "bf16":  # (fp32 also has the whole-module kernels for small batches)
            assert fcm.variant_name(fcm.plan("dw_pw", fcm.desc_from_case(case)).variant).startswith("k_dwpw9<")
