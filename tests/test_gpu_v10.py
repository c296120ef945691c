"""GPU parity of the DW -> PW kernels for few pixels (k_few10), forced through explicit plans:
every variant against the CPU oracle, over pixel counts that leave partial blocks and cross
rows and images, input channels that leave a partial chunk, one to several chunks per wave
and more chunks than the weights held in registers, partial output tiles and several
output-channel blocks, both strides and padding other than one. A planned bf16 chain puts
them in the place of the deep kernels: their outputs agree bit for bit."""
import pytest
import torch

from paper_2404_19331_amd import fcm
from paper_2404_19331_amd.workloads import Case, make_inputs

from gpu_util import assert_close, dev_inputs, oracle_ref, run_fused, to_np

pytestmark = pytest.mark.gpu

ACTS = [("relu6", "none", "none"), ("none", "relu", "none"), ("relu", "relu6", "none")]
SHAPES = [(1, 7, 7, 960, 160, 1, 1), (1, 1, 1, 8, 8, 1, 1), (3, 5, 3, 40, 24, 1, 1), (2, 13, 11, 144, 136, 2, 1),
          (1, 4, 4, 256, 264, 1, 0), (5, 3, 2, 520, 72, 2, 2), (2, 9, 16, 32, 64, 1, 1), (1, 6, 5, 1032, 48, 1, 1)]
CASES = [Case("dw_pw", n, h, w, ci, ci, co, 3, s, pad, "bf16", "nhwc", ACTS[i % 3], bias=i % 4 != 2, seed=6100 + i,
              name="v10-%dx%dx%dx%d-%d-s%dp%d" % (n, h, w, ci, co, s, pad))
         for i, (n, h, w, ci, co, s, pad) in enumerate(SHAPES)]


def _plans(desc, prefix):
    out = []
    for v in range(fcm.lib().fcm_variant_count()):
        name = fcm.variant_name(v)
        if not name.startswith(prefix):
            continue
        pbk, ct = (int(f) for f in name.split("<")[1].split(",")[:2])
        try:
            out.append(fcm.plan_evaluate("dw_pw", desc, 1, 16 * pbk, 32, 16 * ct, v))
        except fcm.FcmError:
            pass
    return out


@pytest.mark.parametrize("case", CASES, ids=lambda c: c.name)
def test_every_variant(case):
    inp = make_inputs(case)
    ref = oracle_ref(case, inp)
    d = dev_inputs(inp, case.dtype)
    plans = _plans(fcm.desc_from_case(case), "k_dwpw10<")
    assert len(plans) == 7
    for p in plans:
        print(case.name, fcm.variant_name(p.variant), flush=True)
        assert_close(to_np(run_fused(case, d, plan=p)), ref, case.dtype, case.name + " " + fcm.variant_name(p.variant))


@pytest.mark.parametrize("case", [c for c in CASES if c.c_in % 32 == 0], ids=lambda c: c.name)
def test_same_bits_as_the_deep_kernels(case):
    d = dev_inputs(make_inputs(case), case.dtype)
    desc = fcm.desc_from_case(case)
    few = [run_fused(case, d, plan=p) for p in _plans(desc, "k_dwpw10<")]
    seen = set()
    for p in fcm.plan_candidates("dw_pw", desc, 60):
        if not fcm.variant_name(p.variant).startswith("k_dwpw7<"):
            continue
        seen.add(p.variant)
        other = run_fused(case, d, plan=p)
        for y in few:
            assert torch.equal(y.view(torch.int16), other.view(torch.int16)), fcm.variant_name(p.variant)
    assert seen
