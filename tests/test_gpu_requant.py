"""int8 requantisation over the whole int32 accumulator range, bit-exact against integer
arithmetic. With zero weights the accumulator of an output channel is its int32 bias, so a
layer's biases put any accumulator through its epilogue: values on and beside the rounding
ties, the clamp's ends and the ends of int32, for every kind of multiplier and shift."""
import numpy as np
import pytest

from paper_2404_19331_amd import fcm

pytestmark = pytest.mark.gpu

SCALES = [(1, 0), (1, 8), (3, 1), (19001, 22), (16777217, 31), (2147483647, 31), (2147483647, 62), (-40503, 20),
          (-2147483648, 40), (0, 5)]


def _expected(acc, mult, shift, qmin, qmax, zp, act):
    t = int(acc) * int(mult)
    if shift:
        q, r = t >> shift, t & ((1 << shift) - 1)
        half = 1 << (shift - 1)
        q += 1 if (r > half or (r == half and q & 1)) else 0
    else:
        q = t
    q = max(qmin, min(qmax, q + zp))
    return max(q, zp) if act != "none" else q


def _accumulators(mult, shift, count):
    """Ends of int32, values around ties of acc * mult / 2^shift, and random ones."""
    vals = [0, 1, -1, 2, -2, 2**31 - 1, -2**31, 2**24, 2**24 + 1, -2**24 - 1]
    for k in range(-130, 131):  # acc just below, at and above (k + 1/2) * 2^shift / mult
        if mult:
            at = ((2 * k + 1) << shift) // (2 * mult)
            vals += [at - 1, at, at + 1]
    rng = np.random.default_rng(7)
    vals += [int(v) for v in rng.integers(-2**31, 2**31, count)] + [int(v) for v in rng.integers(-2**15, 2**15, count)]
    vals = [v for v in vals if -2**31 <= v < 2**31]
    return np.array(vals[:count], dtype=np.int32)


@pytest.mark.parametrize("layout", ["nhwc", "nchw"])  # persistent and first-generation kernels
@pytest.mark.parametrize("op", ["pw", "dw", "pw_pw"])
@pytest.mark.parametrize("zp,act", [(0, "none"), (-128, "relu"), (3, "none"), (127, "relu6")])
def test_requant_whole_range(op, layout, zp, act):
    import torch

    c, ci = 1024, 16
    for mult, shift in SCALES:
        qmin, qmax = -127, 127
        rq = (mult, shift, qmin, qmax, zp)
        b = _accumulators(mult, shift, 240 if op == "pw_pw" else c)
        co = len(b) // 4 * 4
        b = b[:co]
        bias = torch.from_numpy(b).cuda()
        if op == "dw":
            b = b[: co // 16 * 16]
            co, bias = len(b), bias[: co // 16 * 16].contiguous()
            x = torch.zeros((1, co, 3, 3) if layout == "nchw" else (1, 3, 3, co), dtype=torch.int8, device="cuda")
            y = fcm.dw(x, torch.zeros(co, 3, 3, dtype=torch.int8, device="cuda"), bias, act=act, rq=rq, layout=layout)
        else:
            x = torch.zeros((1, ci, 2, 3) if layout == "nchw" else (1, 2, 3, ci), dtype=torch.int8, device="cuda")
            w = torch.zeros(co, ci, dtype=torch.int8, device="cuda")
            if op == "pw":
                y = fcm.pw(x, w, bias, act=act, rq=rq, layout=layout)
            else:  # the second convolution of a pair; the first gives zeros
                w1 = torch.zeros(64, ci, dtype=torch.int8, device="cuda")
                w2 = torch.zeros(co, 64, dtype=torch.int8, device="cuda")
                y = fcm.pw_pw(x, w1, w2, None, bias, act=("none", act), rq=[(1, 0, -127, 127), rq], layout=layout)
        y = y.cpu().numpy()
        y = np.moveaxis(y, 1, -1) if layout == "nchw" else y
        want = np.array([_expected(v, mult, shift, qmin, qmax, zp, act) for v in b], dtype=np.int8)
        assert (y == want).all(), (mult, shift)
