"""The binding's memo of descriptors: calls that differ in any value get descriptors of their
own with those values, equal calls share one, per-channel descriptors (which hold tensors) are
never kept, and the memo stays bounded."""
from paper_2404_19331_amd import fcm

BASE = dict(n=1, h=9, w=8, ci=16, cm=16, co=32, k=3, stride=1, pad=1, dt="i8", layout="nhwc", act=("relu", "none"),
            rq=[(3, 5, -127, 127), (1, 4, -128, 127, 2)], rq_channel=None, zp_in=0)
OTHER = dict(n=2, h=10, w=7, ci=32, cm=32, co=16, k=5, stride=2, pad=2, dt="bf16", layout="nchw",
             act=["none", "relu6"], rq=[(3, 6, -127, 127), (1, 4, -128, 127, 2)], zp_in=-3)


def test_every_value_is_part_of_the_key():
    a = fcm._desc(**BASE)
    assert fcm._desc(**BASE) is a
    assert fcm._desc(**dict(BASE, act=list(BASE["act"]), rq=tuple(BASE["rq"]))) is a
    for name, value in OTHER.items():
        args = dict(BASE, **{name: value})
        d = fcm._desc(**args)
        assert d is not a, name
        full = {**args, "dtype": args["dt"]}
        want = fcm.make_desc(*[full[f] for f in ("n", "h", "w", "ci", "cm", "co", "k", "stride", "pad", "dtype",
                                                 "layout", "act", "rq")], zp_in=full["zp_in"])
        assert bytes(d) == bytes(want), name


def test_the_memo_is_bounded():
    for n in range(1, 3 * fcm._DESCS_MOST // 2):
        fcm._desc(**dict(BASE, n=n))
        assert len(fcm._DESCS) <= fcm._DESCS_MOST
