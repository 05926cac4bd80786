"""A waiting evaluation whose reduction cannot be launched leaves its error bits
on the device; the next waiting call must not report them (on a stand-in for
the HIP runtime: it clears the word before its evaluation)."""
import pytest

import hip_stub

CALLS = {
    "eval": "pmp.pmp_eval_population(x, m, 70, f, None, ON_DEVICE, None)",
    "per client": "pmp.pmp_eval_population(x, m, 70, f, None, ON_DEVICE | 8, None)",
    "no allocation": "pmp.pmp_eval_population_noalloc(x, m, 70, f, None, ON_DEVICE, None)",
    "hbp": "pmp.pmp_hbp_eval(h, m, 70, f, None, ON_DEVICE, None)",
}


@pytest.mark.parametrize("name", CALLS)
def test_bits_of_a_failed_call_are_not_reported_by_the_next(tmp_path_factory, name):
    hip_stub.run(tmp_path_factory.getbasetemp(), f"""
pmp.pmp_hbp_eval.argtypes = [vp, vp, i32, vp, vp, C.c_uint32, vp]
x, h, m, f = instance(60, 90, 5), vp(), buf(8 * 70 * 2), buf(8 * 70)
ok(pmp.pmp_hbp_reduce(x, None, C.byref(h)))


def kernels(call):
    clear()
    ok(call())
    return [next(k for k in ("k_zero", "k_reduce", "eval") if k in r[1]) for r in log("launch")]


def call():
    return {CALLS[name]}


plain = ["eval", "k_reduce"]
assert kernels(call) == plain
stub.stub_fail_launch(b"k_reduce")
assert call() != 0
assert kernels(call) == ["k_zero"] + plain
assert kernels(call) == plain
""")
