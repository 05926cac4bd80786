"""An entry point whose stream is being captured asks the driver for device
memory whatever is cached (so that it does not depend on what happens to be
cached whether the call is accepted), on a stand-in for the HIP runtime."""
import pytest

import hip_stub

CALLS = {
    "preprocess": "out = vp(); return pmp.pmp_preprocess(d, 90, 60, 90, 5, ON_DEVICE | ASYNC, s, C.byref(out))",
    "preprocess, waiting": "out = vp(); return pmp.pmp_preprocess(d, 90, 60, 90, 5, ON_DEVICE, s, C.byref(out))",
    "eval": "return pmp.pmp_eval_population(instance(60, 90, 5, d=d), m, 70, f, None, ON_DEVICE, s)",
    "hbp": "h = vp(); r = pmp.pmp_hbp_reduce(x, s, C.byref(h)); pmp.pmp_hbp_destroy(h); return r",
    "enumeration": "return pmp.pmp_exhaustive(y, None, None, None, s)",
    "ga step": "g = gas.pop(); pmp.pmp_ga_step(g, 3, s); pmp.pmp_ga_best(g, None, None, None, s); pmp.pmp_ga_destroy(g)",
    "features": "return pmp.pmp_features(x, hm, 3, C.c_float(0), hf, 0, s)",
}


@pytest.mark.parametrize("name", CALLS)
def test_capture_leaves_the_cache_alone(tmp_path_factory, name):
    hip_stub.run(tmp_path_factory.getbasetemp(), f"""
pmp.pmp_exhaustive.argtypes = [vp] * 5
pmp.pmp_features.argtypes = [vp, vp, i32, C.c_float, vp, C.c_uint32, vp]
d, m, f = buf(4 * 60 * 90), buf(8 * 70 * 2), buf(8 * 70)
hm, hf = (C.c_uint64 * 6)(), (C.c_float * (3 * 90 * 16))()
x, y = instance(60, 90, 5, d=d), instance(10, 9, 2)
gas = [ga(x, 64), ga(x, 64)]


def call(s):
    {CALLS[name]}


s = new_stream()
pmp.pmp_instance_destroy(instance(60, 90, 5, d=d))
call(s)                                   # the cache holds what the call needs
pmp.pmp_instance_destroy(instance(60, 90, 5, d=d))
stub.hipStreamBeginCapture(s, 0)
clear()
call(s)
assert log("malloc"), log()
""")
