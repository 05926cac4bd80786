"""Device memory of destroyed objects, on a stand-in for the HIP runtime: a
block is kept only when the library has waited for everything it enqueued for
the object, which needs no wait for the device (not allowed while any stream
is being captured); otherwise it goes to hipFree as without a cache."""
import pytest

import hip_stub


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    folder = tmp_path_factory.mktemp("stub")
    return lambda code, env=None: hip_stub.run(folder, code, env)


def test_destroy_beside_a_capture(run):
    run("""
d, cap = buf(4 * 60 * 90), new_stream()
a, b = instance(60, 90, 5, d=d), instance(60, 90, 5, ON_DEVICE | ASYNC, d=d)
g = ga(instance(60, 90, 5, d=d), 64)
ok(pmp.pmp_ga_step(g, 8, None))
assert stub.hipStreamBeginCapture(cap, 0) == 0
clear()
pmp.pmp_instance_destroy(a)      # waited for: kept
pmp.pmp_instance_destroy(b)      # its tables may still be being made
pmp.pmp_ga_destroy(g)            # its generations may still be running
assert not log("devsync"), log()
assert len(log("free")) >= 2
graph = vp()
assert stub.hipStreamEndCapture(cap, C.byref(graph)) == 0
""")


USES = {
    # name: (what is done with instance x on streams s, t; whether it is kept)
    "waiting": ("ok(pmp.pmp_eval_population(x, m, 70, f, None, ON_DEVICE, s))", True),
    "left": ("ok(pmp.pmp_eval_population(x, m, 70, f, None, ON_DEVICE | ASYNC, s))", False),
    "left, then waited": (
        "ok(pmp.pmp_eval_population(x, m, 70, f, None, ON_DEVICE | ASYNC, s))\n"
        "ok(pmp.pmp_instance_check(x, s))", True),
    "left, another stream waited": (
        "ok(pmp.pmp_eval_population(x, m, 70, f, None, ON_DEVICE | ASYNC, s))\n"
        "ok(pmp.pmp_instance_check(x, t))", False),
    "left on two streams": (
        "ok(pmp.pmp_eval_population(x, m, 70, f, None, ON_DEVICE | ASYNC, s))\n"
        "ok(pmp.pmp_eval_population(x, m, 70, f, None, ON_DEVICE | ASYNC, t))\n"
        "ok(pmp.pmp_instance_check(x, t))", False),
    "no allocation, left": (
        "ok(pmp.pmp_eval_population_noalloc(x, m, 70, f, None, ON_DEVICE | ASYNC, s))", False),
    "captured": (
        "ok(pmp.pmp_eval_population(x, m, 70, f, None, ON_DEVICE, s))\n"
        "stub.hipStreamBeginCapture(s, 0)\n"
        "ok(pmp.pmp_eval_population_noalloc(x, m, 70, f, None, ON_DEVICE | ASYNC, s))\n"
        "g = vp()\n"
        "assert stub.hipStreamEndCapture(s, C.byref(g)) == 0\n"
        "ok(pmp.pmp_instance_check(x, s))", False),
    "tables copied, left": ("ok(pmp.pmp_instance_tables(x, buf(2 * 60 * 90), None, None, "
                            "ON_DEVICE | ASYNC, s))", False),
    "failed launch": ("stub.stub_fail_launch(b'k_reduce')\n"
                      "assert pmp.pmp_eval_population(x, m, 70, f, None, ON_DEVICE, s) != 0", False),
    "a run's steps": ("g = ga(x, 64); ok(pmp.pmp_ga_step(g, 3, s))", False),
    "a run's steps, read": ("g = ga(x, 64); ok(pmp.pmp_ga_step(g, 11, s))\n"
                            "ok(pmp.pmp_ga_best(g, None, None, None, s))", True),
    "a batch's steps": ("g = ga(x, 64); b = batch([g]); ok(pmp.pmp_batch_step(b, 3, s))\n"
                        "ok(pmp.pmp_batch_check(b, None, s))", False),
    "a batch's steps, read": ("g = ga(x, 64); b = batch([g]); ok(pmp.pmp_batch_step(b, 3, s))\n"
                              "ok(pmp.pmp_ga_best(g, None, None, None, s))", True),
    "the reduced polynomial": ("h = vp(); ok(pmp.pmp_hbp_reduce(x, s, C.byref(h)))", True),
}


@pytest.mark.parametrize("name", USES)
def test_kept_only_when_waited_for(run, name):
    code, kept = USES[name]
    run(f"""
s, t = new_stream(), new_stream()
m, f = buf(8 * 70 * 2), buf(8 * 70)
x = instance(60, 90, 5, stream=s)
{code}
clear()
pmp.pmp_instance_destroy(x)
frees = len(log("free"))
assert not log("devsync")
assert (frees == 0) == {kept}, log()
""")


def test_steps_beside_instances_closed_by_another_thread(run):
    """Every step's first call captures a graph; the instances closed meanwhile
    by the other thread must not spoil it."""
    run("""
d = buf(4 * 60 * 90)
gas = [ga(instance(60, 90, 5, d=d), 64) for _ in range(200)]
stub.stub_quiet(1)
stop, bad = [], []


def close():
    while not stop:
        pmp.pmp_instance_destroy(instance(60, 90, 5, d=d))


th = threading.Thread(target=close)
th.start()
for g in gas:
    bad.append(pmp.pmp_ga_step(g, 8, None))
stop.append(1)
th.join()
assert not any(bad), bad
""")
