"""When device memory kept from destroyed handles goes back to the driver (on a
stand-in for the HIP runtime)."""
import pytest

import hip_stub


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    folder = tmp_path_factory.mktemp("stub")
    return lambda code, env=None: hip_stub.run(folder, code, env)


def test_trim(run):
    run("""
d = buf(4 * 60 * 90)
live = instance(50, 90, 5, d=d)
a, b = instance(60, 90, 5, d=d), instance(40, 90, 5, d=d)
g = ga(live, 64)
clear()
for x in (a, b):
    pmp.pmp_instance_destroy(x)
pmp.pmp_ga_destroy(g)
assert not log("free")
ok(pmp.pmp_device_cache_trim())
frees = {r[1] for r in log("free")}
assert len(frees) >= 4
ok(pmp.pmp_device_cache_trim())
assert len(log("free")) == len(frees)
clear()
pmp.pmp_instance_destroy(instance(60, 90, 5, d=d))   # nothing was kept
assert log("malloc")
ok(pmp.pmp_eval_population(live, buf(16 * 70), 70, buf(8 * 70), None, ON_DEVICE, None))
""")


def test_idle_blocks_go_at_the_next_allocation(run):
    run("""
d = buf(4 * 60 * 90)
pmp.pmp_instance_destroy(instance(60, 90, 5, d=d))
clear()
time.sleep(10.3)
x = instance(10, 9, 2, d=d)            # (of another size)
assert len(log("free")) == 1, log()
""")


def test_nothing_is_kept_at_a_limit_of_zero(run):
    run("""
d = buf(4 * 60 * 90)
x = instance(60, 90, 5, d=d)
clear()
pmp.pmp_instance_destroy(x)
assert len(log("free")) == 1
""", {"PMP_DEVICE_CACHE_MB": "0"})


def test_the_oldest_go_past_the_limit(run):
    run("""
d = buf(4 * 300 * 300)                 # tables of 10 * 300 * 320 bytes
x = [instance(300 - k, 300, 5, d=d) for k in range(3)]
clear()
pmp.pmp_instance_destroy(x[0])
assert not log("free")
pmp.pmp_instance_destroy(x[1])
first = log("free")
assert len(first) == 1
pmp.pmp_instance_destroy(x[2])
assert len(log("free")) == 2
assert len({r[1] for r in log("free")}) == 2
""", {"PMP_DEVICE_CACHE_MB": "1"})


def test_out_of_memory_gives_everything_back(run):
    run("""
d = buf(4 * 300 * 300)
for n in (300, 200):
    pmp.pmp_instance_destroy(instance(n, 300, 5, d=d))
big = buf(4 * 3000 * 300)
clear()
stub.stub_fail_malloc(5000000)
out = vp()
assert pmp.pmp_preprocess(big, 300, 3000, 300, 5, ON_DEVICE, None, C.byref(out)) == 2
kinds = [r[0] for r in log("nomem", "free")]
assert kinds == ["nomem"] + ["free"] * (len(kinds) - 2) + ["nomem"] and len(kinds) >= 3, kinds
stub.stub_fail_malloc(-1)
ok(pmp.pmp_preprocess(big, 300, 3000, 300, 5, ON_DEVICE, None, C.byref(out)))
""")


def test_binding():
    import paper_1610_10061_amd as pm
    pm.pmp_device_cache_trim()


def test_many_blocks(run):
    """Taking and keeping a block costs about the same however many are kept."""
    run("""
stub.stub_quiet(1)
d = buf(4 * 40 * 40)


def again(count):  # us per instance, made of kept blocks and destroyed
    for rep in range(2):
        t = time.perf_counter()
        for x in [instance(8 + k % 32, 40, 5, d=d) for k in range(count)]:
            pmp.pmp_instance_destroy(x)
    return (time.perf_counter() - t) / count


few, many = again(1000), again(20000)
assert many < 5 * few, (few, many)
""")
