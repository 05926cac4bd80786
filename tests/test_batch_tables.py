"""A batch whose autotune call fails for want of memory keeps the tables it
had, and steps with them (on a stand-in for the HIP runtime)."""
import hip_stub


def test_failed_autotune_keeps_the_tables(tmp_path):
    # 16 runs with long walks fill the chip with 16 client tiles each; common
    # counts give them more tiles, whose launch table is larger
    hip_stub.run(tmp_path, """
x = instance(1000, 1000, 4)


def evals():
    return [r[2] for r in log("launch") if "k_batch_eval" in r[1]]


def stepped():
    b = batch([ga(x, 256) for _ in range(16)])
    clear()
    ok(pmp.pmp_batch_step(b, 1, None))
    return b, evals()


b, first = stepped()
clear()
stub.stub_fail_malloc(0)
assert pmp.pmp_batch_autotune(b, None, None) != 0
stub.stub_fail_malloc(-1)
assert log("nomem") and not log("free"), log()
clear()
ok(pmp.pmp_batch_step(b, 1, None))
assert evals() == first, (evals(), first)
""")
