"""The static sums' launch asks for its LDS when the counts (dynamic) and the
columns' parts (8 KB, static) together pass 64 KB (on a stand-in for the HIP
runtime)."""
import pytest

import hip_stub


@pytest.mark.parametrize("m,asked", [(28672, False), (28673, True), (30001, True),
                                     (32768, True), (32769, True), (65535, True)])
def test_large_lds_is_asked_for(tmp_path_factory, m, asked):
    hip_stub.run(tmp_path_factory.getbasetemp(), f"""
x = instance(3, {m}, 5)
rows = [r for r in log("attr", "launch") if "k_static" in r[1]]
(launch,) = [r for r in rows if r[0] == "launch"]
lds = int(launch[5])
assert lds == 4 * (({m} + 1) // 2)
assert ([int(r[2]) for r in rows if r[0] == "attr"] == [lds]) == {asked}, rows
assert (lds + 8192 > 65536) == {asked}
""")
