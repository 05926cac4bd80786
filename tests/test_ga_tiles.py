"""Workgroups of a run's evaluation launches (on a stand-in for the HIP runtime
with 256 CUs, two workgroups of 16 waves on each)."""
import pytest

import hip_stub


@pytest.fixture(scope="module")
def evals(tmp_path_factory):
    """n, m, p, P, NT -> workgroups of a generation's evaluations: the
    population's first, the mutants' last."""
    folder = tmp_path_factory.mktemp("stub")

    def f(n, m, p, P, NT):
        out = hip_stub.run(folder, f"""
stub.stub_quiet(1)
g = ga(instance({n}, {m}, {p}), {P}, {NT})
stub.stub_quiet(0)
ok(pmp.pmp_ga_step(g, 1, None))
print(*[r[2] for r in log("launch") if "6k_evalI" in r[1]])
""", {"PMP_GA_MODE": "kernels"})
        return [int(x) for x in out.split()]
    return f


def filled(workgroups, round):
    """Share of the last round's workgroups."""
    return (workgroups % round or round) / round


# n, m, p, P, NT, workgroups of a round.  A client tile is a whole number of
# clients of one size, so a round is not always quite full.
@pytest.mark.parametrize("n,m,p,P,NT,round", [
    (5000, 5000, 10, 256, 256, 256), (5000, 5000, 60, 256, 256, 256),
    (5000, 1000, 20, 512, 256, 512), (5000, 200, 1, 512, 256, 512),
    (5000, 5000, 500, 1024, 256, 512), (3000, 3000, 100, 512, 256, 512),
    (900, 900, 90, 1024, 256, 512), (2000, 2000, 200, 1024, 256, 512),
])
def test_mutants_fill_whole_rounds(evals, n, m, p, P, NT, round):
    w = evals(n, m, p, P, NT)[-1]
    assert filled(w, round) > 0.85, w
