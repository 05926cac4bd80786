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


# n, m, p, P, NT, client tiles that the next stage adds up in a round (16: at
# most 1024 facilities), rounds
@pytest.mark.parametrize("n,m,p,P,NT,tiles,rounds", [
    # walks of a chunk or two, or as many workgroups as CUs in a round
    (900, 900, 90, 64, 64, 16, 1), (400, 400, 20, 256, 256, 16, 1),
    (1500, 1500, 75, 256, 256, 64, 1), (5000, 5000, 10, 256, 256, 64, 1),
    (1000, 1000, 5, 1024, 256, 16, 1),
    # long walks of small populations
    (8000, 8000, 8, 64, 64, 64, 4), (5000, 5000, 10, 64, 64, 64, 3),
    (5000, 5000, 100, 64, 64, 64, 2), (8000, 1000, 3, 64, 64, 16, 8),
    (1000, 1000, 5, 64, 64, 16, 2), (5000, 500, 3, 128, 128, 16, 4),
])
def test_population_tiles_by_rounds(evals, n, m, p, P, NT, tiles, rounds):
    # (of client tiles after their clients are rounded up to whole waves)
    w = evals(n, m, p, P, NT)[0]
    assert -(-w // (P // 64) // tiles) == rounds, w


# n, m, p, P, NT, runs, client tiles of each: one round where the runs fill the
# chip, as many as alone where one run is all there is
@pytest.mark.parametrize("n,m,p,P,NT,runs,tiles", [
    (1000, 1000, 4, 256, 64, 16, 16), (8000, 8000, 8, 64, 64, 1, 250),
    (8000, 1000, 3, 64, 64, 1, 250),
])
def test_batch_tiles_by_rounds(tmp_path, n, m, p, P, NT, runs, tiles):
    out = hip_stub.run(tmp_path, f"""
stub.stub_quiet(1)
b = batch([ga(instance({n}, {m}, {p}), {P}, {NT}) for _ in range({runs})])
stub.stub_quiet(0)
clear()
ok(pmp.pmp_batch_step(b, 1, None))
print(*[r[2] for r in log("launch") if "k_batch_eval" in r[1]])
""")
    want = runs * (P // 64) * tiles
    assert all(want <= int(x) < want + 8 for x in out.split()), out


# n, p, P, runs: few client tiles of many chromosome tiles
@pytest.mark.parametrize("n,p,P,runs", [
    (100, 10, 16384, 1), (100, 10, 4096, 2), (200, 20, 8192, 3), (64, 5, 8192, 4),
    (100, 10, 64, 1), (500, 50, 1024, 2),
])
def test_batch_uses_every_xcd(tmp_path, n, p, P, runs):
    """The launch is eight lists of workgroups, one per XCD, padded to the
    longest: with equal runs they are of about one length."""
    out = hip_stub.run(tmp_path, f"""
stub.stub_quiet(1)
b = batch([ga(instance({n}, {n}, {p}), {P}) for _ in range({runs})])
stub.stub_quiet(0)
clear()
ok(pmp.pmp_batch_step(b, 1, None))
print(*[r[2] for r in log("launch") if "k_batch_eval" in r[1]])
""", {"PMP_BATCH_CLIENTS": str(n)})
    # (one client tile a run)
    tiles = runs * (P // 64)
    assert all(tiles <= int(x) <= 1.125 * tiles + 8 for x in out.split()), (out, tiles)


@pytest.mark.parametrize("waves", ["4", "8", "16"])
def test_batch_tiles_fit_the_partial_sums(tmp_path, waves):
    """Whatever the batch's rule says when the batch is made (a count set
    meanwhile, here): no more client tiles than the run has room for."""
    hip_stub.run(tmp_path, """
x = instance(900, 900, 90)
clear()
g = ga(x, 256)
room = max(int(r[1]) for r in log("malloc"))  # two sets of 12 bytes a cell
os.environ["PMP_CLIENTS_PER_BLOCK"] = "4"
b = batch([g])
clear()
ok(pmp.pmp_batch_step(b, 1, None))
for r in log("launch"):
    if "k_batch_eval" in r[1]:
        assert (int(r[2]) - 7) * 64 * 24 <= room, (r, room)
""", {"PMP_EVAL_WAVES": waves})
