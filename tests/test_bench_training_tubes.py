"""The benchmark's training ensemble (CPU): one tube is left out by its number, any other that fails is an error."""
import numpy as np
import pytest

import bench
from paper_2004_11286_amd import workloads as W


def test_one_marginal_tube_is_left_out_by_number():
    every = W.tube_ensemble(ntubes=4096, ny=1, nz=1, seed=11286)
    tubes, left_out = bench.training_tubes()
    assert left_out == [2110] and len(tubes) == 4095
    p = every[2110][0]
    assert p["nx"] == 251 and list(p["molar_mass"]) == [2.0, 16.0, 40.0]
    for got, want in ((tubes[2109], every[2109]), (tubes[2110], every[2111]), (tubes[-1], every[-1])):
        assert got[0]["nx"] == want[0]["nx"]
        np.testing.assert_array_equal(got[1]["X"], want[1]["X"])


def test_a_failing_tube_stops_the_benchmark(monkeypatch):
    """A tube whose fields become non-finite must not be dropped and trained around."""
    SG = pytest.importorskip("paper_2004_11286_amd.surrogate")

    class Went_on(Exception):
        pass

    calls = []

    def trajectories(tubes, **kw):
        calls.append(len(tubes))
        if len(calls) > 1:
            raise Went_on
        err = ValueError("tubes [7] became non-finite")
        err.tubes = [7]
        raise err

    monkeypatch.setattr(SG, "trajectories", trajectories)
    with pytest.raises(ValueError):
        bench.surrogate_bench()
    assert calls == [4095]
