"""Steps captured in a HIP graph and replayed (tlb_step only enqueues).

A call of n >= 2 steps leaves the state where it found it in memory, so its
graph advances the state by n steps at every replay, though the handle's own
time stands still; what is read afterwards is the state's, never something
kept from an earlier read."""
import numpy as np
import pytest
import torch

from paper_2109_12565_amd import Simulation

from test_gpu_parity import posts_case

pytestmark = pytest.mark.gpu


def make(case, precision):
    return Simulation(case["params"], case["rho_a"], case["rho_b"], case["temp"], solid=case["solid"],
                      t_bottom=case["t_bottom"], precision=precision)


def same(a, b, where):
    fa, fb = a.fields(), b.fields()
    for k in fa:
        assert np.array_equal(fa[k], fb[k]), (where, k)
    oa, ob = a.observables(), b.observables()
    assert {k: v for k, v in oa.items() if k != "step"} == {k: v for k, v in ob.items() if k != "step"}, where
    sa, sb = a.stress(), b.stress()
    for k in sa:
        assert np.array_equal(sa[k], sb[k]), (where, k)
    assert np.array_equal(a.populations(), b.populations()), where


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16dev"])
@pytest.mark.parametrize("n", [2, 3, 4, 5, 6, 7])
def test_replayed_steps_are_observed_afresh(precision, n):
    case = posts_case()
    print(precision, n, flush=True)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        a, b = make(case, precision), make(case, precision)
        for s in (a, b):
            s.step(n)
        same(a, b, "eager")
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            a.step(n)
        for k in range(4):
            graph.replay()
            b.step(n)
            same(a, b, ("replay", k))
            if k == 1:
                for s in (a, b):
                    s.set_bottom_temperature(1.3 * case["t_bottom"])
                same(a, b, "new bottom temperature")
        for s in (a, b):
            s.step(3)
        same(a, b, "eager again")
