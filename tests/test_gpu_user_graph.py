"""Steps of run-time-length grids captured into a graph of the caller's own: without the
library's graphs a call launches its passes directly, so a program may capture it on its
stream.  Every replay is then one whole call: its steps, their records and the scale, bit for
bit as launched, with eager work of the context between the replays."""
import numpy as np
import pytest

from paper_1601_04640_amd import inputs as I
from tests.gpu_util import banner, oparams

pytestmark = pytest.mark.gpu

# one-stage and two-stage finalisations, two and three axes
GRIDS = [("3d", (22, 18, 14)), ("2dxy", (90, 70, 1)), ("3d", (150, 130, 110))]


@pytest.mark.parametrize("imag", [True, False], ids=["imag", "real"])
@pytest.mark.parametrize("per_call", [1, 3])
@pytest.mark.parametrize("geom,n", GRIDS, ids=lambda v: v if isinstance(v, str) else "x".join(map(str, v)))
def test_captured_steps_replay_as_launched(geom, n, per_call, imag, gpu_lib):
    import torch
    from paper_1601_04640_amd.binding import Solver
    banner("steps in the caller's graph", geom, n, per_call, imag)
    w = dict(geom=geom, nx=n[0], ny=n[1], nz=n[2], dx=0.2, dy=0.2, dz=0.2, dt=0.001, gamma=1.0,
             nu=1.2, lam=2.0, g=20.0, gdd=6.0, R=2.0 if geom == "3d" else 0.0)
    p = oparams(w)
    psi0 = I.random_complex(p.shape(), 71, p.dV())
    replays, runs = 4, []
    for captured in (False, True):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            s = Solver(w, prec="fp64", stream=st)
            step = s.step_imag if imag else s.step_real
            s.set_psi(psi0)
            step(2)                    # with the library's graphs: a finalisation may be outstanding
            s.use_graphs(False)
            torch.cuda.synchronize()
            states = []
            if captured:
                graph = torch.cuda.CUDAGraph()
                with torch.cuda.graph(graph, stream=st):
                    step(per_call)
            for _ in range(replays):
                if captured:
                    graph.replay()
                else:
                    step(per_call)
                torch.cuda.synchronize()
                states.append(s.get_psi())
                states.append(s.dipolar_potential())
            hist = s.history(2 + replays * per_call)
            runs.append((states, hist, s.energy()))
            if captured:
                del graph
            s.close()
    assert len(runs[1][1]) == 2 + replays * per_call
    for a, b in zip(runs[0][0], runs[1][0]):
        assert np.array_equal(a, b)
    assert runs[0][1] == runs[1][1]
    assert runs[0][2] == runs[1][2]
