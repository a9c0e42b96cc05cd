"""fl_apply_D_noalloc captured into a graph, as its callers do that cannot
allocate: one kernel for separate fields, the fixed scratch array where the
result goes over the input.  Several replays on new inputs, with eager work
between them, each against the eager result."""
import pytest

import synth_inputs as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,nrhs", [((4, 4, 4, 6), 2), ((8, 8, 8, 16), 6)])
@pytest.mark.parametrize("over_input", [False, True])
def test_captured_operator_replays(dims, nrhs, over_input):
    import torch
    import paper_1108_2473_amd as F
    lat = F.Lattice(dims, -1)
    lat.set_gauge(S.random_links(dims, 0.5, 95))
    lat.set_kappa(0.12)
    inputs = [torch.from_numpy(S.random_spinors(dims, nrhs, 96 + k)).cuda() for k in range(4)]
    want = [lat.apply_D(x) for x in inputs]
    x = inputs[0].clone()
    y = x if over_input else torch.empty_like(x)
    lat.apply_D_noalloc(x, y)  # before the capture: links packed, code loaded
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        lat.apply_D_noalloc(x, y)
    for k in (0, 1, 2, 3, 1):
        x.copy_(inputs[k])
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want[k])
        assert torch.equal(lat.apply_D(inputs[k]), want[k])
    del g
    lat.close()
