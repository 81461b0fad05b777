"""mot_sinkhorn returns with the plan's stream done, whatever the number of sweeps."""
import numpy as np
import pytest

from paper_2208_03120_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sweeps", [0, 1, 3])
def test_stream_is_done(sweeps):
    import torch
    from paper_2208_03120_amd import mot
    inst = W.make_instance(np.random.Generator(np.random.PCG64(1)), 2, [50, 60], 2, W.TREE, 0.1, parent=[-1, 0])
    a = torch.ones(8192, 8192, dtype=torch.bfloat16, device="cuda")
    out = torch.empty_like(a)
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        plan = mot.Plan(inst.points, inst.weights, W.TREE, inst.parent, 0.1, path=mot.DIRECT)
        torch.mm(a, a, out=out)
        plan.sinkhorn(1)
        for _ in range(40):  # some 40 ms of work ahead of the call
            torch.mm(a, a, out=out)
        _, done, _, _ = plan.sinkhorn(sweeps)
        idle = stream.query()
        plan.close()
    torch.cuda.synchronize()
    assert done == sweeps and idle
