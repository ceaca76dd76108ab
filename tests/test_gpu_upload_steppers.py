"""bb_factor_upload makes the tables of the fused steppers of large batches,
ragged ones included: the first step of an uploaded factor can be captured in
a graph, which a table allocated inside the capture would end.  Every replay
gives what eager calls give."""
import numpy as np
import pytest
import torch

from paper_2107_05395_amd import inputs
from tests.gpu_util import dev, host, say

pytestmark = pytest.mark.gpu


# one chunk per wave: 64 rows; 32 rows (2^16 to 2^17 lanes of 64-row chunks);
# one chunk; a full decomposition and one of more than 8 chunks beside them
@pytest.mark.parametrize("kind,n,m", [("penta", 500, 8192), ("tri", 200, 20000), ("tri", 200, 32768),
                                      ("penta", 40, 1 << 16), ("penta", 24, 1 << 16),
                                      ("tri", 512, 1 << 15), ("tri", 1000, 4096)])
def test_first_steps_after_upload_are_captured(kind, n, m):
    from paper_2107_05395_amd import Factor
    bands, w = (inputs.cn_diffusion_problem if kind == "tri" else inputs.cn_hyperdiffusion_problem)(n, 0.8)
    make = Factor.tri if kind == "tri" else Factor.penta
    c0 = dev(inputs.uniform_batch(n, m, seed=n))
    outs = [torch.empty_like(c0), None]

    def work(f):
        f.cn_step(c0, w, steps=3, out=outs[0])
        outs[1] = f.adjoint_trajectory(c0, 1)

    other = make(*bands, cyclic=True)      # loads the kernels
    work(other)
    torch.cuda.synchronize()
    eager = [host(o) for o in outs]
    f = make(*bands, cyclic=True)
    f.upload()
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            work(f)
    torch.cuda.current_stream().wait_stream(side)
    for rep in range(3):
        for o in outs:
            o.fill_(float("nan"))
        other.solve(c0, out=torch.empty_like(c0))   # unrelated eager work between replays
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for i, o in enumerate(outs):
            assert np.array_equal(host(o), eager[i]), (rep, i)
    say("captured after upload", kind, n, m, "ok")
