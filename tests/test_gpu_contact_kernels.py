"""Which contact gradient kernel runs: two wavefronts per four systems for few
systems, one for many (what the comparison of the two kernels takes for
given)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2109_07719_amd import synth
from test_gpu_tiling_default import events

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,kernel", [(5, "k_contact_adj_pair"), (8000, "k_contact_adj")])
def test_gradient_kernel_by_batch(B, kernel):
    from torch.profiler import ProfilerActivity, profile

    from paper_2109_07719_amd.contact import ContactBatch
    T = 3
    d = synth.landing_quadruped(1, T)
    cb = ContactBatch([d[0]] * B, d[4], [d[5]] * B, [d[6]] * B, mu=0.7, beta=0.2, niter=10, dtype=torch.float32)
    f = lambda x: torch.tensor(np.ascontiguousarray(np.repeat(np.asarray(x)[..., None], B, -1)), dtype=torch.float32,
                               device="cuda")
    qT, qdT, tr = cb.rollout(f(d[1]), f(d[2]), f(d[3]), 1e-3)[:3]
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as prof:
        cb.grad(tr, f(d[3]), 1e-3, torch.ones_like(qT), torch.ones_like(qdT))
        torch.cuda.synchronize()
    names = [e["name"].split("<")[0] for e in events(prof) if "k_contact_adj" in e["name"]]
    print("case", B, names, flush=True)
    assert len(names) == 1 and names[0].endswith(kernel)
