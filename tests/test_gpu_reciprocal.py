"""The FP64 reciprocal of the planar and base-frame kernels at the ends of the
range: a joint inertia whose reciprocal overflows gives the division's
infinity, not a NaN."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2109_07719_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("inertia,ref", [(1e-310, np.inf), (2.3e-308, 1 / 2.3e-308), (4.0, 0.25), (1.7e308, 1 / 1.7e308)])
def test_reciprocal_ends(inertia, ref):
    from paper_2109_07719_amd.sim import Sim
    s = synth.System(parent=np.array([-1]), jtype=np.array([0]), E_T=np.eye(3)[None], r_T=np.zeros((1, 3)),
                     axis=np.array([[0.0, 0.0, 1.0]]), mass=np.ones(1), com=np.zeros((1, 3)),
                     Ic=np.array([[1.0, 1.0, inertia, 0.0, 0.0, 0.0]]))
    sim = Sim([s], (0.0, 0.0, 0.0), dtype=torch.float64)
    assert sim.info["chain"] and sim.info["frames_identity"]
    z = torch.zeros(1, dtype=torch.float64, device="cuda")
    assert sim.aba(z, z, z + 1.0).item() == ref
