"""The checkpoint distance of rollout: what is no distance is refused before
anything is computed (a negative one gave a wrong gradient, one that int() takes
to zero an endless loop)."""
import pytest

torch = pytest.importorskip("torch")
autograd = pytest.importorskip("paper_1411_6121_amd.autograd")


@pytest.mark.parametrize("segment", [-1, -3, 0.5, -0.5])
def test_refused(segment):
    cfg = dict(lattice=9, dtype="f64", n=(4, 4, 1), L=(4.0, 4.0, 1.0), rho0=1.0, RT=1 / 3, tau=0.4, dt=0.2, bc=(0,) * 6)
    force = torch.zeros(2, 1, 4, 4, dtype=torch.float64, requires_grad=True)
    with pytest.raises(ValueError, match="segment"):
        autograd.rollout(cfg, force, torch.zeros_like(force), 5, segment)
