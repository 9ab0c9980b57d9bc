"""A vector's H psi and a state's Sigma do not depend on how many vectors share
the launch: in complex FP64, where the order of a projector's partial sums
shows in the last bits, on a cluster whose projectors reach many tiles."""
import numpy as np
import pytest
import torch

from conftest import make_ctx
from paper_2601_21005_amd import sgw, systems

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cluster():
    species, pos = systems.si_cluster(5, seed=3)
    return systems.cluster_model(species, pos, n=24, h=0.6, ecut=28.0)


@pytest.mark.parametrize("prec", [sgw.SGW_C128, sgw.SGW_C64])
@pytest.mark.parametrize("nvec", [1, 2, 9, 16, 17, 32, 33, 65])
def test_hpsi_is_the_same_in_every_batch(cluster, prec, nvec):
    """One call on nvec vectors against the same vectors in chunks of 8
    (max_nvec) and in the chunks of sgw_apply_H_noalloc (here one)."""
    wide = make_ctx(cluster, prec, max_nvec=nvec)
    few = make_ctx(cluster, prec, max_nvec=8)
    g = torch.Generator(device="cpu").manual_seed(nvec)
    x = torch.randn((nvec, wide.N), generator=g, dtype=torch.complex128).to(wide.cdtype).cuda()
    y = [torch.zeros_like(x) for _ in range(3)]
    wide.apply_H(x, y[0])
    few.apply_H(x, y[1])
    few.apply_H_noalloc(x, y[2])
    torch.cuda.synchronize()
    wide.close()
    few.close()
    assert torch.isfinite(torch.view_as_real(y[0])).all()
    assert torch.equal(y[0], y[1]) and torch.equal(y[0], y[2])


def test_first_state_is_bitwise_the_single_state_call(cluster):
    """sgw_sigma_estimate_states with two states (24 orbitals a launch) against
    the single-state call (16), complex FP64."""
    s = cluster
    ctx = make_ctx(s, sgw.SGW_C128, max_nvec=16)
    lo, hi = ctx.bounds()
    rs = np.random.default_rng(4)
    phis = rs.standard_normal((2, ctx.N))
    phis /= np.sqrt(np.sum(phis * phis, axis=1, keepdims=True) * s.grid.h ** 3)
    kw = dict(seed=9, n_zeta=2, n_eta=4, n_tau=3, dt=0.1, m_sub=2, mu=-1.0, beta=4.0, ncoef=60,
              emin=lo, emax=hi, n_xi=64, f_g=0.05, batch=2)
    sig, x, _ = ctx.sigma_estimate_states(phis, **kw)
    s1, x1, _ = ctx.sigma_estimate(phis[0], **kw)
    ctx.close()
    assert np.all(np.isfinite(sig))
    assert np.array_equal(sig[0], s1) and np.array_equal(x[0], x1)
