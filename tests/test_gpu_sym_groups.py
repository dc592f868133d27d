"""The symmetric passes with one wave per 64-source group (blocks of 256, and
of 512 in FP64 and FP32): last blocks with empty groups, with one particle in a
group, and whole; one band and many. Sampled rows, the last block's among
them, against the oracle: the library's accuracy targets for the force and
the potential; for the adjoint's J^T lam and G^T lam of a random lam those of
the FP32 pair arithmetic on sums that cancel (1e-4, 1e-12 in FP64)."""

import numpy as np
import pytest
import torch

import oracle
import paper_2411_18889_amd as nb
from nbody_inputs import plummer_sphere
from tests.gpu_util import DEV, TOL, host, rel, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ("mix_tilec", "f32", "f64"))
@pytest.mark.parametrize("n", (12288, 12289, 12288 + 64, 12288 + 129, 24575, 24576 + 1, 30001))
def test_ragged_blocks(prec, n):
    x, v, m = plummer_sphere(n, 950 + n % 17)
    m = m * np.random.default_rng(n).uniform(0.5, 1.5, size=n)
    m[::97] = 0.0  # test particles: they feel the others and weigh nothing
    eps = 2.0 ** -7
    xd, _, md = to_dev(x, v, m, prec)
    xh, mh = host(xd), host(md)
    idx = np.unique(np.concatenate([np.random.default_rng(n).choice(n, 200, replace=False),
                                    np.arange(n - min(n, 70), n)]))
    assert nb.pass_info(1, n, prec)["symmetric"] == 1
    a, p = nb.accel(xd, md, eps, prec=prec, potential=True)
    assert torch.equal(a, nb.accel(xd, md, eps, prec=prec))
    ao, po = oracle.accel_sampled(xh, mh, eps, idx, potential=True)
    assert rel(host(a)[:, idx], ao) <= TOL[prec]
    assert rel(host(p)[idx], po) <= TOL[prec]
    # the entry pass, and a walked-back step from the same state (whose pass
    # also sums the force), in one band and in many
    lam = np.random.default_rng(n + 1).normal(size=(3, n))
    bar = 1e-12 if prec == "f64" else 1e-4
    dt = 2.0 ** -9
    full = nb.workspace_size(2, n, prec)
    for ws in (full, full // 3):
        w = torch.empty(ws, dtype=torch.uint8, device=DEV)
        lx = torch.zeros_like(xd)
        lv = torch.tensor(lam, dtype=xd.dtype, device=DEV)
        lm = torch.zeros(n, dtype=torch.float64, device=DEV)
        acc, vd = a.clone(), torch.zeros_like(xd)
        nb.step_adjoint(xd, vd, md, acc, lx, lv, lm, eps, dt, 0, prec=prec, entry_half=True,
                        workspace=w)
        jt, gt = oracle.vjp_sampled(xh, mh, host(lv), eps, idx)
        assert rel(host(lx)[:, idx], 0.5 * dt * jt) <= bar
        assert rel(host(lm)[idx], 0.5 * dt * gt) <= bar
        xs = xd.clone()
        lx.zero_()
        lm.zero_()
        nb.step_adjoint(xs, vd, md, acc, lx, lv, lm, eps, dt, 1, prec=prec, workspace=w)
        jt, gt = oracle.vjp_sampled(host(xs), mh, host(lv), eps, idx)
        assert rel(host(lx)[:, idx], 0.5 * dt * jt) <= bar
        assert rel(host(lm)[idx], 0.5 * dt * gt) <= bar
        ao = oracle.accel_sampled(host(xs), mh, eps, idx)
        assert rel(host(acc)[:, idx], ao) <= TOL[prec]


@pytest.mark.parametrize("prec", ("mix_tilec", "f32", "f64"))
@pytest.mark.parametrize("n", (12288, 24576))
@pytest.mark.parametrize("heavy", (3, 77, 250))
def test_source_side_chains(prec, n, heavy):
    """A source-side sum is made of chains of at most 128 terms: with one
    particle of mass 1 in the first block and half a rounding unit, 2^-25 (FP64:
    2^-54), in every other, all in one place, each term that follows the heavy
    one in its chain is lost and no other, so that a particle of the last block
    misses at most 127 of them in the potential (eps = 1) and in J^T lam of a
    lam that is 1 there and 0 elsewhere (the sum of the other masses). Joining
    the chains and the slots rounds a few terms more: 136 in all."""
    light = 2.0 ** -54 if prec == "f64" else 2.0 ** -25
    m = np.full(n, light)
    m[heavy] = 1.0
    xd, vd, md = to_dev(np.zeros((3, n)), np.zeros((3, n)), m, prec)
    last = np.arange(n - 256, n)
    whole = np.longdouble(1.0) + np.longdouble(light) * (n - 2)  # of the others

    def lost(sums):
        return float(np.max(np.abs(np.asarray(sums, dtype=np.longdouble) - whole)) / light)

    _, p = nb.accel(xd, md, 1.0, prec=prec, potential=True)
    assert lost(-host(p)[last]) <= 136
    lam = np.zeros((3, n))
    lam[:, last] = 1.0
    acc, lx = torch.zeros_like(xd), torch.zeros_like(xd)
    lv = torch.tensor(lam, dtype=xd.dtype, device=DEV)
    lm = torch.zeros(n, dtype=torch.float64, device=DEV)
    # (the other particles of the last block have the same lam: their terms
    # m_j lam_i - m_i lam_j cancel)
    nb.step_adjoint(xd, vd, md, acc, lx, lv, lm, 1.0, 2.0, 0, prec=prec, entry_half=True)
    whole = np.longdouble(1.0) + np.longdouble(light) * (n - 257)
    assert lost(-host(lx)[:, last]) <= 136
