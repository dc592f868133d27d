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
