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


@pytest.mark.parametrize("n", (1000, 6001, 12287, 12289, 16384, 24577, 40001))
def test_fp32_adjoint_rounding(n):
    """J^T lam and G^T lam of the FP32 policy within the rounding that its terms
    and sums can leave: with u = 2^-24, the terms' relative errors (a few u:
    rounding of d and s, one ulp of the reciprocal square root, its third power,
    the products) and the running sums of some 128 terms of either sign each
    add about 6 u and 5 u of the root of the sum of the squared term bounds
    2 r^3 (m_i |lam_j| + m_j |lam_i|) and r^3 |d| |lam_j|; three times their
    combination, 24 u, over all sampled particles, and over the first and the
    last eighth, which are nearly all sink side and all source side."""
    x, v, m = plummer_sphere(n, 960 + n % 13)
    m = m * np.random.default_rng(n).uniform(0.5, 1.5, size=n)
    eps, dt, u = 2.0 ** -7, 2.0 ** -9, 2.0 ** -24
    xd, vd, md = to_dev(x, np.zeros_like(x), m, "f32")
    lam = np.random.default_rng(n + 1).normal(size=(3, n))
    rng = np.random.default_rng(n + 2)
    e8 = n // 8
    idx = np.concatenate([np.sort(rng.choice(e8, 100, replace=False)),
                          e8 + np.sort(rng.choice(n - 2 * e8, 100, replace=False)),
                          n - e8 + np.sort(rng.choice(e8, 100, replace=False))])
    mh = host(md)
    acc = nb.accel(xd, md, eps, prec="f32")
    lx = torch.zeros_like(xd)
    lv = torch.tensor(lam, dtype=xd.dtype, device=DEV)
    lm = torch.zeros(n, dtype=torch.float64, device=DEV)
    nb.step_adjoint(xd, vd, md, acc, lx, lv, lm, eps, dt, 0, prec="f32", entry_half=True)
    for walked in (False, True):
        if walked:
            lx.zero_()
            lm.zero_()
            nb.step_adjoint(xd, vd, md, acc, lx, lv, lm, eps, dt, 1, prec="f32")
        xh, lh = host(xd), host(lv)
        jt, gt = oracle.vjp_sampled(xh, mh, lh, eps, idx)
        ej = np.linalg.norm(host(lx)[:, idx] / (0.5 * dt) - jt, axis=0)
        eg = np.abs(host(lm)[idx] / (0.5 * dt) - gt)
        ln = np.linalg.norm(lh, axis=0)
        bj, bg = np.empty(len(idx)), np.empty(len(idx))
        for q, i in enumerate(idx):
            d2 = ((xh - xh[:, i:i + 1]) ** 2).sum(0)
            r3 = (d2 + eps * eps) ** -1.5
            bj[q] = np.sqrt(((2 * r3 * (mh[i] * ln + mh * ln[i])) ** 2).sum())
            bg[q] = np.sqrt((r3 * r3 * d2 * ln * ln).sum())
        for part in (slice(None), slice(0, 100), slice(200, 300)):
            assert np.linalg.norm(ej[part]) <= 24 * u * np.linalg.norm(bj[part]), (walked, part)
            assert np.linalg.norm(eg[part]) <= 24 * u * np.linalg.norm(bg[part]), (walked, part)
