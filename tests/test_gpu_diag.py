"""The diagnostics at the edges of their tiles, groups and launch rules,
against the oracle. A pair term carries a few 1e-15 (one Newton step on the
hardware reciprocal square root) and an FP64 sum over n particles of like
sign a few roundings more: 1e-13 relative. The momenta, angular momenta and
the centre of mass cancel, so they are bound by 1e-14 of the sum of their
terms' magnitudes."""

import numpy as np
import pytest

import oracle
import paper_2411_18889_amd as nb
from tests.gpu_util import DEV, host, to_dev  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,n", [("f64", 1), ("f64", 2), ("f64", 16), ("f64", 17), ("f64", 255),
                                    ("f64", 257), ("f32", 511), ("f64", 512), ("f64", 513),
                                    ("mix_tilec", 528), ("f64", 529), ("f32", 1025),
                                    ("mix_tilec", 5003), ("f64", 24575), ("mix_tilec", 24576),
                                    ("f64", 39999), ("f32", 40000), ("f64", 41013)])
def test_edges(prec, n):
    rng = np.random.default_rng(n)
    x, v = rng.normal(size=(3, n)), rng.normal(size=(3, n))
    m = rng.uniform(0.5, 1.5, size=n) / n
    eps = 2.0 ** -6
    xd, vd, md = to_dev(x, v, m, prec)
    d = nb.diag_dict(nb.diag(xd, vd, md, eps, prec=prec))
    x, v, m = host(xd), host(vd), host(md)
    o = oracle.diag(x, v, m, eps)
    for k in ("KE", "M"):
        assert abs(d[k] - o[k]) <= 1e-13 * abs(o[k]), k
    scale = abs(o["KE"]) + abs(o["PE"])
    for k in ("PE", "E"):
        assert abs(d[k] - o[k]) <= 1e-13 * scale, k
    r, s = np.linalg.norm(x, axis=0), np.linalg.norm(v, axis=0)
    for k in ("Px", "Py", "Pz"):
        assert abs(d[k] - o[k]) <= 1e-14 * float((m * s).sum()), k
    for k in ("Lx", "Ly", "Lz"):
        assert abs(d[k] - o[k]) <= 1e-14 * float((m * r * s).sum()), k
    for k in ("COMx", "COMy", "COMz"):
        assert abs(d[k] - o[k]) <= 1e-14 * float((m * r).sum() / m.sum()), k
