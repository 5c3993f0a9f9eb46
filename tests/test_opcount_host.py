"""tgks_flop_counts: pins of the counts that depend on how the parameters reach
the counted sequences, and of the selections (exact weights, nothing else)."""
import pytest


def counts(**kw):
    from paper_2309_10534_amd import tgks
    D = kw.pop("D", 2)
    return tgks.tgks_flop_counts(tgks.tgks_params_default(D, [64] * D, [0.1] * D, **kw))


def test_weno_ao_counts():
    """The same for every choice of the linear weights, and with each of the
    products by the three ratios of the linear weights counted: where the
    ratios reach the sequence as one value (zero), two of the three products
    merge in every reconstruction (199 operations instead of 201)."""
    for kw in ({}, dict(d_hi=0.7, d_lo=0.9), dict(eps_w=1e-6)):
        f = counts(scheme="weno_ao", **kw)
        assert (f["normal"], f["face"], f["face_stage2"]) == (201.0, 5105.0, 4997.0), (kw, f)


@pytest.mark.parametrize("mu", [0.0, 1e-3])
def test_characteristic_counts(mu):
    """The characteristic kernel's face: the basis, projections, exact
    selections, power-series values and face-frame fluxes; the shared
    differences of the certain decisions (17 per field) are no part of it."""
    f = counts(recon=1, mu=mu, prandtl=0.7)
    ref = (7160.0, 7144.0) if mu == 0.0 else (7727.0, 7711.0)
    assert (f["face"], f["face_stage2"]) == ref, f
