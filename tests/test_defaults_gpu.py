"""The forms that the library picks by itself, each named and checked against
the oracle at the sizes where it can go wrong: the column forms' tiles, the
accumulating rows, the mass operator's three forms, scattering with one moment,
infinities and NaN beside padded tiles, and arrays at the 32-bit limit."""
import math

import numpy as np
import pytest
import torch

from helpers import TOL_F64, componentwise_err, contraction_inputs, dev, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1904_08555_amd as P
    P.sj_init(0)
    return P


@pytest.fixture(scope="module")
def orc():
    import oracle
    oracle.lib()
    return oracle


def contraction(P, orc, k, layout, Z, G, D, NM, accumulate, spec):
    """Runs the specialization into a guarded buffer and compares it with the oracle."""
    L, Lp, psi, phi = contraction_inputs(53, layout, Z, G, D, NM)
    if k == P.SJ_LTIMES:
        W, x, n = L, psi, NM
        ref, scale = orc.ltimes(layout, Z, G, D, NM, L, psi), orc.ltimes_absscale(layout, Z, G, D, NM, L, psi)
    else:
        W, x, n = Lp, phi, D
        ref, scale = orc.lplustimes(layout, Z, G, D, NM, Lp, phi), orc.ltimes_absscale(layout, Z, G, NM, D, Lp, phi)
    old = np.random.default_rng(n).uniform(-1, 1, n * G * Z) if accumulate else np.full(n * G * Z, np.nan)
    out = dev(np.concatenate([old, np.full(64, 7.0)]))
    P.sj_run(P.sj_specialize(k, **spec), [dev(W), dev(x), out])
    got = host(out)
    assert (got[-64:] == 7.0).all()
    if accumulate:
        ref, scale = ref + old, scale + np.abs(old)
    assert componentwise_err(got[:-64], ref, scale) <= TOL_F64


# weights straight from memory, by one wave and split over waves; staged weights with 512 threads, at the most
# moments and outputs too; two columns a lane; columns numbered through all records
@pytest.mark.parametrize("layout,Z,G,D,NM,wdirect,split,flat,tile,block", [
    ("DGZ", 100, 1, 128, 64, 1, (4, 4), 0, 1, 64), ("DGZ", 16384, 1, 128, 64, 1, (2, 2), 0, 2, 64),
    ("GDZ", 5000, 3, 40, 16, 1, (1, 2), 1, 2, 64), ("DGZ", 16386, 1, 128, 64, 0, (1, 1), 0, 1, 512),
    ("GDZ", 8336, 2, 120, 49, 0, (1, 1), 0, 1, 512), ("ZDG", 1200, 22, 128, 64, 0, (1, 1), 1, 1, 512),
    ("DZG", 33001, 1, 96, 64, 0, (1, 1), 0, 1, 512), ("DGZ", 131104, 1, 65, 64, 0, (1, 1), 0, 2, 256),
    ("ZDG", 22001, 6, 9, 4, 0, (1, 1), 1, 2, 256)])
@pytest.mark.parametrize("accumulate", [False, True])
def test_column_forms(P, orc, layout, Z, G, D, NM, wdirect, split, flat, tile, block, accumulate):
    for i, k in enumerate((P.SJ_LTIMES, P.SJ_LPLUSTIMES)):
        spec = dict(layout=layout, Z=Z, G=G, D=D, NM=NM, flags=P.SJ_FLAG_ACCUMULATE if accumulate else 0)
        src = P.sj_emit_source(k, **spec)
        info = P.sj_handle_info(P.sj_specialize(k, **spec))
        assert info["kernel_name"].endswith("_cols_mfma_" + layout.lower()) and info["scratch_bytes"] == 0
        assert (info["tile_n"], info["block"]) == (tile, block)
        for name, value in (("WDIRECT", wdirect), ("OS", split[i]), ("FLAT", flat)):
            assert "#define SJ_%s %d\n" % (name, value) in src, (k, name)
        contraction(P, orc, k, layout, Z, G, D, NM, accumulate, spec)


# more tiles than 2048 workgroups hold at once: one tile a wave, and full rounds with a ragged last tile
@pytest.mark.parametrize("layout,Z,G,D,NM", [("ZDG", 53001, 5, 17, 4), ("ZDG", 140003, 2, 8, 3), ("DGZ", 270016, 1, 33, 64), ("ZDG", 135001, 2, 72, 33)])
@pytest.mark.parametrize("accumulate", [False, True])
def test_column_rounds(P, orc, layout, Z, G, D, NM, accumulate):
    for k in (P.SJ_LTIMES, P.SJ_LPLUSTIMES):
        spec = dict(layout=layout, Z=Z, G=G, D=D, NM=NM, variant=P.SJ_VAR_MFMA, flags=P.SJ_FLAG_ACCUMULATE if accumulate else 0)
        contraction(P, orc, k, layout, Z, G, D, NM, accumulate, spec)


# accumulating rows: two tiles a wave, one, and operands read by the lanes; rows that end inside a group
@pytest.mark.parametrize("Z,D,NM,tile,order", [(20003, 113, 25, 1, 2), (70001, 125, 16, 1, 2), (70001, 112, 25, 2, 2), (8203, 256, 36, 1, 1),
                                               (8195, 127, 64, 1, 2), (8200, 273, 16, 1, 1)])
def test_accumulating_rows(P, orc, Z, D, NM, tile, order):
    spec = dict(layout="ZGD", Z=Z, G=1, D=D, NM=NM, flags=P.SJ_FLAG_ACCUMULATE)
    r = P.sj_resolve(P.SJ_LPLUSTIMES, **spec)
    assert (r["tile_n"], r["order"]) == (tile, order)
    contraction(P, orc, P.SJ_LPLUSTIMES, "ZGD", Z, 1, D, NM, True, spec)
    contraction(P, orc, P.SJ_LTIMES, "ZGD", Z, 1, D, NM, True, spec)


# the three forms of the mass operator, by name; the staged form at the workgroup form's tile too
@pytest.mark.parametrize("form,tile", [("hex", {}), ("hex", dict(order=1, tile_n=1, block=128)), ("staged", dict(order=1)),
                                       ("staged", dict(order=1, tile_n=1, block=128, tile_k=1)), ("staged", dict(tile_n=1))])
@pytest.mark.parametrize("D1D,Q1D", [(8, 12), (3, 9)])
def test_mass_forms(P, orc, form, tile, D1D, Q1D):
    NE = 37
    rng = np.random.default_rng(D1D)
    B1 = rng.uniform(-1, 1, Q1D * D1D)
    Dq, X = rng.uniform(0, 1, NE * Q1D ** 3), rng.uniform(-1, 1, NE * D1D ** 3)
    Y = dev(np.concatenate([np.full(X.size, np.nan), np.full(64, 7.0)]))
    h = P.sj_specialize(P.SJ_MASS, D=D1D, NM=Q1D, inputs=3, count=NE, **tile)
    name = P.sj_handle_info(h)["kernel_name"]
    assert ("sj_mass_pa_hex_" in name) == (form == "hex")
    P.sj_run(h, [dev(B1), dev(Dq), dev(X), Y])
    got = host(Y)
    assert (got[-64:] == 7.0).all()
    assert componentwise_err(got[:-64], orc.mass(3, D1D, Q1D, B1, Dq, X), orc.mass(3, D1D, Q1D, B1, Dq, X, absolute=True)) <= TOL_F64


# one moment: nestings that hold the same arrays give the same values, whichever form each takes
@pytest.mark.parametrize("Z,G", [(1001, 17), (3000, 24), (777, 55), (201, 5), (200001, 33)])
def test_scattering_one_moment(P, orc, Z, G):
    rng = np.random.default_rng(Z)
    nmat = 3
    S = rng.uniform(-1, 1, (nmat, 1, G, G))
    mat = rng.integers(0, nmat, Z).astype(np.int32)
    for same in (("DGZ", "GDZ", "GZD"), ("DZG", "ZDG", "ZGD")):
        phi = rng.uniform(-1, 1, G * Z)
        ref = orc.scattering(same[0], Z, G, 1, S, mat, phi)
        scale = orc.scattering(same[0], Z, G, 1, np.abs(S), mat, np.abs(phi))
        for layout in same:
            out = dev(np.concatenate([np.full(G * Z, np.nan), np.full(64, 7.0)]))
            P.sj_run(P.sj_specialize(P.SJ_SCATTERING, layout=layout, Z=Z, G=G, NM=1, count=nmat), [dev(S.ravel()), dev(mat), dev(phi), out])
            got = host(out)
            assert (got[-64:] == 7.0).all()
            assert componentwise_err(got[:-64], ref, scale) <= TOL_F64, layout


# an infinity or NaN in one column, or in the last of the inputs beside a tile's padding, reaches that
# column's outputs and no others, where the oracle has it too
@pytest.mark.parametrize("layout,Z,G,D,NM", [("DGZ", 37, 1, 13, 5), ("ZDG", 3, 7, 21, 17), ("DGZ", 16400, 1, 50, 19), ("ZGD", 19, 1, 13, 5),
                                             ("GZD", 8209, 1, 13, 5), ("ZGD", 33, 2, 45, 18)])
def test_contractions_beside_padding(P, orc, layout, Z, G, D, NM):
    L, Lp, psi, phi = contraction_inputs(59, layout, Z, G, D, NM)
    for n, x in ((D, psi), (NM, phi)):
        size = dict(D=n, G=G, Z=Z)
        v = x.reshape([size[a] for a in layout]).transpose([layout.index(a) for a in "DGZ"])
        v[n - 1, G - 1, Z - 1] = np.inf
        v[0, 0, Z // 2] = np.nan
        v[n // 2, G // 2, 0] = -np.inf
    for k, W, x, m, ref in ((P.SJ_LTIMES, L, psi, NM, orc.ltimes(layout, Z, G, D, NM, L, psi)),
                            (P.SJ_LPLUSTIMES, Lp, phi, D, orc.lplustimes(layout, Z, G, D, NM, Lp, phi))):
        out = dev(np.full(m * G * Z, 7.0))
        P.sj_run(P.sj_specialize(k, layout=layout, Z=Z, G=G, D=D, NM=NM), [dev(W), dev(x), out])
        np.testing.assert_array_equal(host(out)[~np.isfinite(ref)], ref[~np.isfinite(ref)])
        assert np.isfinite(host(out)[np.isfinite(ref)]).all() and (~np.isfinite(ref)).any()
    phi_ref = orc.ltimes(layout, Z, G, D, NM, L, psi)
    want = orc.lplustimes(layout, Z, G, D, NM, Lp, phi_ref)
    out, mom = dev(np.full(D * G * Z, 7.0)), dev(np.full(NM * G * Z, 7.0))
    P.sj_run(P.sj_specialize(P.SJ_LTIMES_LPLUS, layout=layout, Z=Z, G=G, D=D, NM=NM), [dev(L), dev(Lp), dev(psi), out, mom])
    for got, ref in ((host(mom), phi_ref), (host(out), want)):
        assert (np.isfinite(got) == np.isfinite(ref)).all()


@pytest.mark.parametrize("layout,Z,G,NM", [("DZG", 70, 37, 4), ("DGZ", 70, 19, 3), ("ZGD", 70, 9, 5), ("GZD", 40, 35, 4)])
def test_scattering_beside_padding(P, orc, layout, Z, G, NM):
    import sj_inputs as gen
    rng = np.random.default_rng(Z + G)
    nmat, nl = 3, math.isqrt(NM - 1) + 1
    S = rng.uniform(0.5, 1, (nmat, nl, G, G))
    logical = rng.uniform(0, 1, (NM, G, Z))
    logical[NM - 1, G - 1, Z - 1] = np.inf
    logical[0, 0, Z // 2] = np.nan
    phi, mat = gen.to_layout(logical, layout).ravel(), rng.integers(0, nmat, Z).astype(np.int32)
    spec = dict(layout=layout, Z=Z, G=G, NM=NM, count=nmat)
    assert P.sj_resolve(P.SJ_SCATTERING, **spec)["tile_k"] > 0          # sorted by material
    out = dev(np.full(phi.size, 7.0))
    P.sj_run(P.sj_specialize(P.SJ_SCATTERING, **spec), [dev(S.ravel()), dev(mat), dev(phi), out])
    ref = orc.scattering(layout, Z, G, NM, S, mat, phi)
    np.testing.assert_array_equal(host(out)[~np.isfinite(ref)], ref[~np.isfinite(ref)])
    assert np.isfinite(host(out)[np.isfinite(ref)]).all() and (~np.isfinite(ref)).any()


def test_mass_beside_padding(P, orc):
    D1D, Q1D, NE = 5, 8, 9                                               # a ragged last group of elements
    rng = np.random.default_rng(1)
    B1 = rng.uniform(0.5, 1, Q1D * D1D)
    Dq, X = rng.uniform(0.5, 1, NE * Q1D ** 3), rng.uniform(0.5, 1, NE * D1D ** 3)
    X[3 * D1D ** 3 + 7], Dq[-1] = np.nan, np.inf
    Y = dev(np.full(X.size, 7.0))
    h = P.sj_specialize(P.SJ_MASS, D=D1D, NM=Q1D, inputs=3, count=NE)
    assert "_hex_" in P.sj_handle_info(h)["kernel_name"]
    P.sj_run(h, [dev(B1), dev(Dq), dev(X), Y])
    got = host(Y).reshape(NE, -1)
    assert np.isnan(got[3]).all() and (got[NE - 1] == np.inf).all()
    rest = [e for e in range(NE - 1) if e != 3]
    assert np.isfinite(got[rest]).all()


# one value a column or row: the output is the input times one weight, exactly; the largest index is just
# below 2^31, where a tile reaches past it
@pytest.mark.parametrize("layout,Z,G", [("ZDG", 536870911, 4), ("ZGD", 2147483647, 1)])
def test_arrays_at_the_index_limit(P, layout, Z, G):
    n = Z * G
    x = torch.empty(n, dtype=torch.float64, device="cuda")
    for i in range(0, n, 1 << 28):
        x[i:i + (1 << 28)] = torch.arange(i, min(n, i + (1 << 28)), dtype=torch.float64, device="cuda")
    W = torch.full((2,), 0.5, dtype=torch.float64, device="cuda")[:1]
    y = torch.full((n,), -1.0, dtype=torch.float64, device="cuda")
    P.sj_run(P.sj_specialize(P.SJ_LTIMES, layout=layout, Z=Z, G=G, D=1, NM=1), [W, x, y])
    for i in range(0, n, 1 << 28):
        assert torch.equal(y[i:i + (1 << 28)], 0.5 * x[i:i + (1 << 28)]), i
    del x, y
    torch.cuda.empty_cache()
