"""Kernel structures at the sizes where their tiling can go wrong (edges of
tiles, remainders, the smallest and largest of a range), against the oracle."""
import numpy as np
import pytest
import torch

from helpers import TOL_F64, componentwise_err, dev, host

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


# rows around the 16- and 32-row tiles and the one-workgroup limit; units and inputs around the
# 16-wide blocks; the widest network; one wave and sixteen
@pytest.mark.parametrize("F,H,R,block", [(16, 16, 15, 0), (15, 17, 16, 0), (17, 15, 17, 0), (33, 48, 32, 0), (8, 64, 33, 0),
                                         (37, 64, 53, 0), (64, 31, 257, 64), (1, 126, 97, 0), (48, 100, 65, 1024),
                                         (24, 64, 20000, 0)])
def test_mlp_tiles(P, orc, F, H, R, block):
    rng = np.random.default_rng(F + H + R)
    n = orc.mlp_nparams(F, H)
    theta = (rng.standard_normal(n) * (1.0 / np.sqrt(H))).astype(np.float32)
    X = rng.standard_normal((R, F)).astype(np.float32)
    t = rng.standard_normal(R).astype(np.float32)
    spec = dict(dtype=P.SJ_F32, rows=R, inputs=F, width=H, block=block)
    th_d, X_d, t_d = dev(theta), dev(X), dev(t)
    y_d = torch.full((R,), float("nan"), dtype=torch.float32, device="cuda")
    P.sj_run(P.sj_specialize(P.SJ_MLP_FWD, **spec), [th_d, X_d, y_d])
    y_ref = orc.mlp_forward(F, H, theta.astype(np.float64), X.astype(np.float64))
    # FP32: three sums of at most 127 terms of magnitude about 1, gamma_130 = 8e-6 against the outputs' size
    assert np.abs(host(y_d) - y_ref).max() <= 1e-5 * max(1.0, np.abs(y_ref).max())
    g_d = torch.full((n,), float("nan"), dtype=torch.float32, device="cuda")
    loss_d = torch.full((1,), float("nan"), dtype=torch.float32, device="cuda")
    # the workspace's end is guarded: partial gradients have to stay inside it
    ws = torch.full((R * (4 * H + 2) + 64,), 7.0, dtype=torch.float32, device="cuda")
    hb = P.sj_specialize(P.SJ_MLP_BWD, **spec)
    P.sj_run(hb, [th_d, X_d, t_d, g_d, loss_d, ws])
    loss_ref, g_ref = orc.mlp_loss_grad(F, H, theta.astype(np.float64), X.astype(np.float64), t.astype(np.float64))
    g = host(g_d).astype(np.float64)
    assert (host(ws)[-64:] == 7.0).all()
    assert abs(float(host(loss_d)[0]) - loss_ref) <= 1e-5 * max(1.0, loss_ref)
    assert np.linalg.norm(g - g_ref) <= 1e-4 * np.linalg.norm(g_ref)   # the bound of the backward pass' other test
    g2, l2 = torch.empty_like(g_d), torch.empty_like(loss_d)
    P.sj_run(hb, [th_d, X_d, t_d, g2, l2, torch.empty_like(ws)])
    assert torch.equal(g2, g_d) and torch.equal(l2, loss_d)            # a fixed order of summation


# one and several elements a workgroup, a ragged last group, more elements than resident workgroups
# hold at once (a second round with prefetched loads), each thread count of the default tile
@pytest.mark.parametrize("D1D,Q1D,NE", [(3, 4, 13), (3, 4, 41003), (1, 7, 700), (5, 8, 4101), (4, 5, 5), (7, 7, 6001), (8, 12, 5),
                                        (2, 14, 4100), (9, 15, 3), (12, 12, 2), (12, 5, 7), (16, 16, 2), (20, 4, 3)])
def test_mass_hex_groups(P, orc, D1D, Q1D, NE):
    rng = np.random.default_rng(D1D * Q1D + NE)
    B1 = rng.uniform(-1, 1, Q1D * D1D)
    Dq, X = rng.uniform(0, 1, NE * Q1D ** 3), rng.uniform(-1, 1, NE * D1D ** 3)
    Y = torch.full((X.size,), float("nan"), dtype=torch.float64, device="cuda")
    h = P.sj_specialize(P.SJ_MASS, D=D1D, NM=Q1D, inputs=3, count=NE)
    P.sj_run(h, [dev(B1), dev(Dq), dev(X), Y])
    r = P.sj_resolve(P.SJ_MASS, D=D1D, NM=Q1D, inputs=3, count=NE)
    assert r["order"] == 1
    assert P.sj_specialize(P.SJ_MASS, D=D1D, NM=Q1D, inputs=3, count=NE, order=1, tile_n=r["tile_n"], block=r["block"]) == h
    # the oracle's direct sum is long: the first and last 300 elements
    es = np.unique(np.r_[0:min(300, NE), max(0, NE - 300):NE])
    Ds, Xs = Dq.reshape(NE, -1)[es].ravel(), X.reshape(NE, -1)[es].ravel()
    got = host(Y).reshape(NE, -1)
    assert np.isfinite(got).all()
    assert componentwise_err(got[es].ravel(), orc.mass(3, D1D, Q1D, B1, Ds, Xs),
                             orc.mass(3, D1D, Q1D, B1, Ds, Xs, absolute=True)) <= TOL_F64


# the column structures AUTO picks: one partial tile; output blocks shared by two to five waves and a ragged
# last block; two columns a lane with records shorter than a tile; records crossing tiles with odd lengths; the
# sizes on both sides of the weights-from-memory line (16,384 columns) and of each structure's line; a tile whose
# registers send it back to the staged weights
@pytest.mark.parametrize("layout,Z,G,D,NM,tile", [
    ("DGZ", 11, 1, 40, 7, {}), ("DZG", 5, 3, 84, 64, {}), ("DGZ", 70, 2, 33, 49, {}), ("ZDG", 31, 6, 130, 16, {}),
    ("ZDG", 1800, 6, 24, 16, {}), ("GDZ", 41, 7, 57, 25, {}), ("ZDG", 23, 41, 20, 36, {}), ("DGZ", 4096, 4, 48, 16, {}),
    ("DGZ", 4097, 4, 48, 16, {}), ("ZDG", 8300, 2, 27, 9, {}), ("ZDG", 5500, 3, 16, 4, {}), ("DZG", 13107, 5, 20, 16, {}),
    ("DZG", 13108, 5, 20, 16, {}), ("DGZ", 65538, 2, 16, 64, {}), ("DGZ", 300, 4, 64, 64, dict(variant=3, unroll=16, block=512)),
    ("ZDG", 50, 12, 20, 17, dict(variant=3, tile_n=4, unroll=3, order=2))])
@pytest.mark.parametrize("accumulate", [False, True])
def test_columns(P, orc, layout, Z, G, D, NM, tile, accumulate):
    from helpers import contraction_inputs
    L, Lp, psi, phi = contraction_inputs(31, layout, Z, G, D, NM)
    fl = P.SJ_FLAG_ACCUMULATE if accumulate else 0
    spec = dict(layout=layout, Z=Z, G=G, D=D, NM=NM, flags=fl, **tile)
    for k, W, x, n, ref, scale in ((P.SJ_LTIMES, L, psi, NM, orc.ltimes(layout, Z, G, D, NM, L, psi),
                                    orc.ltimes_absscale(layout, Z, G, D, NM, L, psi)),
                                   (P.SJ_LPLUSTIMES, Lp, phi, D, orc.lplustimes(layout, Z, G, D, NM, Lp, phi),
                                    orc.ltimes_absscale(layout, Z, G, NM, D, Lp, phi))):
        old = np.random.default_rng(n).uniform(-1, 1, n * G * Z) if accumulate else np.full(n * G * Z, np.nan)
        buf = np.concatenate([old, np.full(64, 7.0)])           # the end of the output is guarded
        out = dev(buf)
        h = P.sj_specialize(k, **spec)
        P.sj_run(h, [dev(W), dev(x), out])
        got = host(out)
        assert (got[-64:] == 7.0).all()
        if accumulate:
            ref, scale = ref + old, scale + np.abs(old)
        assert componentwise_err(got[:-64], ref, scale) <= TOL_F64


# zones sorted by material: one zone, a full block and its neighbours, a material for every zone;
# the group counts around 16-wide blocks; cut-off degrees, odd and even runs of moments; the larger
# blocks of lines (nm not innermost)
@pytest.mark.parametrize("layout,Z,G,NM,nmat", [
    ("DGZ", 1, 17, 1, 1), ("GDZ", 63, 32, 5, 3), ("DGZ", 129, 28, 9, 200), ("GDZ", 8201, 31, 17, 5), ("DZG", 8200, 33, 17, 5),
    ("DZG", 64, 33, 4, 1), ("ZDG", 65, 48, 10, 70), ("DGZ", 130, 49, 3, 4), ("ZDG", 77, 64, 16, 2), ("GDZ", 1, 64, 2, 3),
    ("ZGD", 1, 8, 2, 1), ("GZD", 65, 9, 3, 3), ("ZGD", 1030, 16, 7, 4), ("GZD", 100, 32, 9, 150), ("ZGD", 4100, 32, 16, 4),
    ("GZD", 20, 24, 25, 6), ("ZGD", 33, 33, 50, 5), ("GZD", 33, 55, 4, 7), ("ZGD", 17, 64, 64, 2), ("GZD", 9, 32, 64, 9)])
def test_scattering_sorted(P, orc, layout, Z, G, NM, nmat):
    import math
    import sj_inputs as gen
    rng = np.random.default_rng(Z + G)
    nl = math.isqrt(NM - 1) + 1
    S = rng.uniform(-1, 1, (nmat, nl, G, G))
    phi = gen.to_layout(rng.uniform(-1, 1, (NM, G, Z)), layout).ravel()
    spec = dict(layout=layout, Z=Z, G=G, NM=NM, count=nmat)
    r = P.sj_resolve(P.SJ_SCATTERING, **spec)
    assert r["tile_k"] > 0
    h = P.sj_specialize(P.SJ_SCATTERING, **spec)
    assert P.sj_specialize(P.SJ_SCATTERING, **spec, variant=P.SJ_VAR_DIRECT, tile_k=r["tile_k"]) == h
    for bad in (dict(tile_k=r["tile_k"] + 1), dict(tile_k=r["tile_k"], block=64), dict(tile_k=r["tile_k"], tile_n=1)):
        with pytest.raises(P.SJError):
            P.sj_specialize(P.SJ_SCATTERING, **spec, variant=P.SJ_VAR_DIRECT, **bad)
    for mat in (rng.integers(0, nmat, Z), np.arange(Z) % nmat, np.arange(Z) * nmat // Z, np.full(Z, nmat - 1)):
        mat = mat.astype(np.int32)
        ref = orc.scattering(layout, Z, G, NM, S, mat, phi)
        scale = orc.scattering(layout, Z, G, NM, np.abs(S), mat, np.abs(phi))
        out = dev(np.concatenate([np.full(NM * G * Z, np.nan), np.full(64, 7.0)]))   # the end is guarded
        P.sj_run(h, [dev(S.ravel()), dev(mat), dev(phi), out])
        got = host(out)
        assert (got[-64:] == 7.0).all()
        assert componentwise_err(got[:-64], ref, scale) <= TOL_F64
    mat[rng.integers(0, Z)] = -1
    mat[0] = nmat                                           # no such material: NaN, and only there
    P.sj_run(h, [dev(S.ravel()), dev(mat), dev(phi), out])
    after = host(out)[:-64]
    bad = gen.to_layout(np.broadcast_to((mat < 0) | (mat >= nmat), (NM, G, Z)).copy(), layout).ravel()
    assert np.isnan(after[bad]).all() and (after[~bad] == got[:-64][~bad]).all()


# fused contractions on the matrix cores: one column, one and two columns per lane, columns that end
# inside a tile or cross rows, directions fewer than the waves' steps, around 16-wide blocks and beyond
# the loads in flight, the most moments
@pytest.mark.parametrize("layout,Z,G,D,NM", [
    ("DGZ", 2, 1, 1, 1), ("GDZ", 17, 3, 5, 4), ("ZDG", 5, 3, 17, 15), ("DZG", 33, 2, 15, 17), ("ZDG", 400, 22, 31, 16),
    ("DGZ", 4099, 2, 33, 33), ("GDZ", 8193, 1, 130, 9), ("DZG", 1200, 11, 129, 25), ("DGZ", 100, 1, 64, 128), ("GDZ", 4098, 3, 65, 113),
    ("ZDG", 2049, 4, 144, 48)])
def test_fused_columns(P, orc, layout, Z, G, D, NM):
    from helpers import contraction_inputs
    L, Lp, psi, _ = contraction_inputs(47, layout, Z, G, D, NM)
    spec = dict(layout=layout, Z=Z, G=G, D=D, NM=NM)
    r = P.sj_resolve(P.SJ_LTIMES_LPLUS, **spec)
    assert r["tile_k"] == 16 * r["tile_n"] > 0
    h = P.sj_specialize(P.SJ_LTIMES_LPLUS, **spec)
    assert P.sj_specialize(P.SJ_LTIMES_LPLUS, **spec, variant=P.SJ_VAR_DIRECT, tile_n=r["tile_n"], tile_k=r["tile_k"],
                           block=r["block"], order=r["order"]) == h
    ref_phi = orc.ltimes(layout, Z, G, D, NM, L, psi)
    s_phi = orc.ltimes_absscale(layout, Z, G, D, NM, L, psi)
    ref = orc.lplustimes(layout, Z, G, D, NM, Lp, ref_phi)
    scale = orc.ltimes_absscale(layout, Z, G, NM, D, Lp, s_phi)
    for want_phi in (True, False):
        out = dev(np.concatenate([np.full(D * G * Z, np.nan), np.full(64, 7.0)]))     # the ends are guarded
        phi = dev(np.concatenate([np.full(NM * G * Z, np.nan), np.full(64, 7.0)]))
        P.sj_run(h, [dev(L), dev(Lp), dev(psi), out] + ([phi] if want_phi else []))
        got, gphi = host(out), host(phi)
        assert (got[-64:] == 7.0).all() and (gphi[-64:] == 7.0).all()
        assert componentwise_err(got[:-64], ref, scale) <= TOL_F64
        assert np.isnan(gphi[:-64]).all() if not want_phi else componentwise_err(gphi[:-64], ref_phi, s_phi) <= TOL_F64


# few rows as columns: one row, a tile and its neighbours, ragged outputs and reductions, the last
# row count of the rule
@pytest.mark.parametrize("layout,Z,G,D,NM", [
    ("ZGD", 1, 1, 1, 1), ("GZD", 15, 1, 5, 17), ("ZGD", 17, 3, 33, 16), ("GZD", 16, 4, 96, 25), ("ZDG", 130, 1, 113, 36),
    ("ZGD", 33, 31, 120, 64), ("GZD", 64, 64, 48, 49), ("ZGD", 8192, 1, 31, 9)])
@pytest.mark.parametrize("accumulate", [False, True])
def test_few_rows(P, orc, layout, Z, G, D, NM, accumulate):
    for k in (P.SJ_LTIMES, P.SJ_LPLUSTIMES):
        spec = dict(layout=layout, Z=Z, G=G, D=D, NM=NM)
        h = P.sj_specialize(k, **spec)
        assert "cols_mfma" in P.sj_handle_info(h)["kernel_name"]
        r = P.sj_resolve(k, **spec)
        assert P.sj_specialize(k, **{f: r[f] for f in ("layout", "Z", "G", "D", "NM", "variant", "tile_n", "tile_k", "unroll",
                                                       "block", "order", "flags")}) == h
    test_columns(P, orc, layout, Z, G, D, NM, {}, accumulate)


# odd row lengths as flat runs: pairs that straddle rows, one value past the last pair, rows that end
# inside a group, outputs wider than the reduction's blocks
@pytest.mark.parametrize("layout,Z,G,D,NM", [
    ("ZGD", 9999, 1, 1, 1), ("GZD", 2733, 3, 5, 3), ("ZGD", 4097, 2, 33, 16), ("GZD", 8200, 1, 17, 31), ("ZGD", 8209, 1, 113, 9),
    ("GZD", 21847, 3, 4, 3), ("ZGD", 65537, 1, 16, 25), ("ZDG", 65552, 1, 8, 1)])
@pytest.mark.parametrize("accumulate", [False, True])
def test_odd_rows(P, orc, layout, Z, G, D, NM, accumulate):
    for k in (P.SJ_LTIMES, P.SJ_LPLUSTIMES):
        spec = dict(layout=layout, Z=Z, G=G, D=D, NM=NM)
        h = P.sj_specialize(k, **spec)
        assert "rows_mfma_lds" in P.sj_handle_info(h)["kernel_name"]
        r = P.sj_resolve(k, **spec)
        assert P.sj_specialize(k, **{f: r[f] for f in ("layout", "Z", "G", "D", "NM", "variant", "tile_n", "tile_k", "unroll",
                                                       "block", "order", "flags")}) == h
    test_columns(P, orc, layout, Z, G, D, NM, {}, accumulate)
