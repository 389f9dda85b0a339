"""What the library picks by itself: the default specializations fit the
registers, can be launched, and lie in the tuner's set.  Compiled with
SJ_FLAG_COMPILE_ONLY; nothing is launched."""
import json
import os
import subprocess
import sys

import pytest

import paper_1904_08555_amd as P
from paper_1904_08555_amd import picker, tune

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# hiprtc comes with ROCm and, another version, with torch; the one loaded first serves the process
_SCRATCH = """
import json, sys
if {torch}:
    import torch
from multiprocessing import Pool
import paper_1904_08555_amd as P

def one(spec):
    spec = dict(spec)
    k = getattr(P, spec.pop("kernel"))
    h = P.sj_specialize(k, **dict(spec, flags=spec.get("flags", 0) | P.SJ_FLAG_COMPILE_ONLY))
    return P.sj_handle_info(h)["scratch_bytes"]

if __name__ == "__main__":
    specs = json.load(sys.stdin)
    with Pool(4) as p:
        print(json.dumps([s for s, n in zip(specs, p.map(one, specs, chunksize=1)) if n != 0]))
"""


def spilling(specs, torch):
    """The specs whose kernels use scratch (private memory)."""
    r = subprocess.run([sys.executable, "-c", _SCRATCH.format(torch=torch)], input=json.dumps(specs), cwd=ROOT, text=True,
                       capture_output=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads(r.stdout.splitlines()[-1])


# the three sizes of column tiles (16,384 and 131,072 columns between them)
@pytest.mark.parametrize("torch", [False, True])
def test_columns_without_scratch(torch):
    specs = [dict(kernel="SJ_LPLUSTIMES", layout="DGZ", Z=Z, G=2, D=D, NM=NM, flags=fl)
             for Z in (8000, 40000, 70000) for D in (64, 96, 121, 128) for NM in (36, 49, 64) for fl in (0, 0x40)]
    assert spilling(specs, torch) == []


# accumulating rows, whose lanes also hold old outputs: around the line at which a wave takes one tile, and
# beyond the longest rows of the flat form
@pytest.mark.parametrize("torch", [False, True])
def test_accumulating_rows_without_scratch(torch):
    specs = [dict(kernel="SJ_LPLUSTIMES", layout="ZGD", Z=Z, G=1, D=D, NM=NM, flags=0x40)
             for Z in (40000, 369097) for D, NM in ((112, 25), (112, 36), (113, 25), (117, 25), (125, 25), (127, 64), (128, 64),
                                                    (256, 36), (273, 16), (384, 16))]
    assert spilling(specs, torch) == []


def test_accumulating_rows_on_request():
    """Order 2 asked for stays accepted where it needs scratch, as before."""
    for D, NM, tile in ((256, 36, {}), (384, 16, {}), (128, 16, dict(tile_n=2, block=64)), (384, 16, dict(tile_n=1, block=64))):
        r = P.sj_resolve(P.SJ_LPLUSTIMES, layout="ZGD", Z=40000, G=1, D=D, NM=NM, variant=P.SJ_VAR_MFMA, order=2,
                         flags=P.SJ_FLAG_ACCUMULATE, **tile)
        assert r["order"] == 2


# a launch of 2^32 threads or more is refused by the runtime: the largest scattering that sorts its zones by
# material, one zone more, and 158 GB
@pytest.mark.parametrize("layout", ["DZG", "ZDG", "GZD", "ZGD"])
@pytest.mark.parametrize("Z,G", [(64 * (2 ** 22 - 1), 33), (64 * (2 ** 22 - 1) + 1, 33), (300000000, 33), (64 * (2 ** 23 - 1) + 1, 49)])
def test_scattering_launch_limit(layout, Z, G):
    h = P.sj_specialize(P.SJ_SCATTERING, layout=layout, Z=Z, G=G, NM=1, count=1, flags=P.SJ_FLAG_COMPILE_ONLY)
    info = P.sj_handle_info(h)
    assert 0 < info["grid"] * info["block"] < 2 ** 32


# one moment: DGZ, GDZ and GZD are the same arrays, and so are DZG, ZDG and ZGD, on both sides of the rules' lines
@pytest.mark.parametrize("Z,G", [(196608, 44), (30000, 24), (1000, 33), (5000, 55), (1001, 17), (300001, 24), (300000, 5), (1000000, 15),
                                 (500001, 31), (2000003, 5)])
def test_scattering_one_moment(Z, G):
    for same in (("DGZ", "GDZ", "GZD"), ("DZG", "ZDG", "ZGD")):
        picks = set()
        for layout in same:
            spec = dict(layout=layout, Z=Z, G=G, NM=1, count=3)
            r = P.sj_resolve(P.SJ_SCATTERING, **spec)
            src = P.sj_emit_source(P.SJ_SCATTERING, **spec)
            picks.add((r["variant"], r["tile_k"]) + tuple("#define SJ_NT_%s 1" % w in src for w in ("LOAD", "STORE")))
        assert len(picks) == 1, (same, picks)


def refused(kernel, **spec):
    try:
        P.sj_resolve(kernel, **spec)
    except P.SJError as e:
        return e.status in (P.SJ_ERR_UNSUPPORTED, P.SJ_ERR_INVALID_ARG)
    return False


# flat runs of odd rows: named by tile_k 16 with MFMA where AUTO takes them, and there only
@pytest.mark.parametrize("layout,Z,D,NM,taken", [("ZGD", 40, 63, 45, True), ("ZGD", 40, 12, 45, False), ("GZD", 65535, 16, 9, False),
                                                 ("ZGD", 65536, 16, 9, True), ("GZD", 9000, 17, 31, True)])
def test_odd_runs_on_request(layout, Z, D, NM, taken):
    for k in (P.SJ_LTIMES, P.SJ_LPLUSTIMES):
        spec = dict(layout=layout, Z=Z, G=1, D=D, NM=NM, order=2)
        assert refused(k, **spec) and refused(k, variant=P.SJ_VAR_MFMA, **spec)
        assert refused(k, tile_k=16, **spec)                 # AUTO has no structure for the field to name
        assert refused(k, variant=P.SJ_VAR_MFMA, tile_k=16, **spec) != taken


def test_few_rows_form_is_named_with_its_structure():
    """tile_k 4 names the column form of few rows with MFMA; with AUTO it is STAGED's field, as it was."""
    spec = dict(layout="ZGD", Z=100, G=1, D=96, NM=16, tile_n=1, unroll=8, block=64, order=1, tile_k=4)
    assert P.sj_resolve(P.SJ_LTIMES, variant=P.SJ_VAR_MFMA, **spec)["tile_k"] == 4
    assert P.sj_resolve(P.SJ_LTIMES, **spec)["tile_k"] == 16


def mass(**kw):
    spec = dict(dict(D=8, NM=12, inputs=3, count=20000), **kw)
    r = P.sj_resolve(P.SJ_MASS, **spec)
    named = {f: r[f] for f in ("tile_n", "tile_k", "block", "order")}
    assert P.sj_emit_source(P.SJ_MASS, **dict(spec, **named)) == P.sj_emit_source(P.SJ_MASS, **spec)
    return P.sj_handle_info(P.sj_specialize(P.SJ_MASS, **dict(spec, flags=P.SJ_FLAG_COMPILE_ONLY)))["kernel_name"]


# order 1 is the staged form of a wave's elements, also where its default tile (one element, 128 threads) is
# the workgroup form's; that is the default, and order 1 with its tile and block
@pytest.mark.parametrize("D,Q", [(8, 12), (9, 9), (2, 14), (5, 10)])
def test_mass_forms_by_name(D, Q):
    hexa, staged = "sj_mass_pa_hex_3d_d%d_q%d" % (D, Q), "sj_mass_pa_3d_d%d_q%d" % (D, Q)
    assert mass(D=D, NM=Q) == hexa and mass(D=D, NM=Q, order=1, tile_n=1, block=128) == hexa
    for other in (dict(order=1), dict(order=1, tile_n=1), dict(order=1, block=128), dict(order=1, block=64),
                  dict(order=1, tile_n=1, block=128, tile_k=1)):
        assert mass(D=D, NM=Q, **other) == staged, other
    for refused_ in (dict(tile_k=1), dict(order=2, tile_k=1), dict(order=1, block=64, tile_k=1), dict(order=1, tile_k=2),
                     dict(order=1, tile_k=-1), dict(inputs=2, order=1, tile_k=1)):
        assert refused(P.SJ_MASS, D=D, NM=Q, **dict(dict(inputs=3, count=20000), **refused_)), refused_


def test_mass_range_is_one_for_every_request():
    """Elements too large for the staged form's LDS are refused, also where the workgroup form is named."""
    for spec in ({}, dict(order=1), dict(order=1, tile_n=1, block=512)):
        assert refused(P.SJ_MASS, D=19, NM=19, inputs=3, count=3, **spec), spec
        assert not refused(P.SJ_MASS, D=18, NM=18, inputs=3, count=3, **spec), spec


# arrays whose last element is near 2^31 while a tile or group of elements reaches past it
@pytest.mark.parametrize("kernel,spec", [
    ("SJ_LTIMES", dict(layout="ZDG", Z=536870911, G=4, D=1, NM=1)), ("SJ_LPLUSTIMES", dict(layout="ZDG", Z=306783378, G=7, D=1, NM=1)),
    ("SJ_LTIMES", dict(layout="ZGD", Z=2147483647, G=1, D=1, NM=1)), ("SJ_LPLUSTIMES", dict(layout="GZD", Z=2147483617, G=1, D=1, NM=1)),
    ("SJ_LTIMES", dict(layout="ZGD", Z=715827882, G=1, D=3, NM=1)), ("SJ_MASS", dict(D=8, NM=4, inputs=3, count=4194303)),
    ("SJ_MASS", dict(D=2, NM=14, inputs=3, count=782610))])
def test_largest_arrays(kernel, spec):
    k = getattr(P, kernel)
    P.sj_specialize(k, flags=P.SJ_FLAG_COMPILE_ONLY, **spec)
    assert "typedef long long sj_index_t" in P.sj_emit_source(k, **spec)


# the tuner's set holds what the library takes by itself, so that tuning never returns something slower than
# not tuning: on both sides of the rules' lines
@pytest.mark.parametrize("Z,G,D,NM", [(3001, 1, 96, 36), (4096, 8, 48, 16), (32768, 32, 96, 16), (20000, 2, 128, 64), (65538, 2, 16, 64),
                                      (1800, 6, 24, 16), (8300, 2, 27, 9), (17576, 21, 80, 25), (64, 9, 16, 1), (512, 3, 113, 36)])
def test_tuner_holds_the_default(Z, G, D, NM):
    for k in (P.SJ_LTIMES, P.SJ_LPLUSTIMES):
        for layout in P.LAYOUTS:
            spec = dict(layout=layout, Z=Z, G=G, D=D, NM=NM)
            cands = tune.candidates(k, layout, Z, G, D, NM)
            want = P.sj_emit_source(k, **spec)
            assert any(want == P.sj_emit_source(k, **spec, **c) for c in tune.distinct(k, spec, cands)
                       if not refused(k, **spec, **c)), (k, layout)


def test_tuner_holds_the_bf16_default():
    spec = dict(layout="DGZ", Z=4096, G=8, D=48, NM=16, dtype=P.SJ_BF16X3)
    want = P.sj_emit_source(P.SJ_LTIMES, **spec)
    assert want in [P.sj_emit_source(P.SJ_LTIMES, **spec, **c) for c in tune.candidates(P.SJ_LTIMES, "DGZ", 4096, 8, 48, 16, P.SJ_BF16X3)]


def test_features_of_few_rows():
    """Few rows as columns are described as the column kernel that runs, with full tiles."""
    s = dict(Z=3000, G=1, D=96, NM=36, dtype=P.SJ_F64)
    f = picker.features(s, dict(layout="ZGD"))
    assert (f[15], f[16]) == (1.0, 0.0) and f[27] == 3000 / 3008
    f = picker.features(s, dict(layout="ZGD", variant=P.SJ_VAR_MFMA))
    assert (f[15], f[16]) == (0.0, 1.0)


# the column kernel's workgroups: one tile a wave where the weights are few, else rounds of at most 2048 that
# are all full, and never a launch of 2^32 threads
@pytest.mark.parametrize("kernel,layout,Z,G,D,NM,grid", [
    ("SJ_LPLUSTIMES", "ZDG", 60000, 5, 72, 9, 2344), ("SJ_LTIMES", "ZDG", 150000, 2, 72, 9, 2344), ("SJ_LTIMES", "DGZ", 300000, 1, 128, 64, 1172),
    ("SJ_LPLUSTIMES", "DGZ", 262144, 1, 128, 64, 2048), ("SJ_LTIMES", "ZDG", 750000, 2, 72, 36, 1954), ("SJ_LPLUSTIMES", "ZDG", 400000000, 5, 1, 1, 1041667)])
def test_column_rounds(kernel, layout, Z, G, D, NM, grid):
    h = P.sj_specialize(getattr(P, kernel), layout=layout, Z=Z, G=G, D=D, NM=NM, flags=P.SJ_FLAG_COMPILE_ONLY)
    info = P.sj_handle_info(h)
    assert "cols_mfma" in info["kernel_name"] and info["grid"] == grid and grid * info["block"] < 2 ** 32


# even long rows: ordinary stores, but nontemporal ones where every other line of more than 512 MiB is cut in half
@pytest.mark.parametrize("layout,Z,G,D,NM,stores", [("GDZ", 54360, 25, 64, 9, "NONTEMPORAL"), ("GDZ", 54360, 9, 64, 9, "CACHED"),
                                                    ("GDZ", 54366, 40, 64, 9, "CACHED"), ("DGZ", 250002, 4, 96, 16, "NONTEMPORAL"),
                                                    ("GDZ", 50002, 10, 64, 9, "CACHED"), ("GDZ", 54365, 40, 64, 9, "CACHED")])
def test_stores_of_half_lines(layout, Z, G, D, NM, stores):
    for kernel in (P.SJ_LPLUSTIMES, P.SJ_LTIMES_LPLUS):
        flags = P.sj_resolve(kernel, layout=layout, Z=Z, G=G, D=D, NM=NM)["flags"]
        assert flags & getattr(P, "SJ_FLAG_STORES_" + stores)


# nm innermost: few groups of many moments by a thread per line, from 150,000 lines on
@pytest.mark.parametrize("layout", ["ZGD", "GZD"])
@pytest.mark.parametrize("Z,G,NM,sorted_", [(20001, 8, 16, False), (9376, 8, 16, False), (9374, 8, 16, True), (20001, 8, 15, True), (20001, 9, 16, True),
                                            (5001, 9, 36, False), (5001, 10, 36, False), (20001, 10, 25, True), (5001, 11, 36, True), (3001, 9, 36, True)])
def test_sorted_scattering_of_many_moments(layout, Z, G, NM, sorted_):
    info = P.sj_resolve(P.SJ_SCATTERING, layout=layout, Z=Z, G=G, NM=NM, count=4)
    assert bool(info["tile_k"]) == sorted_
