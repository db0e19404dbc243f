"""GPU parity of the stencil applies (Wilson, Brillouin, staggered, their adjoints) against the oracle.

Bars: FP64 1e-12 and FP32 1e-5 relative, each on two metrics (the worst per-RHS column 2-norm error
and the element-wise max error over max |ref|, so that a localized error is not diluted), with the
oracle evaluated in FP64 on the same rounded inputs; BF16 storage is reported and held to a sanity
bound of 2e-2 (bfloat16 keeps 8 significant bits).
"""
import numpy as np
import pytest
import torch

import synthetic_inputs as si
from oracle.brillouin import (brillouin_apply, brillouin_apply_dagger, brillouin_apply_sites, brillouin_links,
                              brillouin_links_all)
from oracle.dense import wilson_dense
from oracle.staggered import staggered_apply, staggered_apply_dagger
from oracle.wilson import free_wilson_symbol, wilson_apply, wilson_apply_dagger
from paper_2112_14640_amd import dirac
from tests.gpu_helpers import (at_sites, bf16_pairs_to_host, col_rel_err, host, parity, round_bf16, round_c64,
                               sample_sites, to_bf16_pairs, to_dev)

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32": 1e-5, "bf16": 2e-2}

ORACLE = {
    ("wilson", False): wilson_apply,
    ("wilson", True): wilson_apply_dagger,
    ("brillouin", False): brillouin_apply,
    ("brillouin", True): brillouin_apply_dagger,
    ("staggered", False): staggered_apply,
    ("staggered", True): staggered_apply_dagger,
}


def _inputs(op, dims, nc, nv, seed, kind="haar"):
    rng = np.random.default_rng(seed)
    U = si.gauge_field(rng, dims, nc, kind, 0.3)
    if op == "staggered":
        u = si.staggered_vector(rng, dims, nc, nv)
    else:
        u = si.wilson_vector(rng, dims, nc, nv)
    gauge = brillouin_links(U) if op == "brillouin" else U
    return gauge, u


def _run(op, prec, gauge, u, mass, apbc, dagger):
    """Device result (as complex128 host array) and the oracle's input values."""
    if prec == "fp64":
        g_in, u_in = gauge, u
        gd, ud = to_dev(gauge), to_dev(u)
    elif prec == "fp32":
        g_in, u_in = round_c64(gauge), round_c64(u)
        gd, ud = to_dev(gauge, torch.complex64), to_dev(u, torch.complex64)
    else:
        g_in, u_in = round_c64(gauge), round_bf16(u)
        gd, ud = to_dev(gauge, torch.complex64), to_bf16_pairs(u)
    fn = dirac.apply_dagger if dagger else dirac.apply
    v = fn(op, gd, ud, mass, antiperiodic_t=apbc)
    torch.cuda.synchronize()
    vh = bf16_pairs_to_host(v) if prec == "bf16" else host(v).astype(np.complex128)
    return vh, g_in, u_in


def test_wilson_4x4_dense_fp64():
    """Wilson 4^4, Nc=3, Nv=1, Haar links, m=0.1, antiperiodic t: D u and D^dagger u vs the dense 3072^2 matrix."""
    cfg = si.config("wilson_4x4_dense")
    rng = np.random.default_rng(cfg["seed"])
    U = si.gauge_field(rng, cfg["dims"], cfg["nc"], "haar")
    u = si.wilson_vector(rng, cfg["dims"], cfg["nc"], cfg["nv"])
    d = wilson_dense(U, cfg["mass"], True)
    cols = u.reshape(-1, 1)
    for dagger, mat in ((False, d), (True, d.conj().T)):
        v, _, _ = _run("wilson", "fp64", U, u, cfg["mass"], True, dagger)
        parity(v, (mat @ cols).reshape(u.shape), 1e-12, dagger)


SMALL = [
    # dims (Nx,Ny,Nz,Nt), nc, nv, antiperiodic: several blocks of threads and a ragged last block
    ((6, 4, 4, 10), 3, 3, True),
    ((4, 6, 2, 8), 3, 12, True),
    ((4, 2, 6, 4), 2, 4, False),
    ((2, 2, 2, 2), 4, 2, True),
    ((4, 4, 2, 6), 1, 1, True),
]


@pytest.mark.parametrize("op", ["wilson", "staggered", "brillouin"])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("case", range(len(SMALL)))
def test_small_lattice_parity(op, prec, case):
    dims, nc, nv, apbc = SMALL[case]
    gauge, u = _inputs(op, dims, nc, nv, seed=100 + case)
    for dagger in (False, True):
        v, g_in, u_in = _run(op, prec, gauge, u, 0.07, apbc, dagger)
        ref = ORACLE[(op, dagger)](g_in, u_in, 0.07, apbc)
        parity(v, ref, TOL[prec], (op, prec, dims, nc, nv, dagger))


# odd extents (the staggered phases need even ones) and an odd RHS count: (5,3,3,5) x 13 takes the row kernels
# with 65 threads per row and one RHS per thread, (3,5,3,3) x 5 the direct kernels
ODD = [((5, 3, 3, 5), 3, 13, True), ((3, 5, 3, 3), 2, 5, True), ((5, 3, 3, 5), 3, 13, False)]


@pytest.mark.parametrize("op", ["wilson", "brillouin"])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("case", range(len(ODD)))
def test_odd_extents_and_rhs_parity(op, prec, case):
    dims, nc, nv, apbc = ODD[case]
    gauge, u = _inputs(op, dims, nc, nv, seed=140 + case)
    for dagger in (False, True):
        v, g_in, u_in = _run(op, prec, gauge, u, 0.07, apbc, dagger)
        ref = ORACLE[(op, dagger)](g_in, u_in, 0.07, apbc)
        parity(v, ref, TOL[prec], (op, prec, dims, nc, nv, dagger))


@pytest.mark.parametrize("op", ["wilson", "staggered", "brillouin"])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_largest_rhs_count(op, prec):
    """N_v = 256, the largest the library takes (Wilson and staggered rows of 512 and 256 threads, Brillouin on
    the direct kernel), and N_v = 257 refused before any launch."""
    dims, nc, nv = (2, 2, 2, 4), 3, 256
    gauge, u = _inputs(op, dims, nc, nv, seed=150)
    for dagger in (False, True):
        v, g_in, u_in = _run(op, prec, gauge, u, 0.07, True, dagger)
        parity(v, ORACLE[(op, dagger)](g_in, u_in, 0.07, True), TOL[prec], (op, prec, nv, dagger))
    _, u_big = _inputs(op, dims, nc, nv + 1, seed=151)
    with pytest.raises(Exception):
        _run(op, prec, gauge, u_big, 0.07, True, False)


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("op", ["wilson", "staggered", "brillouin"])
def test_apply_16x32_nv12_sampled(op, prec):
    """Config 16^3x32, Nc=3, Nv=12, links exp(i 0.3 H), m=0.05: ~1000 sampled output sites + t boundaries.
    Brillouin runs on the links W the GPU builds from U; the oracle forms all 81 W_d at the sampled
    sites from the same (FP32-rounded) U."""
    cfg = si.config("apply_16x32")
    rng = np.random.default_rng(cfg["seed"])
    dims, nc, nv, m = cfg["dims"], cfg["nc"], cfg["nv"], cfg["mass"]
    U = si.gauge_field(rng, dims, nc, "near", cfg["spread"])
    u = si.staggered_vector(rng, dims, nc, nv) if op == "staggered" else si.wilson_vector(rng, dims, nc, nv)
    sites = sample_sites(dims, 1000)
    if prec == "fp32":
        ud, u_in = to_dev(u, torch.complex64), round_c64(u)
    else:
        ud, u_in = to_bf16_pairs(u), round_bf16(u)
    U32 = to_dev(U, torch.complex64)
    gauge = dirac.brillouin_links(U32) if op == "brillouin" else U32
    W81 = brillouin_links_all(round_c64(U), sites=sites) if op == "brillouin" else None
    for dagger in (False, True):
        fn = dirac.apply_dagger if dagger else dirac.apply
        v = fn(op, gauge, ud, m)
        vh = bf16_pairs_to_host(v) if prec == "bf16" else host(v).astype(np.complex128)
        if op == "brillouin":
            ref = brillouin_apply_sites(W81, u_in, m, sites, True, dagger)
        else:
            ref = ORACLE[(op, dagger)](round_c64(U), u_in, m, True, sites=sites)
        parity(at_sites(vh, sites), ref, 1e-5 if prec == "fp32" else TOL["bf16"], (op, prec, dagger))


def test_brillouin_links_parity():
    dims, nc = (4, 6, 4, 6), 3
    rng = np.random.default_rng(7)
    U = si.gauge_field(rng, dims, nc, "haar")
    ref = brillouin_links(U)
    W = dirac.brillouin_links(to_dev(U))
    assert np.max(np.abs(host(W) - ref)) < 1e-13
    W32 = dirac.brillouin_links(to_dev(U, torch.complex64))
    ref32 = brillouin_links(round_c64(U))
    assert np.max(np.abs(host(W32).astype(np.complex128) - ref32)) < 2e-6


@pytest.mark.parametrize("nc", [1, 2, 3, 4])
@pytest.mark.parametrize("dims", [(3, 3, 2, 3), (2, 4, 3, 2)])
def test_brillouin_links_all_colours_and_ragged_tiles(nc, dims):
    """The level-by-level link build against the oracle's path-by-path averages for every supported N_c, on
    volumes that leave the last work-group's tile of sites partly empty (54 and 48 sites; tiles of 4 sites for
    N_c <= 3, 2 for N_c = 4), with extents of 2 and 3 where the +1 and -1 steps reach the same neighbour."""
    rng = np.random.default_rng(70 + nc)
    U = si.gauge_field(rng, dims, nc, "haar")
    ref = brillouin_links(U)
    assert np.max(np.abs(host(dirac.brillouin_links(to_dev(U))) - ref)) < 1e-13
    ref32 = brillouin_links(round_c64(U))
    W32 = host(dirac.brillouin_links(to_dev(U, torch.complex64))).astype(np.complex128)
    assert np.max(np.abs(W32 - ref32)) < 2e-6


def test_brillouin_links_16x32_sampled():
    cfg = si.config("apply_16x32")
    rng = np.random.default_rng(cfg["seed"])
    U = si.gauge_field(rng, cfg["dims"], 3, "near", cfg["spread"])
    W = host(dirac.brillouin_links(to_dev(U, torch.complex64))).astype(np.complex128)
    sites = sample_sites(cfg["dims"], 150)
    ref = brillouin_links_all(round_c64(U), sites=sites)[:, :40]
    assert np.max(np.abs(at_sites(W, sites) - ref)) < 2e-6


@pytest.mark.parametrize("op", ["wilson", "brillouin"])
def test_gamma5_hermiticity_16x32(op):
    """D^dagger u = gamma5 D gamma5 u at the benchmark size (a property that holds at any size)."""
    cfg = si.config("apply_16x32")
    rng = np.random.default_rng(3)
    dims, nc, nv = cfg["dims"], 3, 12
    U = si.gauge_field(rng, dims, nc, "near", 0.3)
    Ud = to_dev(U, torch.complex64)
    gauge = dirac.brillouin_links(Ud) if op == "brillouin" else Ud
    u = to_dev(si.wilson_vector(rng, dims, nc, nv), torch.complex64)
    lhs = dirac.apply_dagger(op, gauge, u, 0.05)
    rhs = dirac.gamma5(op, dirac.apply(op, gauge, dirac.gamma5(op, u), 0.05))
    parity(host(lhs), host(rhs), 1e-6, op)


def test_staggered_epsilon_hermiticity_16x32():
    cfg = si.config("apply_16x32")
    rng = np.random.default_rng(4)
    dims, nc, nv = cfg["dims"], 3, 12
    U = to_dev(si.gauge_field(rng, dims, nc, "near", 0.3), torch.complex64)
    u = to_dev(si.staggered_vector(rng, dims, nc, nv), torch.complex64)
    lhs = dirac.apply_dagger("staggered", U, u, 0.05)
    rhs = dirac.gamma5("staggered", dirac.apply("staggered", U, dirac.gamma5("staggered", u), 0.05))
    parity(host(lhs), host(rhs), 1e-6)


def test_free_field_plane_wave_16x32():
    """At U = 1 an antiperiodic plane wave is an eigenvector of D_W with the closed-form symbol."""
    dims = (16, 16, 16, 32)
    nx, ny, nz, nt = dims
    U = si.gauge_field(None, dims, 3, "unit")
    p = np.array([2 * np.pi * 3 / nx, 2 * np.pi * 5 / ny, 2 * np.pi * 1 / nz, np.pi * 7 / nt])
    rng = np.random.default_rng(5)
    chi = si.complex_gaussian(rng, (3, 4, 2))
    t, z, y, x = np.meshgrid(np.arange(nt), np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    ph = np.exp(1j * (p[0] * x + p[1] * y + p[2] * z + p[3] * t))
    psi = ph[..., None, None, None] * chi
    expect = ph[..., None, None, None] * np.einsum("st,atr->asr", free_wilson_symbol(p, 0.05), chi)
    v = dirac.apply("wilson", to_dev(U), to_dev(psi), 0.05)
    parity(host(v), expect, 1e-12)


# right-hand sides per thread instantiated for each operator; every other rb is refused
RB_OF = {"wilson": (1, 2), "staggered": (1, 2, 4), "brillouin": (1,)}


@pytest.mark.parametrize("variant", [0, 1, 4])
@pytest.mark.parametrize("rb", [1, 2, 4])
@pytest.mark.parametrize("op", ["wilson", "staggered", "brillouin"])
def test_launch_shapes_agree(op, rb, variant):
    """Every launch shape (RHS per thread, row tiles or direct loads) gives the oracle's result; a shape
    that is not instantiated is refused."""
    if rb not in RB_OF[op]:
        with pytest.raises(Exception):
            dirac.set_launch_shape(op, "fp32", rb, variant)
        dirac.set_launch_shape(op, "fp32", 0, 0)
        return
    dims, nc, nv = (6, 4, 4, 6), 3, 12
    gauge, u = _inputs(op, dims, nc, nv, seed=9)
    try:
        dirac.set_launch_shape(op, "fp32", rb, variant)
        v, g_in, u_in = _run(op, "fp32", gauge, u, 0.1, True, False)
    finally:
        dirac.set_launch_shape(op, "fp32", 0, 0)
    ref = ORACLE[(op, False)](g_in, u_in, 0.1, True)
    parity(v, ref, 1e-5, (op, rb, variant))


ROW_CASES = [
    # dims, nc, nv, antiperiodic: rows of 6, 4, 3 and 10 sites, one to four rows per tile
    ((6, 4, 4, 6), 3, 12, True),
    ((4, 2, 6, 4), 2, 4, False),
    ((3, 2, 2, 4), 3, 6, True),
    ((10, 2, 2, 2), 1, 2, True),
    ((4, 4, 2, 6), 4, 1, True),
    # tile orders with 3 x 1 and 3 x 3 (y, z) block grids (ny = 12 in blocks of 4, nz = 6 in blocks of
    # 2), blocks of one row (ny = 3, nz = 5) and t extents of 10 and 6 (the scalar magic divisions)
    ((8, 12, 6, 10), 3, 12, True),
    ((8, 3, 5, 6), 3, 8, False),
]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("case", range(len(ROW_CASES)))
def test_wilson_row_tiles(case, prec):
    """The row-tiled Wilson kernel (1 and 2 RHS per thread; links staged in LDS at Nv = 12) against the
    oracle."""
    dims, nc, nv, apbc = ROW_CASES[case]
    gauge, u = _inputs("wilson", dims, nc, nv, seed=40 + case)
    for rb in (1, 2):
        if nv % rb:
            continue
        try:
            dirac.set_launch_shape("wilson", prec, rb, 4)
            for dagger in (False, True):
                v, g_in, u_in = _run("wilson", prec, gauge, u, 0.03, apbc, dagger)
                parity(v, ORACLE[("wilson", dagger)](g_in, u_in, 0.03, apbc), TOL[prec], (dims, nc, nv, rb, dagger))
        finally:
            dirac.set_launch_shape("wilson", prec, 0, 0)


BRILLOUIN_ROW_CASES = [
    # dims, nc, nv, antiperiodic: rows of 6, 8 and 7 sites (at least 64 threads per row); the fifth
    # case does not fit a row tile (a site block of 56 bytes) and takes the direct kernel; the last
    # two cut rows of 32 and 48 sites into x-segments with one halo site on each side
    ((6, 4, 4, 6), 3, 12, True),
    ((8, 2, 6, 4), 2, 8, False),
    ((7, 2, 2, 4), 3, 12, True),
    ((6, 2, 2, 4), 4, 12, True),
    ((4, 4, 2, 2), 1, 7, True),
    ((32, 2, 2, 4), 3, 12, True),  # rows cut into segments of 16 sites (FP32, FP64) or 32 (BF16)
    ((48, 2, 2, 2), 3, 12, True),
    ((6, 6, 3, 4), 3, 12, True),  # a 3 x 3 grid of 2 x 1 (y, z) blocks in the tile order
]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("case", range(len(BRILLOUIN_ROW_CASES)))
def test_brillouin_row_tiles(case, prec):
    """The row-tiled Brillouin kernel (27 row copies with link windows in LDS, one RHS per thread, the
    only instantiated shape) against the oracle."""
    dims, nc, nv, apbc = BRILLOUIN_ROW_CASES[case]
    gauge, u = _inputs("brillouin", dims, nc, nv, seed=60 + case)
    try:
        dirac.set_launch_shape("brillouin", prec, 1, 4)
        for dagger in (False, True):
            v, g_in, u_in = _run("brillouin", prec, gauge, u, 0.04, apbc, dagger)
            parity(v, ORACLE[("brillouin", dagger)](g_in, u_in, 0.04, apbc), TOL[prec], (dims, nc, nv, dagger))
    finally:
        dirac.set_launch_shape("brillouin", prec, 0, 0)


STAGGERED_ROW_CASES = [
    # dims (even), nc, nv, antiperiodic: rows of 8 and 16 sites, 64..192 threads per row
    ((8, 4, 4, 6), 3, 12, True),
    ((16, 2, 2, 4), 3, 12, True),
    ((8, 2, 2, 4), 2, 8, False),
    ((8, 2, 2, 2), 4, 12, True),
    ((16, 6, 10, 6), 3, 12, True),  # 3 x 5 grid of 2 x 2 (y, z) blocks
]


# (dims, nc, nv): a thread per chirality and colour row (small launches), whole rows, segments with a halo whose last one
# overlaps, and fewer than 64 threads; then launches large enough for the other forms: several window entries per lane,
# FP64's chirality threads and colour rows on whole rows and on overlapping segments
BRILLOUIN_THREAD_CASES = [
    ((8, 2, 3, 2), 3, 4), ((22, 2, 2, 3), 3, 12), ((8, 2, 2, 2), 3, 1), ((5, 3, 2, 2), 2, 13), ((6, 2, 3, 2), 4, 12),
    ((16, 2, 2, 2), 1, 2), ((7, 2, 2, 3), 4, 5), ((4, 2, 2, 2), 3, 3),
    ((16, 9, 12, 10), 3, 4), ((22, 5, 5, 5), 3, 12), ((11, 9, 8, 9), 3, 7), ((16, 8, 8, 9), 2, 12),
    ((13, 9, 8, 8), 3, 12),
]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("case", range(len(BRILLOUIN_THREAD_CASES)))
def test_brillouin_thread_forms(case, prec):
    dims, nc, nv = BRILLOUIN_THREAD_CASES[case]
    gauge, u = _inputs("brillouin", dims, nc, nv, seed=540 + case)
    dagger = case % 2 == 1
    v, g_in, u_in = _run("brillouin", prec, gauge, u, 0.05, True, dagger)
    parity(v, ORACLE[("brillouin", dagger)](g_in, u_in, 0.05, True), TOL[prec], (prec, dims, nc, nv))


@pytest.mark.parametrize("dims,nc,nv", BRILLOUIN_THREAD_CASES[:8] + [((4, 2, 2, 3), 1, 4), ((6, 2, 2, 2), 2, 2)])
def test_brillouin_bf16_rounds_once(dims, nc, nv):
    """BF16 vectors are summed in FP32 and rounded when they are stored, whatever form a launch takes: each real number
    is within half a unit of its own last place (2^-8 of it) of the exact value, and FP32's error of the largest."""
    gauge, u = _inputs("brillouin", dims, nc, nv, seed=620 + nv)
    for dagger in (False, True):
        v, g_in, u_in = _run("brillouin", "bf16", gauge, u, 0.05, True, dagger)
        ref = ORACLE[("brillouin", dagger)](g_in, u_in, 0.05, True)
        fp32 = TOL["fp32"] * np.max(np.abs(ref))
        for got, want in ((v.real, ref.real), (v.imag, ref.imag)):
            assert np.max(np.abs(got - want) - 2.0 ** -8 * np.abs(want)) < fp32, (dims, nc, nv, dagger)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("op,dims,nc,nv", [("wilson", (5, 3, 2, 3), 3, 1), ("wilson", (3, 4, 2, 2), 3, 2),
                                           ("wilson", (7, 3, 3, 2), 2, 1), ("wilson", (3, 2, 5, 2), 4, 2),
                                           ("wilson", (3, 2, 2, 3), 1, 3), ("staggered", (4, 2, 6, 2), 3, 1),
                                           ("staggered", (2, 4, 2, 2), 4, 2), ("brillouin", (3, 2, 3, 2), 3, 1)])
def test_direct_kernels_few_rhs(op, dims, nc, nv, prec):
    """Shapes below a row tile: site blocks contiguous in a thread (N_v = 1 and 2) and strided."""
    gauge, u = _inputs(op, dims, nc, nv, seed=560 + nv)
    for dagger in (False, True):
        v, g_in, u_in = _run(op, prec, gauge, u, 0.05, True, dagger)
        parity(v, ORACLE[(op, dagger)](g_in, u_in, 0.05, True), TOL[prec], (op, prec, dims, nc, nv, dagger))


# (dims, nc, nv) of the Wilson row form: links staged in LDS with N_v known only at run time, with one and with two
# right-hand sides per thread, and rows whose staged links need more than 64 KiB of LDS
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("dims,nc,nv", [((16, 2, 2, 3), 3, 4), ((11, 3, 2, 2), 2, 7), ((24, 2, 2, 2), 3, 24),
                                        ((32, 2, 2, 2), 3, 12), ((9, 2, 3, 2), 4, 8)])
def test_wilson_staged_links(dims, nc, nv, prec):
    gauge, u = _inputs("wilson", dims, nc, nv, seed=580 + nv)
    for dagger in (False, True):
        v, g_in, u_in = _run("wilson", prec, gauge, u, 0.05, True, dagger)
        parity(v, ORACLE[("wilson", dagger)](g_in, u_in, 0.05, True), TOL[prec], (prec, dims, nc, nv, dagger))


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("case", range(len(STAGGERED_ROW_CASES)))
def test_staggered_row_tiles(case, prec):
    """The row-tiled staggered kernel (1, 2 and 4 RHS per thread, where a row fits; links staged in LDS
    in FP32/BF16, loaded per thread in FP64) against the oracle."""
    dims, nc, nv, apbc = STAGGERED_ROW_CASES[case]
    gauge, u = _inputs("staggered", dims, nc, nv, seed=80 + case)
    for rb in (1, 2, 4):
        if nv % rb:
            continue
        try:
            dirac.set_launch_shape("staggered", prec, rb, 4)
            for dagger in (False, True):
                v, g_in, u_in = _run("staggered", prec, gauge, u, 0.06, apbc, dagger)
                parity(v, ORACLE[("staggered", dagger)](g_in, u_in, 0.06, apbc), TOL[prec],
                       (dims, nc, nv, rb, dagger))
        finally:
            dirac.set_launch_shape("staggered", prec, 0, 0)


def test_invalid_arguments_raise():
    U = torch.zeros((4, 4, 4, 4, 4, 3, 3), dtype=torch.complex64, device="cuda:0")
    u = torch.zeros((4, 4, 4, 4, 3, 4, 2), dtype=torch.complex64, device="cuda:0")
    with pytest.raises(Exception):
        dirac.apply("wilson", U.to(torch.complex128), u, 0.1)  # gauge precision mismatch
    with pytest.raises(Exception):
        dirac.apply("wilson", U, u, 0.1, out=u)  # in-place is rejected by the library
    bad = torch.zeros((3, 4, 4, 4, 3, 2), dtype=torch.complex64, device="cuda:0")
    Us = torch.zeros((3, 4, 4, 4, 4, 3, 3), dtype=torch.complex64, device="cuda:0")
    with pytest.raises(Exception):
        dirac.apply("staggered", Us, bad, 0.1)  # odd extent for staggered
