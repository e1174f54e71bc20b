"""GPU CG solvers judged by the FP64 oracle.

Every solve's true residual ||b - M_e x|| / ||b|| is recomputed by the oracle
(FP64, its own Dslash) from the GPU's solution and must meet the requested
tolerance.  Several solutions are correct within that tolerance, so the
difference to the oracle's own CG solution is only bounded by the condition
number, not compared element by element.
"""
import numpy as np
import pytest
import torch

import hisq_inputs as gen
from oracle import hisq as O

pytestmark = pytest.mark.gpu


def setup(h, w, inner, nrhs, src=None, ctx=None):
    dims, t_bc = w["dims"], w["t_bc"]
    lat = h.lattice(dims, t_bc)
    l64 = h.pack_links_from_host(lat, "fp64", w["fat"], w["naik"])
    lin = None if inner == "fp64" else h.pack_links_from_host(lat, inner, w["fat"], w["naik"])
    src = w["src"][:nrhs] if src is None else src
    b = h.pack_field_from_host(lat, "fp64", src)
    x = h.empty_field(lat, "fp64", nrhs)
    x.zero_()
    ws = h.empty_workspace(h.hisq_cg_workspace_bytes(lat, inner, nrhs, 0))
    return lat, l64, lin, b, x, ws


def oracle_residuals(h, w, lat, x, nrhs, mass, src):
    xs = h.unpack_field_to_host(lat, "fp64", x, nrhs)
    lat_o = O.lattice_from(w)
    return [O.true_residual(lat_o, mass, src[j], xs[j]) for j in range(nrhs)], xs


@pytest.mark.parametrize("t_bc", [+1, -1])
def test_cg_fp64_8x8x8x8(gpu_lib, t_bc):
    """Haar links, m = 0.1, tol 1e-10 (the 8^4 workload, both time BCs)."""
    h = gpu_lib
    w = gen.workload_haar((8, 8, 8, 8), 1, t_bc)
    lat, l64, lin, b, x, ws = setup(h, w, "fp64", 1)
    st, info = h.hisq_cg(lat, 0.1, l64, None, "fp64", 1, b, x, 1e-10, 5000, ws)
    assert st == h.OK, info
    res, xs = oracle_residuals(h, w, lat, x, 1, 0.1, w["src"])
    assert res[0] <= 1e-10 and info[0]["true_residual"] <= 1e-10
    assert abs(res[0] - info[0]["true_residual"]) <= 1e-12
    ref = O.cg(O.lattice_from(w), 0.1, w["src"][0], 1e-12, 5000)
    # kappa(M_e) <= (m^2 + ||D||^2) / m^2 ~ 6e3: the two solutions agree to kappa * tol
    assert O.norm(xs[0] - ref.x) <= 1e4 * 1e-10 * O.norm(ref.x)
    # iteration counts depend on the summation order in finite precision (Haar
    # links make this problem sensitive); they are reported, not pinned
    print(f"\n8^4 t_bc={t_bc}: GPU {info[0]['iterations']} iterations, oracle {ref.iterations}")


@pytest.mark.parametrize("inner,m", [("fp32", 0.02), ("fp16n", 0.2), ("fp32r12", 0.02)])
def test_mixed_precision_reliable_update_cg(gpu_lib, inner, m):
    """FP16 links perturb M_e by ~2^-12 ||D||^2 ~ 1e-2, far above the lowest
    eigenvalues at m = 0.02 (where FP16 inner iterations barely make progress,
    as a CPU emulation of the same algorithm shows); the FP16 case runs at a
    mass where that perturbation is small against m^2."""
    h = gpu_lib
    w = gen.workload_smooth((8, 8, 8, 16), 41, -1, 0.3, 1)
    lat, l64, lin, b, x, ws = setup(h, w, inner, 1)
    st, info = h.hisq_cg(lat, m, l64, lin, inner, 1, b, x, 1e-10, 20000, ws)
    assert st == h.OK, info
    res, _ = oracle_residuals(h, w, lat, x, 1, m, w["src"])
    assert res[0] <= 1e-10
    assert info[0]["reliable_updates"] >= 1


@pytest.mark.parametrize("inner,m", [("fp32", 0.05), ("fp32r12", 0.05), ("fp16n", 0.2)])
def test_multi_rhs_cg_lds_staged_default(gpu_lib, inner, m):
    """Where N_y and N_z divide by 8 and N_x is 16..64, the built-in shape of a
    multi-column solve with FP32 fields stages the x- and y-hop vectors in LDS
    (four columns per thread; six columns: a ragged second group).  Every
    column meets the tolerance by the oracle."""
    h = gpu_lib
    nrhs = 6
    w = gen.workload_smooth((16, 8, 8, 8), 43, -1, 0.3, nrhs)
    lat, l64, lin, b, x, ws = setup(h, w, inner, nrhs)
    if inner != "fp16n":  # the query reports FP16N fields; the iterations use FP32 fields
        assert h.hisq_get_dslash_shape(lat, inner, nrhs, None)[:2] == (2, 4)
    st, info = h.hisq_cg(lat, m, l64, lin, inner, nrhs, b, x, 1e-10, 20000, ws)
    assert st == h.OK, info
    res, _ = oracle_residuals(h, w, lat, x, nrhs, m, w["src"])
    assert max(res) <= 1e-10, res


@pytest.mark.parametrize("inner,nrhs", [("fp64", 3), ("fp32", 16), ("fp32", 5)])
def test_multi_rhs_cg(gpu_lib, inner, nrhs):
    h = gpu_lib
    w = gen.workload_smooth((8, 4, 8, 8), 42, -1, 0.3, nrhs)
    m = 0.05
    src = w["src"] * (10.0 ** np.arange(nrhs) % 7 + 1)[:, None, None]  # uneven norms
    lat, l64, lin, b, x, ws = setup(h, w, inner, nrhs, src=src)
    # one right-hand side per thread and the same block size for the batched
    # and the single solve, in the iterations and in the FP64 true residuals
    # (formed for all columns at once in the batched solve): the same
    # summation order in every reduction
    ctx = h.Context(0)
    for prec in {inner, "fp64"}:
        h.hisq_set_dslash_shape(lat, prec, nrhs, (0, 1, 128, 1), ctx)
        h.hisq_set_dslash_shape(lat, prec, 1, (0, 1, 128, 1), ctx)
    st, info = h.hisq_cg(lat, m, l64, lin, inner, nrhs, b, x, 1e-10, 20000, ws, ctx=ctx)
    assert st == h.OK, info
    res, xs = oracle_residuals(h, w, lat, x, nrhs, m, src)
    assert max(res) <= 1e-10, res
    # each column is an independent solve: the same result as solving it alone
    lat1, l64b, linb, b1, x1, ws1 = setup(h, w, inner, 1, src=src[nrhs - 1:])
    st1, info1 = h.hisq_cg(lat1, m, l64b, linb, inner, 1, b1, x1, 1e-10, 20000, ws1, ctx=ctx)
    assert st1 == h.OK
    assert info1[0]["iterations"] == info[nrhs - 1]["iterations"]
    np.testing.assert_array_equal(h.unpack_field_to_host(lat1, "fp64", x1)[0], xs[nrhs - 1])
    # with the built-in shapes the columns still reach the tolerance
    x.zero_()
    st, info = h.hisq_cg(lat, m, l64, lin, inner, nrhs, b, x, 1e-10, 20000, ws)
    assert st == h.OK and max(oracle_residuals(h, w, lat, x, nrhs, m, src)[0]) <= 1e-10


def test_initial_guess_and_determinism(gpu_lib):
    h = gpu_lib
    w = gen.workload_haar((8, 8, 4, 8), 43, -1)
    lat, l64, lin, b, x, ws = setup(h, w, "fp64", 1)
    st, info = h.hisq_cg(lat, 0.1, l64, None, "fp64", 1, b, x, 1e-10, 5000, ws)
    assert st == h.OK
    x2 = torch.zeros_like(x)
    st2, info2 = h.hisq_cg(lat, 0.1, l64, None, "fp64", 1, b, x2, 1e-10, 5000, ws)
    torch.cuda.synchronize()
    assert torch.equal(x, x2) and info[0]["iterations"] == info2[0]["iterations"]
    # restarting from the solution converges immediately
    st3, info3 = h.hisq_cg(lat, 0.1, l64, None, "fp64", 1, b, x2, 1e-10, 5000, ws)
    assert st3 == h.OK and info3[0]["iterations"] == 0
    # resume: a loose solve, then tighten from it
    x4 = torch.zeros_like(x)
    h.hisq_cg(lat, 0.1, l64, None, "fp64", 1, b, x4, 1e-4, 5000, ws)
    st5, info5 = h.hisq_cg(lat, 0.1, l64, None, "fp64", 1, b, x4, 1e-11, 5000, ws)
    assert st5 == h.OK and info5[0]["true_residual"] <= 1e-11


def test_status_codes(gpu_lib):
    h = gpu_lib
    w = gen.workload_haar((4, 4, 4, 8), 44, -1)
    lat, l64, lin, b, x, ws = setup(h, w, "fp64", 1)
    st, info = h.hisq_cg(lat, 0.05, l64, None, "fp64", 1, b, x, 1e-12, 3, ws)
    assert st == h.NOT_CONVERGED and info[0]["iterations"] == 3
    assert info[0]["true_residual"] > 1e-12
    bad = w["src"].copy()
    bad[0, 0, 0] = np.nan
    bnan = h.pack_field_from_host(lat, "fp64", bad)
    x.zero_()
    st, info = h.hisq_cg(lat, 0.05, l64, None, "fp64", 1, bnan, x, 1e-10, 100, ws)
    assert st == h.BREAKDOWN
    zero = h.pack_field_from_host(lat, "fp64", np.zeros_like(w["src"]))
    x.fill_(0)
    st, info = h.hisq_cg(lat, 0.05, l64, None, "fp64", 1, zero, x, 1e-10, 100, ws)
    assert st == h.OK and info[0]["iterations"] == 0
    small = h.empty_workspace(1024)
    with pytest.raises(h.HisqError) as e:
        h.hisq_cg(lat, 0.05, l64, None, "fp64", 1, b, x, 1e-10, 100, small)
    assert e.value.status == h.WORKSPACE
    with pytest.raises(h.HisqError):
        h.hisq_cg(lat, 0.0, l64, None, "fp64", 1, b, x, 1e-10, 100, ws)


@pytest.mark.parametrize("inner", ["fp64", "fp32", "fp16n", "fp64r12", "fp32r12"])
def test_cg_32x32x32x8_m001(gpu_lib, inner):
    """The 32^3x8 smooth-link workload at m = 0.01 to true residual 1e-10."""
    h = gpu_lib
    w = gen.workload_2()
    lat, l64, lin, b, x, ws = setup(h, w, inner, 1)
    st, info = h.hisq_cg(lat, w["mass"], l64, lin, inner, 1, b, x, 1e-10, 40000, ws)
    assert st == h.OK, info
    res, _ = oracle_residuals(h, w, lat, x, 1, w["mass"], w["src"])
    assert res[0] <= 1e-10
    print(f"\n32^3x8 {inner}: {info[0]}")


def test_multishift_with_r12_inner_links(gpu_lib):
    """Multi-shift CG whose Krylov iterations use reconstruct-12 FP32 links."""
    h = gpu_lib
    w = gen.workload_smooth((8, 8, 8, 8), 44, -1, 0.3, 1)
    lat = h.lattice(w["dims"], w["t_bc"])
    l64 = h.pack_links_from_host(lat, "fp64", w["fat"], w["naik"])
    l12 = h.pack_links_from_host(lat, "fp32r12", w["fat"], w["naik"])
    b = h.pack_field_from_host(lat, "fp64", w["src"][0])
    shifts = [0.0, 0.01, 0.1]
    xs = [h.empty_field(lat, "fp64") for _ in shifts]
    ws = h.empty_workspace(h.hisq_cg_workspace_bytes(lat, "fp32r12", 1, len(shifts)))
    st, info = h.hisq_multishift_cg(lat, 0.05, l64, l12, "fp32r12", shifts, b, xs, 1e-10, 20000, ws)
    assert st == h.OK, info
    lat_o = O.lattice_from(w)
    for k, sh in enumerate(shifts):
        xk = h.unpack_field_to_host(lat, "fp64", xs[k])[0]
        assert O.true_residual(lat_o, 0.05, w["src"][0], xk, shift=sh) <= 1e-10


def test_multi_rhs_zero_column_and_iteration_limit(gpu_lib):
    """Mixed-precision multi-RHS CG with one zero source: that column is done
    before the first iteration (x stays 0) while the others reach the
    tolerance through the batched FP64 true residuals; with a limit of 5
    iterations every nonzero column stops at exactly 5."""
    h = gpu_lib
    nrhs = 4
    w = gen.workload_smooth((8, 8, 8, 8), 46, -1, 0.3, nrhs)
    src = w["src"].copy()
    src[1] = 0.0
    m = 0.1
    lat, l64, lin, b, x, ws = setup(h, w, "fp32", nrhs, src=src)
    st, info = h.hisq_cg(lat, m, l64, lin, "fp32", nrhs, b, x, 1e-10, 20000, ws)
    assert st == h.OK, info
    assert info[1]["iterations"] == 0
    xs = h.unpack_field_to_host(lat, "fp64", x, nrhs)
    assert not np.any(xs[1])
    lat_o = O.lattice_from(w)
    res = [O.true_residual(lat_o, m, src[j], xs[j]) for j in (0, 2, 3)]
    assert max(res) <= 1e-10, res
    x.zero_()
    st, info = h.hisq_cg(lat, m, l64, lin, "fp32", nrhs, b, x, 1e-10, 5, ws)
    assert st == h.NOT_CONVERGED
    assert [i["iterations"] for i in info] == [5, 0, 5, 5]


def test_repeated_solves_on_the_same_buffers(gpu_lib):
    """Solves repeated on the same buffers reuse the captured iteration
    graphs when every launch value repeats, and capture new ones when one
    changes (here the mass, the inner precision's links and the column
    count): each solve must still meet the oracle's FP64 true residual."""
    h = gpu_lib
    w = gen.workload_haar((8, 8, 4, 8), 47, -1, 2)
    lat = h.lattice(w["dims"], w["t_bc"])
    l64 = h.pack_links_from_host(lat, "fp64", w["fat"], w["naik"])
    l32 = h.pack_links_from_host(lat, "fp32", w["fat"], w["naik"])
    b = h.pack_field_from_host(lat, "fp64", w["src"])
    x = h.empty_field(lat, "fp64", 2)
    ws = h.empty_workspace(h.hisq_cg_workspace_bytes(lat, "fp32", 2, 0))
    for mass, nrhs, tol in ((0.1, 2, 1e-10), (0.1, 2, 1e-10), (0.2, 2, 1e-10), (0.1, 1, 1e-9), (0.1, 2, 1e-11)):
        x.zero_()
        st, info = h.hisq_cg(lat, mass, l64, l32, "fp32", nrhs, b, x, tol, 20000, ws)
        assert st == h.OK, (mass, nrhs, tol, info)
        res, _ = oracle_residuals(h, w, lat, x, nrhs, mass, w["src"][:nrhs])
        assert max(res) <= tol, (mass, nrhs, tol, res)


@pytest.mark.parametrize("inner,nrhs", [("fp32", 2), ("fp32", 3)])
@pytest.mark.parametrize("iters", [1, 2, 5, 6])
def test_stop_after_odd_and_even_updates(gpu_lib, inner, nrhs, iters):
    """The two-launch step moves x every second iteration: stopped at the
    iteration limit after an odd and an even number, x has every term.  It is
    the oracle's iterate to the FP32 rounding of a few operator applications
    (each below 100 eps = 1.2e-5 of its result); the last term is far larger."""
    h = gpu_lib
    w = gen.workload_haar((6, 4, 8, 10), 48, -1, nrhs)
    lat, l64, lin, b, x, ws = setup(h, w, inner, nrhs)
    st, info = h.hisq_cg(lat, 0.5, l64, lin, inner, nrhs, b, x, 1e-12, iters, ws)
    assert st == h.NOT_CONVERGED and [i["iterations"] for i in info] == [iters] * nrhs
    _, xs = oracle_residuals(h, w, lat, x, nrhs, 0.5, w["src"])
    for j in range(nrhs):
        ref = O.cg(O.lattice_from(w), 0.5, w["src"][j], 1e-12, iters).x
        before = O.cg(O.lattice_from(w), 0.5, w["src"][j], 1e-12, iters - 1).x if iters > 1 else 0 * ref
        assert O.norm(ref - before) > 1e-2 * O.norm(ref)
        assert O.norm(xs[j] - ref) <= 1e-4 * O.norm(ref)


# Four sites a block: 4096 partial sums a column on 16^3 x 8, more than the fused
# step takes (2048), so these solves run the two-launch step as large lattices do.
UNFUSED, UNFUSED_DIMS = (3, 1, 64, 1), (16, 16, 16, 8)


def unfused(h, w, inner, nrhs, src=None):
    lat, l64, lin, b, x, ws = setup(h, w, inner, nrhs, src=src)
    ctx = h.Context(0)
    for prec in {inner, "fp64"}:
        h.hisq_set_dslash_shape(lat, prec, nrhs, UNFUSED, ctx)
    return lat, l64, lin, b, x, ws, ctx


@pytest.fixture(scope="module")
def unfused_workload():
    return gen.workload_haar(UNFUSED_DIMS, 49, -1, 4)


@pytest.fixture(scope="module")
def unfused_iterates(unfused_workload):
    """The oracle's CG iterates 0 .. 6 for m = 0.5, column by column."""
    w = unfused_workload
    lat = O.lattice_from(w)
    zero = np.zeros_like(w["src"][0])
    return [[zero] + [O.cg(lat, 0.5, w["src"][j], 1e-14, k).x for k in range(1, 7)] for j in range(2)]


@pytest.mark.parametrize("inner,nrhs", [("fp64", 1), ("fp64", 2), ("fp32", 1), ("fp32", 2)])
@pytest.mark.parametrize("iters", [1, 2, 5, 6])
def test_two_launch_step_stops_after_odd_and_even_updates(gpu_lib, unfused_workload, unfused_iterates, inner, nrhs, iters):
    """As above for one column a block and for column pairs of the two-launch
    step: the oracle's iterate to the rounding of a few operator applications
    (FP32: each below 100 eps = 1.2e-5 of its result; FP64: 1e-12)."""
    h = gpu_lib
    w = unfused_workload
    lat, l64, lin, b, x, ws, ctx = unfused(h, w, inner, nrhs)
    st, info = h.hisq_cg(lat, 0.5, l64, lin, inner, nrhs, b, x, 1e-14, iters, ws, ctx=ctx)
    assert st == h.NOT_CONVERGED and [i["iterations"] for i in info] == [iters] * nrhs
    xs = h.unpack_field_to_host(lat, "fp64", x, nrhs)
    for j in range(nrhs):
        ref, before = unfused_iterates[j][iters], unfused_iterates[j][iters - 1]
        assert O.norm(ref - before) > 1e-2 * O.norm(ref)
        assert O.norm(xs[j] - ref) <= (1e-12 if inner == "fp64" else 1e-4) * O.norm(ref)


@pytest.mark.parametrize("inner", ["fp64", "fp32"])
def test_two_launch_step_columns_stop_apart(gpu_lib, unfused_workload, unfused_iterates, inner):
    """Columns that start from different iterates stop after different numbers
    of updates, odd and even, while others go on: each converges to the
    tolerance by the oracle.  In FP64 the recurrence's residual is the true one
    to far less than the tolerance, so no column needs its residual replaced: a
    term of x left out at a stop would show as one."""
    h = gpu_lib
    w = unfused_workload
    start = ((0, 0), (0, 3), (1, 2), (1, 6), (0, 5), (1, 4))
    nrhs, m, tol = len(start), 0.5, 1e-9
    src = w["src"][[j for j, _ in start]]
    lat, l64, lin, b, x, ws, ctx = unfused(h, w, inner, nrhs, src=src)
    x.copy_(h.pack_field_from_host(lat, "fp64", np.stack([unfused_iterates[j][k] for j, k in start])))
    st, info = h.hisq_cg(lat, m, l64, lin, inner, nrhs, b, x, tol, 5000, ws, ctx=ctx)
    assert st == h.OK, info
    stops = [i["iterations"] for i in info]
    print(f"\n{inner}: stopped after {stops}")
    assert len(set(stops)) > 1
    if inner == "fp64":
        assert {n % 2 for n in stops} == {0, 1} and not any(i["reliable_updates"] for i in info)
    res, _ = oracle_residuals(h, w, lat, x, nrhs, m, src)
    assert max(res) <= tol, res


@pytest.mark.parametrize("inner", ["fp64", "fp32", "fp32r12"])
def test_two_launch_step_single_column_solve(gpu_lib, inner):
    """One column: a reliable-update solve (FP64: a plain one) to the tolerance, in
    the step that a 48^3 x 12 lattice takes."""
    h = gpu_lib
    w = gen.workload_smooth(UNFUSED_DIMS, 50, -1, 0.3, 1)
    lat, l64, lin, b, x, ws, ctx = unfused(h, w, inner, 1)
    st, info = h.hisq_cg(lat, 0.05, l64, lin, inner, 1, b, x, 1e-10, 20000, ws, ctx=ctx)
    assert st == h.OK, info
    res, _ = oracle_residuals(h, w, lat, x, 1, 0.05, w["src"])
    assert res[0] <= 1e-10
    assert inner == "fp64" or info[0]["reliable_updates"] >= 1
