"""Host-side checks of libcerar that need no GPU: the library loads and
exports every function include/cerar.h declares; the fp64 plan builder agrees
with the oracle's constructions and closed forms; argument validation and
step ordering fail with the documented status; the ownership table of the
handoff ring is consistent."""

import ctypes
import os
import re
import subprocess

import numpy as np
import pytest

from conftest import ROOT
from oracle import plan as P
from oracle import ring as RG
from paper_2609_23898_amd import cerar as C
from paper_2609_23898_amd import synth

HEADER = os.path.join(ROOT, "include", "cerar.h")


def header_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(cerar_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_function():
    names = header_functions()
    assert len(names) == 22
    lib = C.lib()
    for n in names:
        assert hasattr(lib, n), n
        assert n in C.SIGNATURES, f"binding does not declare {n}"
    out = subprocess.run(["nm", "-D", "--defined-only", C.LIB_PATH], capture_output=True, text=True).stdout
    exported = set(re.findall(r"\bT (cerar_[a-z0-9_]+)", out))
    assert set(names) <= exported, set(names) - exported


def test_struct_layouts_match_header():
    """The ctypes mirrors have the header's field order."""
    text = open(HEADER).read()
    body = lambda name: re.search(r"typedef struct \{((?:(?!typedef).)*?)\} " + name + ";", text, re.S).group(1)
    desc, info = body("cerar_plan_desc"), body("cerar_plan_info")
    strip = lambda s: re.sub(r"/\*.*?\*/", "", s, flags=re.S)
    fields = lambda s: re.findall(r"([A-Za-z_][A-Za-z0-9_]*)\s*(?=[,;])", strip(s))
    assert fields(desc) == [f for f, _ in C.PlanDesc._fields_]
    assert fields(info) == [f for f, _ in C.PlanInfo._fields_]


# --- plan builder vs the oracle -------------------------------------------------

def oracle_mpc(N, c, kind, param, B=None):
    xi = P.chebyshev_nodes(c)
    if kind == "vandermonde":
        B, D = P.vandermonde_base(N, param, xi)
    else:
        D = P.o_eps_perturbation(np.diag(xi), param)
    U, R = P.mpc_plan(B, D)
    return U, R, D


@pytest.mark.parametrize("N,c,kind,param", [
    (4, 4, "vandermonde", 0.5), (3, 5, "vandermonde", 0.3), (4, 5, "o_eps", 0.1),
    (8, 16, "o_eps", 1e-3), (2, 9, "o_eps", 0.2), (4, 4, "o_eps", 0.0), (8, 8, "o_eps", 0.0)])
def test_mpc_plans_match_oracle(N, c, kind, param):
    B = synth.base_matrix(7, N, c)
    plan = C.Plan(N, c, kind, param, base=None if kind == "vandermonde" else B)
    U, R = plan.matrices()
    Uo, Ro, D = oracle_mpc(N, c, kind, param, B)
    info = plan.info()
    # inverse of A_l loses ~kappa * u64 relative accuracy
    tol = 1e-13 * max(1.0, info["kappa_U"])
    np.testing.assert_allclose(U, Uo, rtol=0, atol=tol * np.abs(Uo).max())
    np.testing.assert_allclose(R, Ro, rtol=0, atol=1e-13 * np.abs(Ro).max())
    assert info["L"] == c + N - 2 and info["r_star"] == P.r_star(N, c)
    assert info["comm_rate"] == pytest.approx(1 + (N - 2) / c)
    assert info["storage_rate"] == pytest.approx(1 + N / c)
    assert info["phi_closed_form"] == pytest.approx(P.phi_mpc_closed_form(N, D), rel=1e-10, abs=1e-25)
    assert info["phi"] == pytest.approx(P.phi(Uo, Ro), rel=1e-6, abs=1e-12)
    assert info["kappa_M"] == pytest.approx(P.max_kappa_M(Uo), rel=1e-6)
    assert info["kappa_U"] == pytest.approx(max(P.kappa2(u) for u in Uo), rel=1e-6)
    assert info["kappa_R"] == pytest.approx(max(P.kappa2(r) for r in Ro), rel=1e-6)
    if kind == "vandermonde":
        assert info["phi_closed_form"] == pytest.approx(P.phi_vandermonde_closed_form(N, param, P.chebyshev_nodes(c)), rel=1e-12)


@pytest.mark.parametrize("N,c,eps", [(8, 16, 0.1), (4, 10, 0.1), (4, 8, 0.05), (3, 7, 0.2)])
def test_node_permutation_choice_matches_oracle(N, c, eps):
    """With candidate node permutations the library takes the H of the
    largest gamma (Sec. II-C assumption) and builds the same plan as the
    oracle from that H; without them it reports gamma of diag(nodes)."""
    B = synth.base_matrix(5, N, c)
    perms = synth.node_permutations(9, 24, c)
    xi = P.chebyshev_nodes(c)
    plain = C.Plan(N, c, "o_eps", eps, base=B).info()
    assert plain["h_choice"] == -1
    assert plain["gamma"] == pytest.approx(P.gamma(B, np.diag(xi)), rel=1e-9)
    plan = C.Plan(N, c, "o_eps", eps, base=B, node_perms=perms)
    info = plan.info()
    t, g = P.select_node_permutation(B, xi, perms)
    assert info["h_choice"] == t and info["gamma"] == pytest.approx(g, rel=1e-9)
    assert info["gamma"] >= plain["gamma"] * (1 - 1e-12)          # the identity is candidate 0
    D = P.o_eps_perturbation(np.diag(xi[perms[t]]), eps)
    Uo, Ro = P.mpc_plan(B, D)
    U, R = plan.matrices()
    np.testing.assert_allclose(U, Uo, rtol=0, atol=1e-13 * max(1.0, info["kappa_U"]) * np.abs(Uo).max())
    np.testing.assert_allclose(R, Ro, rtol=0, atol=1e-13 * np.abs(Ro).max())
    assert info["phi"] == pytest.approx(plain["phi"], rel=1e-8)      # same node set, same Phi
    assert info["kappa_M"] == pytest.approx(P.max_kappa_M(Uo), rel=1e-6)


def test_node_permutations_start_the_kappa_design():
    """The KAPPA design starts from the O(eps0) plan of the chosen H."""
    N, c = 4, 9
    B = synth.base_matrix(13, N, c)
    perms = synth.node_permutations(2, 16, c)
    xi = P.chebyshev_nodes(c)
    t, _ = P.select_node_permutation(B, xi, perms)
    plan = C.Plan(N, c, "kappa", 1e3, base=B, eps0=0.3, als_iters=6, als_order=1, node_perms=perms)
    assert plan.info()["h_choice"] == t
    Uo, Ro = P.kappa_design(B, np.diag(xi[perms[t]]), 0.3, 1e3, 6, order="projected")
    U, R = plan.matrices()
    np.testing.assert_allclose(U, Uo, rtol=0, atol=1e-7 * np.abs(Uo).max())
    np.testing.assert_allclose(R, Ro, rtol=0, atol=1e-7 * np.abs(Ro).max())


def test_invalid_node_permutations():
    B = synth.base_matrix(1, 4, 6)
    good = synth.node_permutations(1, 3, 6)
    bad = good.copy()
    bad[1, 0] = bad[1, 1]                                          # a repeated index
    cases = [dict(kind="o_eps", param=0.1, node_perms=bad),
             dict(kind="o_eps", param=0.1, node_perms=good, perturb=np.eye(6)),
             dict(kind="vandermonde", param=0.3, node_perms=good),
             dict(kind="o_eps", param=0.1, node_perms=np.zeros((4097, 6), dtype=np.int32) + np.arange(6))]
    for kw in cases:
        with pytest.raises(C.CerarError) as ei:
            C.Plan(4, 6, base=None if kw["kind"] == "vandermonde" else B, **kw)
        assert ei.value.status == -1


def test_exact_plan_phi_zero():
    plan = C.Plan(4, 4, "o_eps", 0.0, base=synth.base_matrix(3, 4, 4))
    assert plan.info()["phi"] < 1e-20


@pytest.mark.parametrize("N,c,iters", [(4, 6, 8), (4, 9, 15), (8, 16, 10)])
@pytest.mark.parametrize("order", [0, 1])
def test_kappa_design_matches_oracle_iterates(N, c, iters, order):
    """Same steps (U-step, R-step, projection in either order) from the same
    start give the same iterates in both implementations; kappa_2(M_i) <=
    kappa_max holds."""
    B = synth.base_matrix(11, N, c)
    kmax = 1e3
    plan = C.Plan(N, c, "kappa", kmax, base=B, eps0=0.3, als_iters=iters, als_order=order)
    U, R = plan.matrices()
    Uo, Ro = P.kappa_design(B, np.diag(P.chebyshev_nodes(c)), 0.3, kmax, iters,
                            order="paper" if order == 0 else "projected")
    np.testing.assert_allclose(U, Uo, rtol=0, atol=1e-7 * np.abs(Uo).max())
    np.testing.assert_allclose(R, Ro, rtol=0, atol=1e-7 * np.abs(Ro).max())
    info = plan.info()
    assert info["kappa_M"] <= kmax * (1 + 1e-9)
    assert info["phi"] == pytest.approx(P.phi(Uo, Ro), rel=1e-6)
    assert np.sqrt(N) * info["proj_b0"] / info["proj_a0"] == pytest.approx(kmax)
    assert np.isnan(info["phi_closed_form"])


def test_seeded_plan_is_deterministic_and_gaussian_like():
    a = C.Plan(8, 16, "o_eps", 0.1, seed=42)
    b = C.Plan(8, 16, "o_eps", 0.1, seed=42)
    np.testing.assert_array_equal(a.matrices()[0], b.matrices()[0])
    assert a.info()["seed_used"] == 42
    c = C.Plan(8, 16, "o_eps", 0.1, seed=43)
    assert not np.array_equal(a.matrices()[0], c.matrices()[0])


def test_plan_save_and_load(tmp_path):
    plan = C.Plan(8, 32, "kappa", 1e3, seed=5, als_iters=5, als_order=1)
    path = tmp_path / "plan.npz"
    plan.save(path)
    again = C.Plan.load(path)
    U, R = plan.matrices()
    U2, R2 = again.matrices()
    np.testing.assert_array_equal(U, U2)
    np.testing.assert_array_equal(R, R2)
    assert again.info()["phi"] == pytest.approx(plan.info()["phi"], rel=1e-12)
    assert again.info()["kappa_M"] == pytest.approx(plan.info()["kappa_M"], rel=1e-9)


def test_explicit_plan_roundtrip():
    rng = np.random.default_rng(0)
    N, c = 3, 5
    U = rng.standard_normal((N, c, c))
    R = rng.standard_normal((N, c + N - 1, c))
    plan = C.Plan.explicit(U, R)
    U2, R2 = plan.matrices()
    np.testing.assert_array_equal(U, U2)
    np.testing.assert_array_equal(R, R2)
    assert plan.info()["phi"] == pytest.approx(P.phi(U, R), rel=1e-12)


# --- validation and status codes ----------------------------------------------------

@pytest.mark.parametrize("args", [
    (1, 4, "o_eps", 0.1), (65, 65, "o_eps", 0.1), (4, 3, "o_eps", 0.1), (4, 129, "o_eps", 0.1),
    (4, 5, "vandermonde", 0.0), (4, 5, "vandermonde", -1.0), (4, 5, "o_eps", -0.1),
    (4, 5, "o_eps", 1.5), (4, 5, "kappa", 1.9), (4, 5, "o_eps", float("nan"))])
def test_invalid_plan_arguments(args):
    with pytest.raises(C.CerarError) as ei:
        C.Plan(*args)
    assert ei.value.status == -1


def test_invalid_als_order():
    with pytest.raises(C.CerarError) as ei:
        C.Plan(4, 5, "kappa", 1e3, seed=1, als_order=2)
    assert ei.value.status == -1


def test_singular_construction_reported():
    """c > N with D = I repeats rows of A_l (the mechanism of Lemma 1)."""
    with pytest.raises(C.CerarError) as ei:
        C.Plan(4, 6, "o_eps", 0.0, base=synth.base_matrix(1, 4, 6))
    assert ei.value.status == -3
    with pytest.raises(C.CerarError) as ei:
        C.Plan(4, 6, "o_eps", 0.0, seed=5)
    assert ei.value.status == -3


def test_device_calls_validate_before_touching_the_device():
    plan = C.Plan(4, 4, "o_eps", 0.1, seed=1)
    lib = C.lib()
    fake = ctypes.c_void_p(0x100000)
    ws = ctypes.c_void_p(0x200000)
    # ld_work < c * p
    assert lib.cerar_encode_round(plan.handle, 0, 4096, fake, 4096, fake, 100, ws, None) == -1
    # NULL grads
    assert lib.cerar_encode_round(plan.handle, 0, 4096, None, 4096, ctypes.c_void_p(0x300000), 4096, ws, None) == -1
    # grads and work overlapping without being equal
    assert lib.cerar_encode_round(plan.handle, 0, 4096, fake, 4096, ctypes.c_void_p(0x100000 + 64), 4096, ws,
                                  None) == -1
    # work overlapping ws, grads overlapping ws
    assert lib.cerar_encode_round(plan.handle, 0, 4096, fake, 4096, fake, 4096, ctypes.c_void_p(0x100000 + 256),
                                  None) == -1
    assert b"work and ws overlap" in lib.cerar_last_error()
    assert lib.cerar_encode_round(plan.handle, 0, 4096, ctypes.c_void_p(0x5000000), 4096, fake, 4096,
                                  ctypes.c_void_p(0x5000000 + 512), None) == -1
    assert b"grads and ws overlap" in lib.cerar_last_error()
    # step out of range and out of order
    assert lib.cerar_encode_round(plan.handle, 7, 4096, fake, 4096, fake, 4096, ws, None) == -1
    assert lib.cerar_encode_round(plan.handle, 3, 4096, fake, 4096, fake, 4096, ws, None) == -6
    assert b"out of order" in lib.cerar_last_error()
    # decode before the rounds
    out = ctypes.c_void_p(0x900000000)
    assert lib.cerar_decode(plan.handle, 4096, fake, 4096, ws, out, 4096, None) == -6
    # out overlapping work
    assert lib.cerar_decode(plan.handle, 4096, fake, 4096, ws, ctypes.c_void_p(0x100000 + 4), 4096, None) == -1
    # d == 0
    assert lib.cerar_ring_simulate(plan.handle, 0, fake, 1, fake, 1, ws, out, 1, None) == -1
    assert lib.cerar_error_norms(0, 10, fake, 10, out, 10, ws, None) == -1
    assert lib.cerar_copy_f32(None, fake, 10, None) == -1
    assert lib.cerar_plan_prepare_device(None) == -1
    # overlapping buckets
    offs = (ctypes.c_size_t * 2)(0, 100)
    lens = (ctypes.c_size_t * 2)(200, 200)
    assert lib.cerar_ring_simulate_bucketed(plan.handle, 2, offs, lens, fake, 1000, ctypes.c_void_p(0x40000000),
                                            1 << 20, ws, out, 1000, None) == -1
    assert b"overlap" in lib.cerar_last_error()
    # bucketed: work overlapping ws, grads overlapping ws
    offs = (ctypes.c_size_t * 2)(0, 200)
    bwork = 0x40000000
    assert lib.cerar_ring_simulate_bucketed(plan.handle, 2, offs, lens, fake, 1000, ctypes.c_void_p(bwork),
                                            1 << 20, ctypes.c_void_p(bwork + 1024), out, 1000, None) == -1
    assert b"work and ws overlap" in lib.cerar_last_error()
    assert lib.cerar_ring_simulate_bucketed(plan.handle, 2, offs, lens, ctypes.c_void_p(0x5000000), 1000,
                                            ctypes.c_void_p(bwork), 1 << 20, ctypes.c_void_p(0x5000000 + 512),
                                            out, 1000, None) == -1
    assert b"grads and ws overlap" in lib.cerar_last_error()


def test_chunk_len_and_workspace():
    plan = C.Plan(8, 64, "o_eps", 0.3, seed=2)
    for d in (1, 63, 64, 65, 1000, 1_414_647_808):
        p, stride = plan.chunk_len(d)
        assert p == RG.chunk_len(d, 64, 32) and stride % 64 == 0 and p <= stride < p + 64
        assert plan.workspace_bytes(d) == 8 * 8 * stride * 4


# --- ownership table of the handoff ring ----------------------------------------------

@pytest.mark.parametrize("N,c", [(2, 2), (2, 5), (3, 3), (4, 5), (4, 4), (8, 16), (8, 64), (16, 128)])
def test_slot_map_handoffs(N, c):
    plan = C.Plan(N, c, "o_eps", 0.3 if c > N else 0.0, seed=3)
    L = c + N - 2
    maps = [plan.slot_map(k) for k in range(L + 1)]
    nslots = N * c + N * N
    for k, m in enumerate(maps):
        live = m[m >= 0]
        assert live.max() < nslots
        assert len(set(live.tolist())) == live.size, f"two logical buffers share a slot after step {k}"
    m0 = maps[0]
    for i in range(N):
        np.testing.assert_array_equal(m0[i, :c], i * c + np.arange(c))      # in-place encode
        assert m0[i, c + N - 1] >= N * c                                     # x_{i,1} in the pool
    for k in range(1, L + 1):
        prev, cur = maps[k - 1], maps[k]
        for i in range(N):
            sent = prev[(i - 1) % N, c + N - 1]                              # slot of x_{i-1,k}
            if k <= N - 1:
                assert cur[i, c + k - 1] == sent                             # B_{i,k} <- x_{i-1,k}
            else:
                j = k - N + 1
                assert cur[i, j - 1] == sent                                 # D_{i,j} <- x_{i-1,k}
                if k < L:
                    assert cur[i, c + N - 1] == prev[i, j - 1]               # next send reuses delta_{i,j}
            if k == L:
                assert cur[i, c + N - 1] == -1
    # per-worker storage: c + (N-1) + 1 slots of length p (storage rate 1 + N/c)
    used = {s for m in maps for s in m[m >= 0].ravel().tolist()}
    assert len(used) <= nslots
    pool_used = {s for s in used if s >= N * c}
    assert len(pool_used) == N * N


def test_binding_refuses_host_tensors():
    """The Python binding passes raw pointers to kernels, so it refuses
    tensors outside device memory before any library call."""
    import torch
    plan = C.Plan(4, 4, "o_eps", 0.1, seed=1)
    d = 100
    work_floats = plan.c * plan.chunk_len(d)[0]
    g = torch.zeros((4, d))
    w = torch.zeros((4, work_floats))
    ws = torch.zeros(plan.workspace_bytes(d), dtype=torch.uint8)
    out = torch.zeros((4, d))
    for call in (lambda: C.ring_simulate(plan, d, g, w, ws, out),
                 lambda: C.encode_round(plan, 0, d, g, w, ws),
                 lambda: C.decode(plan, d, w, ws, out),
                 lambda: C.ring_simulate_fused(plan, d, g, out),
                 lambda: C.ring_simulate_bucketed(plan, [(0, d)], g, w, ws, out),
                 lambda: C.error_norms(4, d, g, out, torch.zeros(5, dtype=torch.float64)),
                 lambda: C.copy_f32(out, g)):
        with pytest.raises(ValueError, match="must be a tensor on the GPU"):
            call()


def test_jacobi_sweep_cap_is_reported():
    """One-sided Jacobi that stops at its sweep cap is never silent: the
    kappa design fails with E_NOCONV (its kappa bound rests on the
    projection's SVDs, Sec. II-D), and every other plan reports
    svd_converged = 0 (its kappa and gamma figures are then approximate)."""
    ok = C.Plan(8, 32, "o_eps", 0.1, seed=3)
    assert ok.info()["svd_converged"] == 1
    capped = C.Plan(8, 32, "o_eps", 0.1, seed=3, svd_sweeps=1)
    assert capped.info()["svd_converged"] == 0
    U, R = ok.matrices()
    np.testing.assert_array_equal(capped.matrices()[0], U)      # the plan itself does not depend on the SVDs
    with pytest.raises(C.CerarError) as ei:
        C.Plan(8, 32, "kappa", 1e3, seed=3, als_iters=2, svd_sweeps=1)
    assert ei.value.status == -4 and "did not converge" in str(ei.value)
    assert C.Plan(8, 32, "kappa", 1e3, seed=3, als_iters=2).info()["svd_converged"] == 1
    with pytest.raises(C.CerarError) as ei:
        C.Plan(8, 32, "o_eps", 0.1, seed=3, svd_sweeps=-1)
    assert ei.value.status == -1


@pytest.mark.parametrize("N,c,kind,param", [(4, 4, "vandermonde", 0.5), (4, 8, "vandermonde", 0.125),
                                            (8, 16, "o_eps", 1e-3), (8, 64, "kappa", 1e3),
                                            (16, 128, "o_eps", 1e-2)])
def test_default_sweep_cap_suffices_for_the_workload_plans(N, c, kind, param):
    """The workloads' plans (and the ill-conditioned ones among them) get
    converged SVDs at the default cap."""
    kw = {"als_iters": 3} if kind == "kappa" else {}
    plan = C.Plan(N, c, kind, param, seed=1000 + N, **kw)
    assert plan.info()["svd_converged"] == 1


def test_als_restarts_keep_the_least_phi():
    """KAPPA restarts (Sec. II-D: the problem is nonconvex): runs from the
    O(eps0) plans of bases of seeds seed, seed + 8, ...; the kept plan has the
    least Phi of them and still meets the kappa bound.  Each run equals a
    plain plan of that seed."""
    N, c, kmax, it = 4, 12, 60.0, 8
    runs = [C.Plan(N, c, "kappa", kmax, seed=5 + 8 * r, als_iters=it, als_order=1) for r in range(3)]
    phis = [pl.info()["phi"] for pl in runs]
    best = C.Plan(N, c, "kappa", kmax, seed=5, als_iters=it, als_order=1, als_restarts=3)
    info = best.info()
    r = int(np.argmin(phis))
    assert info["restart_used"] == r
    assert info["phi"] == pytest.approx(min(phis), rel=1e-12)
    np.testing.assert_array_equal(best.matrices()[0], runs[r].matrices()[0])
    assert info["kappa_M"] <= kmax * (1 + 1e-9)
    assert info["seed_used"] == runs[r].info()["seed_used"]
    assert runs[0].info()["restart_used"] == 0
    assert C.Plan(N, c, "o_eps", 0.1, seed=5).info()["restart_used"] == -1
    with pytest.raises(C.CerarError) as ei:                # restarts draw new bases
        C.Plan(N, c, "kappa", kmax, base=synth.base_matrix(1, N, c), als_restarts=2)
    assert ei.value.status == -1
    with pytest.raises(C.CerarError) as ei:
        C.Plan(N, c, "kappa", kmax, seed=5, als_restarts=65)
    assert ei.value.status == -1


@pytest.mark.parametrize("N", [2, 3, 4, 7, 8, 9, 16])
@pytest.mark.parametrize("extra", [0, 1, 2, 15, 50])
def test_observations_lie_where_the_one_pass_kernel_writes_them(N, extra):
    """Column k of Y_i after round L: message k + 1 of worker i - 1, in that
    worker's pool for k < N and in its chunk k - N after that; the last column
    is worker i's own last chunk.  The one slot per worker that is no
    observation is its chunk c - 2 (delta_{.,c-1})."""
    c = N + extra
    plan = C.Plan.explicit(np.stack([np.eye(c)] * N), np.zeros((N, c + N - 1, c)))
    sm, K, used = plan.slot_map(plan.L), c + N - 1, set()
    for i in range(N):
        pv = (i - 1) % N
        cols = [sm[i, c + j] for j in range(N - 1)] + [sm[i, j] for j in range(c)]
        assert cols == [N * c + pv * N + k if k < N else (pv * c + k - N if k < K - 1 else i * c + c - 1)
                        for k in range(K)]
        used |= set(cols)
    assert set(range(N * (c + N))) - used == {i * c + c - 2 for i in range(N)}
