"""The one-pass kernel behind ring_simulate, its no-alloc, bucketed and fused
forms, against the step calls: they run the same arithmetic in the same
order, so the outputs, every slot of `work` and every message slot of the
workspace must hold the same bits.  Shapes sit at the edges of its tiles (16
chunks, blocks of 64 or 32 positions), its rules (N = 8 | 9, c = 32 | 33 and
64 | 65) and its rows (any row start, odd lengths, pads of several chunks)."""

import ctypes

import numpy as np
import pytest

from paper_2609_23898_amd import cerar as C

from gpu_util import buffers, host_grads, orthogonal_plan, to_device, torch_dev

pytestmark = pytest.mark.gpu

SHAPES = [
    # N, c, d, row offset in floats (misaligned rows), extra row stride
    (2, 2, 2 * 64, 0, 0), (2, 3, 1, 0, 0), (2, 15, 15 * 96 + 1, 0, 0), (3, 16, 16 * 64, 0, 0),
    (4, 12, 12 * 4096 + 7, 1, 1), (5, 17, 17 * 130 - 3, 0, 3), (6, 31, 31 * 64 - 40, 0, 0), (7, 32, 32 * 95, 3, 2),
    (8, 8, 8 * 65, 0, 0), (8, 20, 20 * 640 + 13, 0, 0), (8, 32, 32 * 64 * 9 + 5, 0, 0), (8, 33, 33 * 97, 1, 0),
    (3, 47, 47 * 32 - 1, 0, 0), (8, 48, 48 * 160 - 65, 0, 1), (2, 49, 49 * 33, 0, 0), (4, 63, 63 * 64 + 2, 2, 0),
    (8, 64, 64 * 333 + 9, 0, 0), (7, 64, 64 * 64, 0, 0), (8, 64, 5, 0, 0),
    (9, 16, 16 * 97, 0, 0), (9, 9, 9 * 64 + 1, 0, 0), (13, 17, 17 * 64 - 5, 1, 1), (16, 16, 16 * 65, 0, 0),
    (16, 32, 32 * 321 - 7, 0, 0),
    # the rounds pass between the step calls' encode and decode
    (9, 33, 33 * 64, 0, 0), (8, 65, 65 * 64 - 1, 0, 0), (2, 128, 128 * 96, 1, 1), (12, 90, 90 * 97 - 3, 0, 0),
    (16, 128, 128 * 160 + 1, 0, 0), (13, 33, 7, 0, 0), (5, 80, 80 * 64 * 3, 3, 0), (17, 40, 40 * 64, 0, 0),
]


def _state(plan, d, work, ws):
    """All N (c + N) slots' p floats: the workers' chunks, then the messages."""
    torch, _ = torch_dev()
    p, stride = plan.chunk_len(d)
    pool = ws.view(torch.float32).view(plan.N * plan.N, stride)[:, :p]
    return work[:, :plan.c * p].clone(), pool.clone()


def _steps(plan, d, grads, work, ws, out):
    for k in range(plan.L + 1):
        C.encode_round(plan, k, d, grads, work, ws)
    C.decode(plan, d, work, ws, out)


@pytest.mark.parametrize("N,c,d,off,extra", SHAPES)
def test_one_pass_leaves_the_step_calls_bits(N, c, d, off, extra):
    torch, _ = torch_dev()
    U, R = orthogonal_plan(N, c, seed=N * 100 + c) if c > N else (
        np.stack([np.linalg.qr(np.random.default_rng(c + k).standard_normal((c, c)))[0] for k in range(N)]),
        np.random.default_rng(c).standard_normal((N, c + N - 1, c)))
    plan = C.Plan.explicit(U, R)
    p, _ = plan.chunk_len(d)
    grads = to_device(host_grads(N, d, seed=c + d), ld=d + extra, align_elems=off)
    got, want = (buffers(plan, d, ld_work=c * p + extra, ld_out=d + extra, work_offset=off, out_offset=off)
                 for _ in range(2))
    C.ring_simulate(plan, d, grads, *got)
    _steps(plan, d, grads, *want)
    torch.cuda.synchronize()
    assert torch.equal(got[2][:, :d], want[2][:, :d])
    assert bool(torch.isnan(got[2][:, d:]).all()) and bool(torch.isnan(got[0][:, c * p:]).all())
    for a, b in zip(_state(plan, d, got[0], got[1]), _state(plan, d, want[0], want[1])):
        assert torch.equal(a, b)
    again = got[2].clone()
    got[2].fill_(float("nan"))
    C.decode(plan, d, got[0], got[1], got[2])       # the observations decode again
    torch.cuda.synchronize()
    assert torch.equal(got[2][:, :d], again[:, :d])


# Several blocks for every workgroup of the launch: the loop with the next
# block's loads under way, LDS used again, and the XCD order of ragged rows.
LONG = [(2, 16, 110_000_000, 0), (4, 12, 40_000_007, 1), (8, 32, 34_000_000, 0), (8, 20, 21_000_001, 0), (3, 48, 9_000_000, 0),
        (8, 64, 3_000_000, 0), (8, 60, 3_000_001, 3), (16, 16, 4_800_000, 0), (9, 25, 7_500_003, 1), (12, 48, 2_000_000, 0),
        (16, 64, 2_000_000, 0), (16, 60, 2_000_001, 1), (4, 100, 90_000_000, 0), (16, 128, 25_000_000, 0), (7, 90, 30_000_001, 2)]


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("N,c,d,off", LONG)
def test_workgroups_with_many_blocks_leave_the_step_calls_bits(N, c, d, off, in_place):
    torch, dev = torch_dev()
    rng = np.random.default_rng(N * 1000 + c)
    U, R = rng.standard_normal((N, c, c)) / c ** 0.5, rng.standard_normal((N, c + N - 1, c)) / c
    plan = C.Plan.explicit(U, R)
    p, _ = plan.chunk_len(d)
    ld = c * p + off
    gen = torch.Generator(dev).manual_seed(c)
    g = torch.randn((N, d), dtype=torch.float32, device=dev, generator=gen)
    res = []
    for call in (lambda *b: C.ring_simulate(plan, d, *b), lambda *b: _steps(plan, d, *b)):
        work = torch.empty(N * ld + off, dtype=torch.float32, device=dev)[off:].view(N, ld)
        ws = torch.zeros(plan.workspace_bytes(d), dtype=torch.uint8, device=dev)
        out = torch.empty(N * (d + off) + off, dtype=torch.float32, device=dev)[off:].view(N, d + off)
        grads = torch.empty(N * ld + off, dtype=torch.float32, device=dev)[off:].view(N, ld)
        grads[:, :d] = g
        if in_place:
            work = grads
        call(grads, work, ws, out)
        torch.cuda.synchronize()
        res.append((out[:, :d], work[:, :c * p], ws))
    for a, b in zip(*res):
        assert all(torch.equal(x, y) for x, y in zip(a, b)) if a.dim() == 2 else torch.equal(a, b)


@pytest.mark.parametrize("N,c,d", [(4, 12, 12 * 320 + 5), (3, 33, 33 * 97), (8, 16, 16 * 640 + 1), (8, 48, 48 * 160 - 65),
                                   (8, 64, 64 * 333 + 9), (20, 32, 32 * 64 * 9 + 5), (18, 128, 128 * 96 - 1),
                                   (24, 70, 70 * 130 + 3)])
@pytest.mark.parametrize("off,extra", [(1, 1), (2, 2), (3, 4)])
def test_step_calls_on_rows_at_any_float(N, c, d, off, extra):
    """The same bits as on 16-byte aligned rows, in `out` and in every message
    round's slots, and nothing written beside the rows."""
    torch, _ = torch_dev()
    U, R = orthogonal_plan(N, c, seed=N + c)
    plan = C.Plan.explicit(U, R)
    p, _ = plan.chunk_len(d)
    host = host_grads(N, d, seed=c + d)
    got = buffers(plan, d, ld_work=c * p + extra, ld_out=d + extra, work_offset=off, out_offset=off)
    want = buffers(plan, d, ld_out=(d + 3) // 4 * 4)
    _steps(plan, d, to_device(host, ld=d + extra, align_elems=off), *got)
    _steps(plan, d, to_device(host, ld=(d + 3) // 4 * 4), *want)
    torch.cuda.synchronize()
    assert torch.equal(got[2][:, :d], want[2][:, :d])
    assert bool(torch.isnan(got[2][:, d:]).all()) and bool(torch.isnan(got[0][:, c * p:]).all())
    for a, b in zip(_state(plan, d, got[0], got[1]), _state(plan, d, want[0], want[1])):
        assert torch.equal(a, b)


@pytest.mark.parametrize("N,c,lens", [(8, 20, [20 * 64 * 5 + 3, 1, 20 * 63, 7777]), (3, 64, [64 * 33, 64 * 31 + 5]),
                                      (4, 12, [97 * (b + 1) for b in range(33)]),
                                      (8, 70, [70 * 64 + 1, 70 * 200, 9]), (16, 64, [64 * 96] * 3),
                                      (18, 32, [32 * 64 * 5 + 3, 1, 32 * 97]), (17, 24, [24 * 65, 7, 24 * 64 + 5]),
                                      (8, 64, [64 * 32 * 400, 64 * 32 * 300 + 5, 64 * 32 * 200 - 1, 70]),
                                      (16, 64, [64 * 32 * 300, 9, 64 * 32 * 350 + 1]), (2, 48, [48 * 32 * 2500, 48 * 32 * 1000 + 1]),
                                      (18, 64, [64 * 200 + 1, 9, 64 * 64]), (24, 63, [63 * 200 + 1, 9, 63 * 64]),
                                      (20, 48, [48 * 64 * 3 - 1, 48 * 65])])
def test_buckets_equal_calls_of_their_own(N, c, lens):
    """Odd offsets and lengths, more buckets than one launch takes: each bucket
    has the bits of its own call."""
    torch, dev = torch_dev()
    U, R = orthogonal_plan(N, c, seed=c)
    plan = C.Plan.explicit(U, R)
    offs = np.concatenate([[0], np.cumsum(lens)[:-1]]).tolist()
    d = sum(lens)
    grads = to_device(host_grads(N, d, seed=c))
    wf, wsb = plan.bucketed_sizes(lens)
    work = torch.full((N, wf), float("nan"), dtype=torch.float32, device=dev)
    ws = torch.zeros(wsb, dtype=torch.uint8, device=dev)
    out = torch.full((N, d), float("nan"), dtype=torch.float32, device=dev)
    C.ring_simulate_bucketed(plan, list(zip(offs, lens)), grads, work, ws, out)
    at = 0
    for o, n in zip(offs, lens):
        one = buffers(plan, n)
        C.ring_simulate(plan, n, grads[:, o:o + n], *one)
        torch.cuda.synchronize()
        cp = c * plan.chunk_len(n)[0]
        assert torch.equal(out[:, o:o + n], one[2]), (o, n)
        assert torch.equal(work[:, at:at + cp], one[0]), (o, n)
        at += cp


@pytest.mark.parametrize("seed", range(5))
def test_infinities_and_nan_stay_in_their_columns(seed):
    """A position whose gradients hold an infinity or NaN gives the step calls'
    results, and no other position sees it (zero padding of the tiles and the
    rows past K meets no such value)."""
    torch, _ = torch_dev()
    N, c = [(8, 20), (3, 33), (12, 48), (16, 64), (8, 80)][seed]
    d = c * 192 - 11
    U, R = orthogonal_plan(N, c, seed=5)
    plan = C.Plan.explicit(U, R)
    p, _ = plan.chunk_len(d)
    g = host_grads(N, d, seed=6)
    bad = [3, 70, 131]
    g[0, bad[0]], g[1, p + bad[1]], g[N - 1, (c - 2) * p + bad[2]] = np.inf, -np.inf, np.nan
    got, want = buffers(plan, d), buffers(plan, d)
    C.ring_simulate(plan, d, to_device(g), *got)
    _steps(plan, d, to_device(g), *want)
    torch.cuda.synchronize()
    a, b = got[2].cpu().numpy(), want[2].cpu().numpy()
    np.testing.assert_array_equal(a, b)
    clean = ~np.isin(np.arange(d) % p, bad)
    assert np.all(np.isfinite(a[:, clean]))


# Entries that three bf16 terms do not hold, alone and among others: below
# 2^-110 (subnormals of bf16 and of fp32 too), at the top of the range, and
# zeros, which they do hold.
MAGNITUDES = {"usual": (-20, 1), "small": (-148, -105), "few": (-20, 1), "large": (127, 128), "mixed": (-140, 128),
              "sparse": (-20, 1)}


def _entries(kind, shape, seed):
    rng = np.random.default_rng(seed)
    lo, hi = MAGNITUDES[kind]
    x = rng.choice([-1.0, 1.0], size=shape) * rng.uniform(1, 2, size=shape) * 2.0 ** rng.integers(lo, hi, size=shape)
    if kind == "few":                               # small ones among usual ones
        x = np.where(rng.random(shape) < 0.01, x * 2.0 ** -125, x)
    if kind == "sparse":
        x[rng.random(shape) < 0.9] = 0.0
    return np.clip(x, -np.finfo(np.float32).max, np.finfo(np.float32).max).astype(np.float32)


SPLIT_PLANS = [(9, 33), (12, 48), (16, 64), (20, 40), (17, 63), (3, 65), (8, 96), (5, 97), (16, 128)]


@pytest.mark.parametrize("kind", MAGNITUDES)
@pytest.mark.parametrize("N,c", SPLIT_PLANS)
def test_split_contractions_keep_every_fp32_entry(N, c, kind):
    """Encoders that permute the chunks and decoders that pick observations:
    every output is one input, whatever its magnitude, bit for bit."""
    torch, _ = torch_dev()
    rng = np.random.default_rng(N + c)
    K, d = c + N - 1, c * 96 - 37
    perm = [rng.permutation(c) for _ in range(N)]
    pick = [rng.integers(0, K, size=c) for _ in range(N)]
    U, R = np.zeros((N, c, c)), np.zeros((N, K, c))
    for i in range(N):
        U[i, perm[i], np.arange(c)] = 1.0
        R[i, pick[i], np.arange(c)] = 1.0
    plan = C.Plan.explicit(U, R)
    p, stride = plan.chunk_len(d)
    g = _entries(kind, (N, d), seed=c)
    grads = to_device(g)
    work, ws, out = buffers(plan, d)
    for k in range(plan.L + 1):
        C.encode_round(plan, k, d, grads, work, ws)
        if k == 0:
            chunks = work.cpu().numpy().reshape(N, c, p)
    G = np.zeros((N, c * p), np.float32)
    G[:, :d] = g
    for i in range(N):
        np.testing.assert_array_equal(chunks[i], G[i].reshape(c, p)[perm[i]])
    y = _entries(kind, (N * c + N * N, p), seed=c + 1)
    work.copy_(torch.from_numpy(y[:N * c].reshape(N, c * p)))
    ws.view(torch.float32).view(N * N, stride)[:, :p].copy_(torch.from_numpy(y[N * c:]))
    C.decode(plan, d, work, ws, out)
    slots = plan.slot_map(plan.L)
    cols = np.concatenate([slots[:, c:c + N - 1], slots[:, :c]], axis=1)       # Y_i = [B | D]
    for i in range(N):
        np.testing.assert_array_equal(out[i].cpu().numpy(), y[cols[i][pick[i]]].reshape(-1)[:d])


@pytest.mark.parametrize("scale", [2.0 ** -122, 2.0 ** 127])
@pytest.mark.parametrize("N,c", [(12, 48), (3, 65), (16, 128)])
def test_split_contractions_keep_every_fp32_coefficient(N, c, scale):
    """Coefficients beyond the split's range: one product per output, so within
    one rounding of it."""
    rng = np.random.default_rng(c)
    d = c * 64
    coef = (rng.uniform(1, 1.99, size=(N, c)) * scale).astype(np.float32).astype(np.float64)
    U = np.stack([np.diag(coef[i]) for i in range(N)])
    plan = C.Plan.explicit(U, np.zeros((N, c + N - 1, c)))
    g = (_entries("usual", (N, d), seed=c) * (1.0 / scale)).astype(np.float32)
    work, ws, _ = buffers(plan, d)
    C.encode_round(plan, 0, d, to_device(g), work, ws)
    want = np.repeat(coef, d // c, axis=1) * g.astype(np.float64)
    np.testing.assert_allclose(work.double().cpu().numpy(), want, rtol=2.0 ** -24, atol=0)


@pytest.mark.parametrize("N,c", [(12, 48), (3, 65), (16, 128)])
def test_small_entries_are_not_scaled_under_large_coefficients(N, c):
    """Sums of scaled entries would overflow under coefficients of 2^100."""
    rng = np.random.default_rng(c)
    d = c * 64
    coef = (rng.uniform(1, 1.99, size=(N, c)) * 2.0 ** 100).astype(np.float32).astype(np.float64)
    plan = C.Plan.explicit(np.stack([np.diag(coef[i]) for i in range(N)]), np.zeros((N, c + N - 1, c)))
    g = _entries("few", (N, d), seed=c)
    work, ws, _ = buffers(plan, d)
    C.encode_round(plan, 0, d, to_device(g), work, ws)
    want = np.repeat(coef, d // c, axis=1) * g.astype(np.float64)
    np.testing.assert_allclose(work.double().cpu().numpy(), want, rtol=2.0 ** -22, atol=0)


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("N,c", [(9, 33), (12, 48), (16, 64), (8, 96), (16, 128)])
def test_one_pass_and_steps_agree_on_entries_beyond_the_split(N, c, in_place):
    """Half-blocks of every magnitude beside ordinary ones: the whole ring and
    the step calls take the same arithmetic for each."""
    torch, _ = torch_dev()
    U, R = orthogonal_plan(N, c, seed=c)
    plan = C.Plan.explicit(U, R)
    d = c * 32 * 37 - 5
    p, _ = plan.chunk_len(d)
    g = np.zeros((N, c * p), np.float32)
    g[:, :d] = _entries("usual", (N, d), seed=c)
    rng = np.random.default_rng(c)
    for kind in ("small", "few", "large", "mixed", "sparse"):
        for h in rng.choice(p // 32, size=4, replace=False):
            i, l = rng.integers(N), rng.integers(c - 2)
            at = l * p + 32 * h
            g[i, at:at + 32] = _entries(kind, 32, seed=int(h))
    g[0, 5], g[1, p + 70], g[N - 1, 2 * p + 200] = np.inf, -np.inf, np.nan
    res = []
    for call in (lambda *b: C.ring_simulate(plan, d, *b), lambda *b: _steps(plan, d, *b)):
        work, ws, out = buffers(plan, d)
        grads = to_device(g)
        if in_place:
            work = grads
        call(grads, work, ws, out)
        torch.cuda.synchronize()
        res.append([t.cpu().numpy() for t in (out, *_state(plan, d, work, ws))])
    for a, b in zip(*res):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("N,d,off", [(1, 1, 0), (2, 3, 1), (8, 1023, 0), (8, 4 * 256 * 3 + 2, 3), (9, 4097, 2),
                                     (16, 5000, 1), (17, 1025, 0), (64, 130, 0)])
def test_error_norms_at_its_edges(N, d, off):
    """Rows that start at any float, lengths around a thread's four entries and
    a workgroup's, worker counts around a grid row's: fp64 sums of d squares,
    within d units of fp64 rounding of each other in any order."""
    torch, dev = torch_dev()
    g, o = host_grads(N, d, seed=N + d), host_grads(N, d, seed=N + d + 1)
    norms = torch.full((N + 1,), float("nan"), dtype=torch.float64, device=dev)
    C.error_norms(N, d, to_device(g, ld=d + off, align_elems=off), to_device(o, ld=d + off, align_elems=off), norms)
    torch.cuda.synchronize()
    S = g.astype(np.float64).sum(axis=0)
    ref = [np.sum((o[i].astype(np.float64) - S) ** 2) for i in range(N)] + [np.sum(S * S)]
    np.testing.assert_allclose(norms.cpu().numpy(), ref, rtol=(d + 4 * N) * 2.0 ** -52)


def _sharing(how, N, d, s):
    """(grads, out) views of one allocation: out on grads itself, some floats
    ahead of or behind it, at another row stride, or in the columns beside it."""
    torch, dev = torch_dev()
    if how == "columns":
        both = torch.empty((N, 2 * d), dtype=torch.float32, device=dev)
        return both[:, :d], both[:, d:]
    flat = torch.empty(N * (d + s) + 2 * s, dtype=torch.float32, device=dev)
    at, stride = {"itself": (s, d), "ahead": (2 * s, d), "behind": (0, d), "stride": (s, d + s)}[how]
    return flat[s:].as_strided((N, d), (d, 1)), flat[at:].as_strided((N, d), (stride, 1))


@pytest.mark.parametrize("how,s", [("itself", 32), ("ahead", 96), ("ahead", 7), ("behind", 4096), ("stride", 320),
                                   ("columns", 0)])
@pytest.mark.parametrize("N,c", [(4, 12), (8, 64), (12, 48)])
def test_outputs_may_lie_on_the_gradients(N, c, how, s):
    """Whatever memory `out` shares with `grads`, the sums are those of buffers
    of their own, in the single, the no-alloc and the bucketed call."""
    torch, dev = torch_dev()
    U, R = orthogonal_plan(N, c, seed=N * c)
    plan = C.Plan.explicit(U, R)
    plan.prepare_device()
    d = c * 64 * 1500 - 3
    g = torch.randn((N, d), dtype=torch.float32, device=dev, generator=torch.Generator(dev).manual_seed(c))
    work, ws, want = buffers(plan, d)
    C.ring_simulate(plan, d, g, work, ws, want)
    for call in (lambda gr, out: C.ring_simulate(plan, d, gr, work, ws, out),
                 lambda gr, out: C.ring_simulate_noalloc(plan, d, gr, work, out)):
        grads, out = _sharing(how, N, d, s)
        grads.copy_(g)
        call(grads, out)
        torch.cuda.synchronize()
        assert torch.equal(out, want)
    lens = [d // 3 + 1, 5, d - d // 3 - 6]
    buckets = list(zip([0, lens[0], lens[0] + 5], lens))
    wf, wsb = plan.bucketed_sizes(lens)
    bwork, bws = torch.empty((N, wf), dtype=torch.float32, device=dev), torch.empty(wsb, dtype=torch.uint8, device=dev)
    C.ring_simulate_bucketed(plan, buckets, g, bwork, bws, want)
    grads, out = _sharing(how, N, d, s)
    grads.copy_(g)
    C.ring_simulate_bucketed(plan, buckets, grads, bwork, bws, out)
    torch.cuda.synchronize()
    assert torch.equal(out, want)


class _Dim3(ctypes.Structure):
    _fields_ = [(a, ctypes.c_uint32) for a in "xyz"]


class _KernelNode(ctypes.Structure):                # hipKernelNodeParams
    _fields_ = [("block", _Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", _Dim3),
                ("params", ctypes.c_void_p), ("lds", ctypes.c_uint32)]


def _launch_grids(call):
    """Workgroups of every kernel that call(stream) enqueues, from a stream
    capture that is never run."""
    torch, _ = torch_dev()
    hip = ctypes.CDLL(sorted(C._hip_runtimes())[0])
    s = torch.cuda.Stream()
    graph, n = ctypes.c_void_p(), ctypes.c_size_t()
    assert hip.hipStreamBeginCapture(ctypes.c_void_p(s.cuda_stream), 1) == 0     # thread-local mode
    try:
        call(s)
    finally:
        assert hip.hipStreamEndCapture(ctypes.c_void_p(s.cuda_stream), ctypes.byref(graph)) == 0
    grids = []
    try:
        assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
        nodes = (ctypes.c_void_p * n.value)()
        assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
        for q in nodes:
            node = _KernelNode()
            assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(q), ctypes.byref(node)) == 0
            grids.append(node.grid.x)
    finally:
        hip.hipGraphDestroy(graph)
    return grids


def test_launch_size_is_the_plans_own():
    """Every kernel's launch is sized by its own registers, whichever plan came
    first in the process: at N = 8 a CU holds three workgroups of the c = 16
    kernel (76 registers, 47 KB of LDS; sixteen sweeps of those) and one of the
    c = 64 kernel (229 registers)."""
    torch, dev = torch_dev()
    cus = torch.cuda.get_device_properties(dev).multi_processor_count
    grids = {}
    for c in (16, 64, 16):
        d = c * 64 * 14000
        plan = C.Plan.explicit(*orthogonal_plan(8, c, seed=c))
        plan.prepare_device()
        grads = torch.zeros((8, d), dtype=torch.float32, device=dev)
        out = torch.empty_like(grads)
        grids[c], = _launch_grids(lambda s: C.ring_simulate_fused(plan, d, grads, out, stream=s))
    assert grids == {16: 3 * 16 * cus, 64: cus}


@pytest.mark.parametrize("N,c", [(8, 64), (16, 48), (16, 128), (17, 32), (17, 40), (18, 64), (24, 63), (20, 48), (18, 80)])
def test_buckets_share_their_launches(N, c):
    """A call launches as often for thirty buckets as for three."""
    torch, dev = torch_dev()
    rng = np.random.default_rng(c)
    plan = C.Plan.explicit(rng.standard_normal((N, c, c)), rng.standard_normal((N, c + N - 1, c)))
    plan.prepare_device()
    counts = []
    for nb in (3, 30):
        lens = [c * 96 + 7] * nb
        grads = torch.zeros((N, sum(lens)), dtype=torch.float32, device=dev)
        wf, wsb = plan.bucketed_sizes(lens)
        work = torch.empty((N, wf), dtype=torch.float32, device=dev)
        ws, out = torch.empty(wsb, dtype=torch.uint8, device=dev), torch.empty_like(grads)
        buckets = [(b * lens[0], lens[0]) for b in range(nb)]
        counts.append(len(_launch_grids(lambda s: C.ring_simulate_bucketed(plan, buckets, grads, work, ws, out, stream=s))))
    assert counts[0] == counts[1]
