"""The all-reduces that are timed, from the smallest call to the largest that
still leaves room for three sets of buffers on one card.

Every case goes through the Python binding's public calls on tensors that
are already on the GPU.  `kind` names the call:

  ring     ring_simulate: encode, all rounds and decode in one call
  noalloc  ring_simulate_noalloc: the same without a caller workspace
  steps    encode_round for steps 0..L, then decode: one call per protocol step
  buckets  ring_simulate_bucketed: one all-reduce per DDP bucket, one call
  fused    ring_simulate_fused: gradients in, sums out, no work or workspace
  norms    error_norms: squared errors of N outputs against the exact sum

The calls that fill a caller's `work` buffer return it beside the outputs: it
then holds the observations from which cerar_decode can be called again.
"""

import functools
import random

import numpy as np
import torch

from paper_2609_23898_amd import cerar as C
from paper_2609_23898_amd import synth

KAPPA_MAX = 1e3                 # the bound of the repository's condition-constrained designs
UNIT_ROUNDOFF = 2.0 ** -24      # fp32
MIB25 = 6_553_600               # floats of a 25 MiB DDP bucket


def listed():
    return [
        # The smallest workload of bench.py: latency of one call on 4096 entries.
        {"name": "tiny N4 c4", "kind": "ring", "N": 4, "c": 4, "d": 4096},
        # One 25 MiB DDP bucket, through the call for code that cannot allocate.
        {"name": "bucket N8 c32 noalloc", "kind": "noalloc", "N": 8, "c": 32, "d": MIB25},
        # The paper's 4-GPU setting (N=4, c=12); odd length, so that the rows of (N, d)
        # tensors are not 16-byte aligned, and c is no multiple of 16.
        {"name": "odd N4 c12", "kind": "ring", "N": 4, "c": 12, "d": 48_000_007},
        # The paper's 8-GPU setting (N=8, c=20), a tenth of its length.
        {"name": "paper N8 c20", "kind": "ring", "N": 8, "c": 20, "d": 100_000_000},
        # The N=8, c=16, d=2^24 workload of bench.py: 4 MiB messages.
        {"name": "iid N8 c16", "kind": "ring", "N": 8, "c": 16, "d": 1 << 24},
        # GPT-2-small's gradient (bench.py's workload) as one instance.
        {"name": "gpt2 N8 c32", "kind": "ring", "N": 8, "c": 32, "d": 124_439_808},
        # The same gradient as its 17 DDP buckets.
        {"name": "gpt2 N8 c32 buckets", "kind": "buckets", "N": 8, "c": 32, "d": 124_439_808, "buckets": 0},
        # A quarter of the Pythia-1.4B gradient (one of four pipeline stages) at the
        # headline's N and c.
        {"name": "pythia/4 N8 c64", "kind": "ring", "N": 8, "c": 64, "d": 353_661_952},
        # The wide code of the heavy-tail workload, at a quarter of its length.
        {"name": "wide N16 c128", "kind": "ring", "N": 16, "c": 128, "d": 100_000_000},
        # A caller that drives the protocol step by step, as a rank of a real ring does.
        {"name": "steps N8 c64", "kind": "steps", "N": 8, "c": 64, "d": 64_000_000},
        # The single-GPU variant at the headline's N and c, a sixteenth of its length.
        {"name": "fused N8 c64", "kind": "fused", "N": 8, "c": 64, "d": 88_415_488},
        # The error report after an all-reduce of GPT-2-small's gradient.
        {"name": "norms N8", "kind": "norms", "N": 8, "c": 32, "d": 124_439_808},
    ]


def draw(rng):
    """One more all-reduce: any call, 2 to 16 workers, c from N to 128, lengths
    from 4096 entries per worker to 2^30 in all, spread over their logarithm."""
    kind = rng.choice(["ring"] * 6 + ["buckets"] * 2 + ["steps", "noalloc", "fused", "fused", "norms"])
    N = rng.choice([2, 3, 4, 5, 6, 7, 8, 8, 8, 12, 16])
    if kind == "fused":                                  # the shapes that call takes
        c = rng.choice([16, 32]) if N > 8 else rng.choice([16, 32, 48, 64])
        c = max(c, N)
    elif rng.random() < 0.5:
        c = 16 * rng.randint(1, 8)
        c = max(c, N)
    else:
        c = rng.randint(max(N, 4), 100)
    top = min(2.0 ** 30 / N, 3.5e8)
    if kind == "noalloc":                                # the static pool's limit
        top = min(top, c * (1 << 24) / (N * N) * 0.9)
    if kind == "steps":                                  # one host call per step
        top = min(top, 6.4e7)
    d = int(4096 * (top / 4096) ** rng.random())
    if kind == "fused" or rng.random() < 0.5:
        d = max(4, d // 4 * 4)                           # 16-byte aligned rows
    case = {"kind": kind, "N": N, "c": c, "d": d}
    if kind == "buckets":
        case["buckets"] = rng.randint(2, 40)
        case["unit"] = rng.choice([1, 256, 256])         # bucket lengths: any, or multiples of a tensor row
        case["d"] = max(d, case["buckets"] * 4096)
    return case


@functools.lru_cache(maxsize=None)
def plan_of(N, c):
    """A program designs its plan once, before training; so does this one."""
    if c <= N:                                           # the exact ring (c = N) has no design to search
        return C.Plan(N, c, "o_eps", 1e-3, seed=1000 + N)
    iters = 20 if c <= 64 else 4
    return C.Plan(N, c, "kappa", KAPPA_MAX, seed=1000 + N, eps0=0.3, als_iters=iters, als_order=1)


def bucket_list(case):
    if case["buckets"] == 0:
        return synth.ddp_buckets(synth.gpt2_small_tensor_sizes())
    r = random.Random(case["buckets"] * 1_000_003 + case["d"])
    unit = case["unit"]
    share = [0.25 + r.random() for _ in range(case["buckets"])]
    lens = [max(1, int(case["d"] * s / sum(share)) // unit) * unit for s in share]
    offs = np.concatenate([[0], np.cumsum(lens)[:-1]])
    return [(int(o), int(n)) for o, n in zip(offs, lens)]


def length(case):
    """Entries per worker: d, or the end of the last bucket."""
    if case["kind"] != "buckets":
        return case["d"]
    return max(o + n for o, n in bucket_list(case))


def gradients(case, seed):
    """Normal entries with a log-normal scale per tensor, shared by the workers."""
    N, d = case["N"], length(case)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    g = torch.randn((N, d), dtype=torch.float32, device="cuda", generator=gen)
    tensors = min(64, max(1, d // 1024))
    scales = torch.randn(tensors, generator=torch.Generator().manual_seed(seed)).exp()
    for t in range(tensors):
        g[:, d * t // tensors:d * (t + 1) // tensors] *= float(scales[t])
    return g


def prepare(case, seed):
    N, c, d, kind = case["N"], case["c"], length(case), case["kind"]
    s = {"kind": kind, "N": N, "d": d, "grads": gradients(case, seed)}
    if kind == "norms":
        out = torch.randn((N, d), dtype=torch.float32, device="cuda",
                          generator=torch.Generator(device="cuda").manual_seed(seed + 1))
        s["out"] = out.mul_(0.03).add_(s["grads"].sum(dim=0))        # a sum that is 3 % off
        s["norms"] = torch.empty(N + 1, dtype=torch.float64, device="cuda")
        return s
    plan = plan_of(N, c)
    plan.prepare_device()
    s["plan"] = plan
    if kind == "buckets":
        s["buckets"] = bucket_list(case)
        work_floats, ws_bytes = plan.bucketed_sizes([n for _, n in s["buckets"]])
        s["work"] = torch.empty((N, work_floats), dtype=torch.float32, device="cuda")
        s["ws"] = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
        s["out"] = torch.empty((N, d), dtype=torch.float32, device="cuda")
    elif kind == "fused":
        s["out"] = torch.empty((N, d), dtype=torch.float32, device="cuda")
    else:
        s["work"], s["ws"], s["out"] = C.allocate(plan, d)
    return s


def run(s):
    kind, d = s["kind"], s["d"]
    if kind == "norms":
        C.error_norms(s["N"], d, s["grads"], s["out"], s["norms"])
        return s["norms"]
    plan = s["plan"]
    if kind == "fused":
        C.ring_simulate_fused(plan, d, s["grads"], s["out"])
        return {"out": s["out"]}
    if kind == "ring":
        C.ring_simulate(plan, d, s["grads"], s["work"], s["ws"], s["out"])
    elif kind == "noalloc":
        C.ring_simulate_noalloc(plan, d, s["grads"], s["work"], s["out"])
    elif kind == "buckets":
        C.ring_simulate_bucketed(plan, s["buckets"], s["grads"], s["work"], s["ws"], s["out"])
    else:
        for step in range(plan.L + 1):
            C.encode_round(plan, step, d, s["grads"], s["work"], s["ws"])
        C.decode(plan, d, s["work"], s["ws"], s["out"])
    return {"out": s["out"], "work": s["work"]}


def work(case):
    """Bytes: the gradients read and the sums written once, and, where the call
    leaves them, the L+1 observations of every worker written once; the step
    calls must move every message between calls.  Flops: both contractions
    and the rounds' sums."""
    N, c, kind = case["N"], case["c"], case["kind"]
    if kind == "norms":
        n = N * case["d"]
        return {"bytes": 8 * n, "flops": 4 * n}
    lens = [n for _, n in bucket_list(case)] if kind == "buckets" else [case["d"]]
    total = sum(lens)
    p = sum(-(-n // c) for n in lens)
    K = c + N - 1
    flops = N * p * (2 * c * c + 2 * K * c + 2 * c - 3)
    if kind == "steps":
        return {"bytes": 4 * N * p * (8 * c + 3 * N - 9), "flops": flops}
    return {"bytes": 8 * N * total + (0 if kind == "fused" else 4 * N * p * K), "flops": flops}


def tolerance(case):
    """A message keeps the rounding of every round before it, and the decode
    amplifies that by up to kappa(M): 0.3 to 1.4 kappa u of relative error was
    measured over these plans (2e-5 at N=8, c=64, kappa 393), and four times the
    most is allowed.  The norms are sums of squares in fp64; sums in another
    order differ by 3e-15 at most."""
    if case["kind"] == "norms":
        return {"rel": 2e-14}
    return {"rel": 4 * 1.4 * plan_of(case["N"], case["c"]).info()["kappa_M"] * UNIT_ROUNDOFF}


def all_reduce_64(g, U, R):
    """The protocol in 64 bits on one instance's gradients (N, d): the update
    equations on whole chunks, in slices of the positions."""
    N, d = g.shape
    c, K = U.shape[1], R.shape[1]
    p = -(-d // c)
    p = -(-p // 32) * 32                                 # the chunk length that cerar_chunk_len documents
    out = torch.empty((N, c, p), dtype=torch.float64, device=g.device)
    if c * p != d:
        g = torch.cat([g, g.new_zeros((N, c * p - d))], dim=1)
    G = g.reshape(N, c, p)
    step = max(1, (1 << 28) // (N * (2 * c + K)))
    for e in range(0, p, step):
        delta = torch.matmul(U.transpose(1, 2).contiguous(), G[:, :, e:e + step].double())
        x = delta[:, 0].clone()
        Y = torch.empty((N, K, delta.shape[2]), dtype=torch.float64, device=g.device)
        for k in range(1, K):                            # round k: worker i receives x of worker i - 1
            x = x.roll(1, 0)
            Y[:, k - 1] = x
            if k >= N:
                x = x - delta[:, k - N]
            if k < c:
                x = x + delta[:, k]
        Y[:, K - 1] = delta[:, c - 1]
        out[:, :, e:e + step] = torch.matmul(R.transpose(1, 2).contiguous(), Y)
    return out.reshape(N, c * p)[:, :d]


def exact(case, seed):
    g = gradients(case, seed)
    N, c, d, kind = case["N"], case["c"], length(case), case["kind"]
    if kind == "norms":
        out = torch.randn((N, d), dtype=torch.float32, device="cuda",
                          generator=torch.Generator(device="cuda").manual_seed(seed + 1))
        out.mul_(0.03).add_(g.sum(dim=0))
        S = torch.zeros(d, dtype=torch.float64, device="cuda")
        for w in range(N):
            S += g[w]
        return torch.stack([(out[w] - S).square().sum() for w in range(N)] + [S.square().sum()])
    U, R = (torch.from_numpy(m).cuda() for m in plan_of(N, c).matrices())
    if kind != "buckets":
        res = all_reduce_64(g, U, R)
    else:
        res = torch.empty((N, d), dtype=torch.float64, device="cuda")
        for o, n in bucket_list(case):
            res[:, o:o + n] = all_reduce_64(g[:, o:o + n], U, R)
    return {"out": res} if kind == "fused" else {"out": res, "work": None}
