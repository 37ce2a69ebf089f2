"""The performance workload of the scan library: what layers built on it ask of its public entry points.

A case is a dict of plain values.  `kind` selects the entry points:

    scan     selective scan of a batch [B,D,L] (real A): `run` is "train" (forward with state checkpoints, then
             backward on them), "forward" (prefill: outputs and the last state) or "backward" (gradients with the
             states recomputed inside the call)
    packed   the same as "train" on a packed variable-length batch of S sequences, L steps in all
    complex  the selective scan with a complex diagonal A, forward and backward
    step     one generated token: the carried state is updated in place
    lti      S5 / LRU recurrence with constant complex poles, forward and adjoint
    diag     recurrence with caller-supplied coefficients (gated layers), forward and adjoint

`listed()` gives the named cases, `draw(rng)` one more of the same ranges, `prepare(case, seed)` the tensors on the
GPU, `run(state)` one pass, `work(case)` the bytes and operations a pass cannot do without, `tolerance(case)` how far
two correct implementations may be apart.
"""
import math
import random

import torch

from paper_2602_08810_amd import api


def listed():
    return [
        # The smallest useful call: a toy layer in float32 (benchmark configuration 0).  Latency of one launch.
        dict(name="tiny_forward_f32", kind="scan", run="forward", B=1, D=16, N=4, L=256, io="f32", gate=False,
             disc="zoh_s6", groups=1),
        # Autoregressive generation, 64 streams of one Mamba-width layer: called once per token and layer.
        dict(name="decode_step", kind="step", B=64, D=1536, N=16, io="bf16", gate=True, disc="zoh_s6", groups=1,
             complex_a=False),
        # Training step of one Mamba block (configuration 2, the benchmark's workload).
        dict(name="train_block", kind="scan", run="train", B=8, D=1536, N=16, L=2048, io="bf16", gate=True,
             disc="zoh_s6", groups=1),
        # Training in float32 on sizes that divide nothing: odd channel count, odd length.
        dict(name="train_ragged_f32", kind="scan", run="train", B=3, D=771, N=16, L=1531, io="f32", gate=True,
             disc="zoh_s6", groups=1),
        # Backward of a large block with activation recomputation (configuration 4): the largest case.
        dict(name="recompute_backward_large", kind="scan", run="backward", B=16, D=2560, N=16, L=4096, io="bf16",
             gate=True, disc="zoh_s6", groups=1),
        # Prefill of one long prompt (configuration 3): outputs and the state that decoding starts from.
        dict(name="prefill_long", kind="scan", run="forward", B=1, D=2048, N=16, L=65536, io="bf16", gate=False,
             disc="zoh_s6", groups=1),
        # Training on one long document: few rows, long time axis.
        dict(name="train_long_few_rows", kind="scan", run="train", B=1, D=768, N=16, L=16384, io="bf16", gate=True,
             disc="zoh_s6", groups=1),
        # Fine-tuning on sequences of mixed lengths packed on one time axis without padding.
        dict(name="train_packed", kind="packed", S=24, D=1536, N=16, L=16384, lengths=1, io="bf16", gate=True,
             disc="zoh_s6", groups=1),
        # Training step of a layer with complex poles and input-dependent maps.
        dict(name="train_complex", kind="complex", B=8, D=1536, N=16, L=2048, io="bf16", gate=True, disc="zoh_s6",
             groups=1),
        # Training step of an S5 / LRU layer of moderate size (configuration 1 and its adjoint).
        dict(name="lti_layer", kind="lti", B=4, P=256, L=4096),
        # The same recurrence at a size well past the caches: the streaming rate of the memory.
        dict(name="lti_large", kind="lti", B=8, P=1024, L=8192),
        # Training step of a gated real recurrence whose gates the caller computes.
        dict(name="diag_gated", kind="diag", B=8, P=1024, L=2048, complex_a=False),
    ]


# ---------------------------------------------------------------- further cases of the same ranges
def _log(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi]."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _options(rng, D):
    groups = rng.choice([1, 1, 1, 1, 2, 4])
    return dict(D=(D + groups - 1) // groups * groups, groups=groups, N=rng.choice([16, 16, 16, 8, 4, 32]),
                io=rng.choice(["bf16", "bf16", "bf16", "f32"]), gate=rng.random() < 0.7,
                disc=rng.choice(["zoh_s6", "zoh_s6", "zoh_s6", "zoh", "bilinear"]))


# state updates (B * D * L * N) of a drawn case: at most a quarter of the largest listed one (an eighth with complex A,
# whose update is four times the work)
_MOST = 16 * 2560 * 4096 * 16 // 4


def draw(rng):
    kind = rng.choice(["scan", "scan", "scan", "scan", "scan", "packed", "complex", "step", "lti", "diag"])
    if kind == "lti":
        P, L = _log(rng, 16, 1024), _log(rng, 64, 16384)
        return dict(kind=kind, B=_log(rng, 1, max(1, min(32, 8 * 1024 * 8192 // (P * L)))), P=P, L=L)
    if kind == "diag":
        P, L = _log(rng, 16, 2048), _log(rng, 64, 16384)
        return dict(kind=kind, B=_log(rng, 1, max(1, min(32, 8 * 1024 * 4096 // (P * L)))), P=P, L=L,
                    complex_a=rng.random() < 0.5)
    if kind == "step":
        c = dict(kind=kind, B=_log(rng, 1, 256), complex_a=rng.random() < 0.25, **_options(rng, _log(rng, 256, 5120)))
        if c["complex_a"]:
            c["N"] = min(c["N"], 16)
        return c
    if kind == "packed":
        c = dict(kind=kind, **_options(rng, _log(rng, 128, 2560)))
        c["L"] = min(_log(rng, 2048, 32768), _MOST // (c["D"] * c["N"]))
        c["S"] = _log(rng, 2, max(2, min(96, c["L"] // 64)))
        c["lengths"] = rng.randrange(1 << 16)
        return c
    c = dict(kind=kind, **_options(rng, _log(rng, 16, 2560)))
    if kind == "complex":
        c["N"] = min(c["N"], 16)
    most = _MOST // (2 if kind == "complex" else 1) // (c["D"] * c["N"])
    c["L"] = min(_log(rng, 64, 65536 if kind == "scan" else 8192), most)
    c["B"] = _log(rng, 1, max(1, min(64, most // c["L"])))
    if kind == "scan":
        c["run"] = rng.choice(["train", "train", "forward", "backward"])
    return c


# ---------------------------------------------------------------- inputs
def _lengths(case):
    """Lengths of the packed sequences: at least 8 steps each, log-normal shares of the rest, L in all."""
    r = random.Random(case["lengths"])
    S, L = case["S"], case["L"]
    share = [r.lognormvariate(0.0, 0.8) for _ in range(S)]
    free, total = L - 8 * S, sum(share)
    edges = [round(free * sum(share[:i]) / total) + 8 * i for i in range(S + 1)]
    return [b - a for a, b in zip(edges, edges[1:])]


class _Draw:
    """Random tensors on the GPU from one seed."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def normal(self, shape, dtype=torch.float32):
        return torch.randn(shape, generator=self.g, device="cuda").to(dtype)

    def uniform(self, shape, lo, hi):
        return torch.rand(shape, generator=self.g, device="cuda") * (hi - lo) + lo

    def complex_normal(self, shape):
        return torch.view_as_complex(self.normal((*shape, 2)) * math.sqrt(0.5))

    def poles(self, shape):
        """r e^{i theta} with r ~ U(0.9, 0.999): decaying states with memories of 10 to 1000 steps."""
        return torch.polar(self.uniform(shape, 0.9, 0.999), self.uniform(shape, 0.0, 2.0 * math.pi))


def _io(case):
    return torch.bfloat16 if case["io"] == "bf16" else torch.float32


def _selective(case, r, rows, maps, complex_a):
    """Keyword arguments of the selective entry points; rows: shape of u, maps: leading shape of Bm and Cm."""
    io, D, N = _io(case), case["D"], case["N"]
    A = -torch.exp(r.uniform((D, N), -1.0, 1.0))
    if complex_a:
        A = torch.complex(A, r.uniform((D, N), -10.0, 10.0))
        pairs = [r.normal((*maps, N, 2), io) * math.sqrt(0.5) for _ in range(2)]
        Bm, Cm = pairs if io == torch.bfloat16 else [torch.view_as_complex(m) for m in pairs]
    else:
        Bm, Cm = r.normal((*maps, N), io), r.normal((*maps, N), io)
    return dict(u=r.normal(rows, io), delta=r.normal(rows, io), A=A, Bm=Bm, Cm=Cm, Dskip=r.normal((D,)),
                delta_bias=r.uniform((D,), -4.0, -2.0), z=r.normal(rows, io) if case["gate"] else None,
                disc=case["disc"])


def prepare(case, seed):
    r = _Draw(seed)
    kind = case["kind"]
    if kind == "lti":
        shape = (case["B"], case["L"], case["P"])
        return dict(case=case, lam=r.poles((case["P"],)), v=r.complex_normal(shape), gx=r.complex_normal(shape))
    if kind == "diag":
        shape = (case["B"], case["L"], case["P"])
        if case["complex_a"]:
            return dict(case=case, a=r.poles(shape), b=r.complex_normal(shape), gx=r.complex_normal(shape))
        return dict(case=case, a=r.uniform(shape, 0.5, 1.0), b=r.normal(shape), gx=r.normal(shape))
    D, N, G = case["D"], case["N"], case["groups"]
    if kind == "step":
        B, cplx = case["B"], case["complex_a"]
        x = r.complex_normal((B, D, N)) if cplx else r.normal((B, D, N))
        return dict(case=case, x=x, args=_selective(case, r, (B, D), (B, G) if G > 1 else (B,), cplx))
    L = case["L"]
    if kind == "packed":
        lens = _lengths(case)
        cu = torch.tensor([sum(lens[:i]) for i in range(len(lens) + 1)], dtype=torch.int64, device="cuda")
        args = _selective(case, r, (D, L), (G, L) if G > 1 else (L,), False)
        return dict(case=case, args=args, cu=cu, longest=max(lens), dy=r.normal((D, L), _io(case)))
    B = case["B"]
    args = _selective(case, r, (B, D, L), (B, G, L) if G > 1 else (B, L), kind == "complex")
    s = dict(case=case, args=args)
    if kind == "complex" or case["run"] != "forward":
        s["dy"] = r.normal((B, D, L), _io(case))
    return s


# ---------------------------------------------------------------- one pass
def run(s):
    kind = s["case"]["kind"]
    if kind == "lti":
        x = api.lrnnx_lti_diag_scan(s["lam"], s["v"])
        dv, dlam, dx0 = api.lrnnx_lti_diag_scan_bwd(s["lam"], x, s["gx"])
        return dict(x=x, dv=dv, dlam=dlam, dx0=dx0)
    if kind == "diag":
        x = api.lrnnx_diag_scan(s["a"], s["b"])
        da, db, dx0 = api.lrnnx_diag_scan_bwd(s["a"], x, s["gx"])
        return dict(x=x, da=da, db=db, dx0=dx0)
    if kind == "step":
        step = api.lrnnx_selective_step_complex if s["case"]["complex_a"] else api.lrnnx_selective_step
        return dict(y=step(s["x"], **s["args"]), x=s["x"])
    if kind == "packed":
        y, ckpt = api.lrnnx_selective_scan_fwd(**s["args"], cu_seqlens=s["cu"], return_ckpt=True)
        g = api.lrnnx_selective_scan_bwd(**s["args"], dy=s["dy"], ckpt=ckpt, cu_seqlens=s["cu"], max_seqlen=s["longest"])
        return dict(y=y, **g)
    if kind == "complex":
        y, ckpt = api.lrnnx_selective_scan_fwd_complex(**s["args"], return_ckpt=True)
        return dict(y=y, **api.lrnnx_selective_scan_bwd_complex(**s["args"], dy=s["dy"], ckpt=ckpt))
    if s["case"]["run"] == "forward":
        y, last = api.lrnnx_selective_scan_fwd(**s["args"], return_last_state=True)
        return dict(y=y, x_last=last)
    if s["case"]["run"] == "backward":
        return api.lrnnx_selective_scan_bwd(**s["args"], dy=s["dy"])
    y, ckpt = api.lrnnx_selective_scan_fwd(**s["args"], return_ckpt=True)
    return dict(y=y, **api.lrnnx_selective_scan_bwd(**s["args"], dy=s["dy"], ckpt=ckpt))


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    """Bytes: every input read once and every output written once.  Operations per state update: 7 forward (the
    multiplier's product and exponential, the input term, the recurrence, the projection) and 22 backward (recompute,
    adjoint, seven gradient terms); a complex multiply-add counts 8."""
    kind = case["kind"]
    if kind in ("lti", "diag"):
        n = case["B"] * case["L"] * case["P"]
        if kind == "lti":                                # v, gx in; x, dv out
            return dict(bytes=8 * 4 * n, flops=8 * 3 * n)
        size, op = (8, 8) if case["complex_a"] else (4, 2)
        return dict(bytes=size * 6 * n, flops=op * 3 * n)        # a, b, gx in; x, da, db out
    D, N = case["D"], case["N"]
    es = 2 if case["io"] == "bf16" else 4
    if kind == "step":
        B, c = case["B"], 2 if case["complex_a"] else 1
        state = 2 * B * D * N * 4 * c                            # read and written
        rows = (3 + case["gate"]) * B * D * es
        return dict(bytes=state + rows + D * N * 4 * c + 2 * B * case["groups"] * N * es * c + 8 * D,
                    flops=7 * B * D * N * (4 if c == 2 else 1))
    B = 1 if kind == "packed" else case["B"]
    c = 2 if kind == "complex" else 1
    row = B * D * case["L"] * es
    maps = 2 * B * case["groups"] * case["L"] * N * c            # elements of Bm and Cm together
    small = D * N * 4 * c + 8 * D
    what = "train" if kind in ("packed", "complex") else case["run"]
    gate = 1 if case["gate"] else 0
    bytes_, ops = 0, 0
    if what in ("train", "forward"):
        bytes_ += row * (3 + gate) + maps * es + small           # u, delta, z, maps in; y out
        ops += 7
    if what == "forward":
        bytes_ += B * D * N * 4
    if what in ("train", "backward"):
        if what == "backward":
            bytes_ += row * (2 + gate) + maps * es + small       # in "train" the forward's reads stand for both
        bytes_ += row * (1 + 2 + gate) + maps * 4 + small        # dy in; du, ddelta, dz, dBm, dCm (float32) out
        ops += 22
    return dict(bytes=bytes_, flops=ops * B * D * case["L"] * N * (4 if c == 2 else 1))


def tolerance(case):
    # float32 (and complex64): sums of up to some 10^4 terms and recurrences with memories of up to 10^3 steps, in any
    # order.  bfloat16 results carry a rounding of 2^-9 each.
    if case.get("io", "f32") == "f32":
        return dict(rel=3e-5, max=2e-3)
    return dict(rel=1e-2, max=0.05)
