"""The performance cases of the output layer: what a decoder has it do, by size, type and entry point.

Four kinds of call, each through the package's public entry points:

  step     one beam-search decode step (``kbest_step``, or ``kbest_step_noalloc`` for a loop that
           may not allocate): the sizes run from one sentence to the largest batch, in float32 and
           bf16, with aligned and odd state and vocabulary sizes, uniform and ragged beams
  argmax   one greedy step (``argmax_step``)
  compact  removal of the finished hypotheses after a step (``compact_beams``) and the gathers of the
           surviving scores and states (``gather_rows``)
  loop     a whole decode of a batch of sentences with removal of finished ones (``decode_loop``),
           which hands every step's continuations to the caller

Inputs follow the synthetic workloads of ``synth``: h ~ N(0, 1), W ~ N(0, 1/sqrt(H)) (unit-variance
logits), bias U(-0.1, 0.1) (flat prior) or -0.5 ln(j + 1) (Zipf-like prior), previous scores U(-5, 0),
sentence lengths U{5..T}.  They are drawn on the GPU.
"""
import math

import torch

import paper_1805_09863_amd as kb
from paper_1805_09863_amd import decode

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


def listed():
    return [
        # one sentence being translated while its reader waits: small model, all latency
        dict(name="step_f32_5x256x8000", kind="step", dtype="f32", S=1, beam=5, H=256, V=8000, k=5),
        # the same on a large model, from a serving loop that may not allocate
        dict(name="step_bf16_5x1024x50000_noalloc", kind="step", dtype="bf16", S=1, beam=5, H=1024, V=50000, k=5,
             noalloc=True),
        # a small online batch whose sentences have shrunk to different beams
        dict(name="step_bf16_ragged37x1024x50000", kind="step", dtype="bf16", S=12, beam=5, ragged=True, H=1024,
             V=50000, k=5),
        # single precision, a batch of sentences (the paper's own precision for most results)
        dict(name="step_f32_320x512x30000", kind="step", dtype="f32", S=64, beam=5, H=512, V=30000, k=5),
        # single precision, state and vocabulary sizes that are no multiple of anything, row normalisers wanted
        dict(name="step_f32_odd_ragged132x500x32003", kind="step", dtype="f32", S=33, beam=8, ragged=True, H=500,
             V=32003, k=6, lse=True),
        # single precision, offline batch at beam 9
        dict(name="step_f32_1152x1024x50000_k9", kind="step", dtype="f32", S=128, beam=9, H=1024, V=50000, k=9,
             prior="zipf"),
        # half precision, a vocabulary as a subword learner leaves it (odd)
        dict(name="step_bf16_odd300x1000x49999", kind="step", dtype="bf16", S=75, beam=4, H=1000, V=49999, k=4,
             lse=True),
        # half precision, a middling batch
        dict(name="step_bf16_640x1024x60000", kind="step", dtype="bf16", S=128, beam=5, H=1024, V=60000, k=5),
        # half precision, the largest batch, beam and vocabulary
        dict(name="step_bf16_3072x1024x90000_k12", kind="step", dtype="bf16", S=256, beam=12, H=1024, V=90000, k=12,
             prior="zipf"),
        # greedy decoding of a large batch
        dict(name="argmax_bf16_1280x1024x90000", kind="argmax", dtype="bf16", N=1280, H=1024, V=90000),
        # after a step of the largest batch: the finished hypotheses leave, states move up
        dict(name="compact_512x12x1024", kind="compact", dtype="bf16", S=512, beam=12, H=1024),
        # a whole decode, from 640 rows down to the longest sentence's last step
        dict(name="loop_bf16_128sent_1024x50000", kind="loop", dtype="bf16", S=128, beam=5, H=1024, V=50000, T=60),
    ]


# a drawn step multiplies at most this many (rows x states x words)
MOST = {"f32": 1152 * 1024 * 50000, "bf16": 3072 * 1024 * 90000}


def _between(rng, lo, hi):
    """A whole number in [lo, hi], spread over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _sizes(rng, dtype):
    """State and vocabulary sizes: half of them the round ones of usual configurations, half odd."""
    if rng.random() < 0.5:
        return rng.choice([256, 512, 1024] if dtype == "f32" else [512, 1024]), _between(rng, 1000, 11250) * 8
    return rng.randint(250, 1024), _between(rng, 8000, 90000)


def draw(rng):
    kind = rng.choice(["step"] * 7 + ["argmax", "compact", "loop"])
    dtype = rng.choice(["f32", "bf16", "bf16"])
    if kind == "compact":
        return dict(kind="compact", dtype=dtype, S=_between(rng, 8, 512), beam=rng.randint(1, 12),
                    H=rng.choice([256, 500, 512, 1000, 1024]))
    H, V = _sizes(rng, dtype)
    if kind == "loop":
        return dict(kind="loop", dtype="bf16", S=_between(rng, 4, 128), beam=rng.randint(1, 5), H=H,
                    V=min(V, 50000), T=rng.randint(20, 60))
    beam = rng.randint(1, 12)
    S = _between(rng, 1, max(1, min(3072 // beam, MOST[dtype] // (beam * H * V))))
    if kind == "argmax":
        return dict(kind="argmax", dtype=dtype, N=S * beam, H=H, V=V)
    c = dict(kind="step", dtype=dtype, S=S, beam=beam, H=H, V=V, k=beam, ragged=rng.random() < 0.4,
             prior=rng.choice(["flat", "flat", "zipf"]), lse=rng.random() < 0.3)
    # a loop without allocation has a fixed scratch array, which holds the partials of these sizes
    if S * beam <= 320 and rng.random() < 0.25:
        c["noalloc"] = True
    return c


def _rows(case):
    """Rows of each sentence: the full beam, or 1 to beam of them."""
    if not case.get("ragged"):
        return [case["beam"]] * case["S"]
    return [1 + (5 * s + 2) % case["beam"] for s in range(case["S"])]


def _normal(shape, std, dtype, g):
    """N(0, std) in blocks of rows, so that float32 draws of a large bf16 array need no memory of its size."""
    out = torch.empty(shape, dtype=dtype, device="cuda")
    for r in range(0, shape[0], 4096):
        x = out[r:r + 4096]
        x.copy_(torch.randn(x.shape, generator=g, device="cuda", dtype=torch.float32) * std)
    return out


def _uniform(n, lo, hi, g):
    return torch.rand(n, generator=g, device="cuda", dtype=torch.float32) * (hi - lo) + lo


def _weights(case, g):
    H, V = case["H"], case["V"]
    W = _normal((H, V), 1.0 / math.sqrt(H), DTYPES[case["dtype"]], g)
    if case.get("prior") == "zipf":
        b = -0.5 * torch.log(torch.arange(1, V + 1, device="cuda", dtype=torch.float64)).float()
    else:
        b = _uniform(V, -0.1, 0.1, g)
    return W, b


def _lengths(case, g):
    lo, T = 5, case["T"]
    return (torch.rand(case["S"], generator=g, device="cuda") * (T - lo + 1)).to(torch.int32).clamp_(max=T - lo) + lo


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dt = DTYPES[case["dtype"]]
    i32 = dict(dtype=torch.int32, device="cuda")
    s = dict(case=case)
    if case["kind"] == "step":
        rows = _rows(case)
        N, S, k = sum(rows), case["S"], case["k"]
        s["h"] = _normal((N, case["H"]), 1.0, dt, g)
        s["W"], s["b"] = _weights(case, g)
        s["prev"] = _uniform(N, -5.0, 0.0, g)
        s["off"] = torch.tensor([0] + rows).cumsum(0).to(**i32)
        s["out"] = (torch.empty((S, k), **i32), torch.empty((S, k), **i32), torch.empty((S, k), device="cuda"))
        s["lse"] = torch.empty(N, device="cuda") if case.get("lse") else None
        if not case.get("noalloc"):
            code = kb.KB_BF16 if case["dtype"] == "bf16" else kb.KB_F32
            s["ws"] = kb.workspace(kb.kbest_workspace_bytes(code, N, case["H"], case["V"], k, S))
    elif case["kind"] == "argmax":
        s["h"] = _normal((case["N"], case["H"]), 1.0, dt, g)
        s["W"], s["b"] = _weights(case, g)
        code = kb.KB_BF16 if case["dtype"] == "bf16" else kb.KB_F32
        s["ws"] = kb.workspace(kb.argmax_workspace_bytes(code, case["N"], case["H"], case["V"]))
        s["out"] = (torch.empty(case["N"], **i32), torch.empty(case["N"], device="cuda"))
    elif case["kind"] == "compact":
        S, k = case["S"], case["beam"]
        M = S * k
        # about one sentence in ten ends at a step, and a few hypotheses of the others
        ended = torch.rand(S, 1, generator=g, device="cuda") < 0.1
        s["alive"] = ((torch.rand(S, k, generator=g, device="cuda") < 0.97) & ~ended).to(torch.uint8).reshape(M)
        s["h"] = _normal((M, case["H"]), 1.0, dt, g)
        s["score"] = _uniform(M, -60.0, 0.0, g).view(M, 1)
        s["out"] = (torch.zeros(M, **i32), torch.zeros(1, **i32), torch.zeros(S + 1, **i32), torch.zeros(S, **i32),
                    torch.zeros(1, **i32))
        s["h_next"] = torch.zeros_like(s["h"])
        s["score_next"] = torch.zeros_like(s["score"])
    else:
        S, k, T = case["S"], case["beam"], case["T"]
        s["table"] = _normal((S * T * k, case["H"]), 1.0, dt, g)
        s["W"], s["b"] = _weights(case, g)
        s["lengths"] = _lengths(case, g)
        s["prev"] = _uniform(S * k, -5.0, 0.0, g)
        # the continuations of every step, as a caller keeps them to read the translations back
        s["hist"] = (torch.zeros((T, S * k), **i32), torch.zeros((T, S * k), **i32),
                     torch.zeros((T, S * k), device="cuda"))
    return s


def run(s):
    case = s["case"]
    if case["kind"] == "step":
        if case.get("noalloc"):
            r = kb.kbest_step_noalloc(s["h"], s["W"], s["b"], s["prev"], s["off"], case["k"], out=s["out"],
                                      row_lse=s["lse"])
        else:
            r = kb.kbest_step(s["h"], s["W"], s["b"], s["prev"], s["off"], case["k"], out=s["out"], ws=s["ws"],
                              row_lse=s["lse"])
        return r + ((s["lse"],) if s["lse"] is not None else ())
    if case["kind"] == "argmax":
        return kb.argmax_step(s["h"], s["W"], s["b"], out=s["out"], ws=s["ws"])
    if case["kind"] == "compact":
        S, k = case["S"], case["beam"]
        keep, kept, noff, ksent, nS = kb.compact_beams(s["alive"], S, k, out=s["out"])
        kb.gather_rows(s["score"], keep, n_dev=kept, n_max=S * k, out=s["score_next"])
        kb.gather_rows(s["h"], keep, n_dev=kept, n_max=S * k, out=s["h_next"])
        return keep, kept, noff, ksent, nS, s["score_next"], s["h_next"]
    tok, par, sc = s["hist"]

    def keep_step(t, st):
        n = st["token"].numel()
        tok[t, :n].copy_(st["token"].view(-1))
        par[t, :n].copy_(st["parent"].view(-1))
        sc[t, :n].copy_(st["score"].view(-1))

    stats = decode.decode_loop(s["table"], s["W"], s["b"], s["lengths"], s["prev"], case["beam"], case["T"],
                               on_step=keep_step)
    return tok, par, sc, stats.total_rows


def _loop_rows(case):
    """Mean live rows of each step: sentence lengths are uniform over 5..T."""
    lo, T = 5, case["T"]
    return [case["S"] * case["beam"] * min(1.0, (T - t) / (T - lo + 1)) for t in range(T)]


def work(case):
    e = 2 if case["dtype"] == "bf16" else 4
    H = case["H"]
    if case["kind"] == "compact":
        M, S = case["S"] * case["beam"], case["S"]
        kept = 0.87 * M
        return dict(bytes=M + 4 * kept + 8 * S + 8 + kept * (8 + 2 * e * H), flops=M)
    V = case["V"]
    fixed = H * V * e + 4 * V
    if case["kind"] == "step":
        N, out = sum(_rows(case)), case["S"] * case["k"]
        return dict(bytes=fixed + N * (H * e + 4) + 4 * case["S"] + 12 * out + (4 * N if case.get("lse") else 0),
                    flops=2 * N * H * V)
    if case["kind"] == "argmax":
        return dict(bytes=fixed + case["N"] * (H * e + 8), flops=2 * case["N"] * H * V)
    rows = _loop_rows(case)
    return dict(bytes=sum(fixed + n * (H * e + 4 + 12) for n in rows), flops=sum(2 * n * H * V for n in rows))


def tolerance(case):
    if case["kind"] == "compact":
        return "exact"
    # float32 sums of exact products: the scores' errors are those of the sums (measured against 64 bits:
    # about 1e-7 of a score), and two candidates that lie closer than that may change places
    return {"rel": 1e-6, "max": 1e-5, "differ": 0.005}


def _merge64(logits, prev, off, k):
    """Log-sum-exp of every row, and the k best continuations of every sentence, best first."""
    lse = torch.logsumexp(logits, 1)
    logits -= (lse - prev)[:, None]
    V = logits.shape[1]
    tok, par, sc = [], [], []
    for a, z in zip(off[:-1], off[1:]):
        x, i = logits[a:z].reshape(-1).topk(k)
        tok.append(i % V)
        par.append(i // V + a)
        sc.append(x)
    return torch.stack(tok).int(), torch.stack(par).int(), torch.stack(sc), lse


def exact(case, seed):
    s = prepare(case, seed)
    if case["kind"] == "compact":
        return None  # nothing is computed: whole numbers and copies
    W, b = s["W"].double(), s["b"].double()
    if case["kind"] == "step":
        off = [0]
        for r in _rows(case):
            off.append(off[-1] + r)
        tok, par, sc, lse = _merge64(s["h"].double() @ W + b, s["prev"].double(), off, case["k"])
        return (tok, par, sc) + ((lse,) if case.get("lse") else ())
    if case["kind"] == "argmax":
        val, tok = (s["h"].double() @ W + b).max(1)
        return tok.int(), val
    S, k, T = case["S"], case["beam"], case["T"]
    lengths = s["lengths"].tolist()
    tok, par = (torch.zeros((T, S * k), dtype=torch.int32, device="cuda") for _ in range(2))
    sc = torch.zeros((T, S * k), dtype=torch.float64, device="cuda")
    live, prev, total = list(range(S)), s["prev"].double(), 0
    for t in range(T):
        rows = torch.tensor([(i * T + t) * k + r for i in live for r in range(k)], device="cuda")
        logits = s["table"][rows].double() @ W + b
        a, p, c, _ = _merge64(logits, prev, list(range(0, len(live) * k + 1, k)), k)
        n = a.numel()
        total += n
        tok[t, :n], par[t, :n], sc[t, :n] = a.view(-1), p.view(-1), c.view(-1)
        stay = [j for j, i in enumerate(live) if t < lengths[i] - 1]
        if not stay:
            break
        prev = c[torch.tensor(stay, device="cuda")].reshape(-1)
        live = [live[j] for j in stay]
    return tok, par, sc, total
