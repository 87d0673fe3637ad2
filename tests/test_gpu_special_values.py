"""Scores that are infinite, NaN or zeros of either sign, on every projection
kernel: they are ranked as the strict '>' scan ranks them (an infinity beats
every number, a NaN is no candidate, -0 equals +0 and the lower word wins)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1805_09863_amd as kb
    kb.lib()
    return kb


# (dtype, N, H, V, forced tile): the 256 x 256 kernel, the DMA pipeline, the
# register-staged kernel in bf16 and float32, the few-row kernel
KERNELS = [("bf16", 300, 128, 2048, "256x256"), ("bf16", 300, 128, 2048, "128x256"), ("bf16", 40, 128, 2048, "32x128"),
           ("bf16", 300, 100, 2051, "256x128"), ("bf16", 40, 100, 2051, "32x512"), ("f32", 300, 128, 2048, "128x256"),
           ("f32", 40, 100, 2051, "32x128"), ("f32", 100, 128, 2048, "64x128"), ("f32", 100, 100, 2051, "64x256"),
           ("f32", 4, 128, 2048, None), ("bf16", 4, 128, 2048, None)]


def _operands(dt, N, H, V):
    g = torch.Generator().manual_seed(N * 7 + V)
    td = torch.bfloat16 if dt == "bf16" else torch.float32
    h = torch.randn(N, H, generator=g).to(td)
    W = (torch.randn(H, V, generator=g) / H ** 0.5).to(td)
    b = torch.rand(V, generator=g) * 0.2 - 0.1
    return h, W, b


def _pin(monkeypatch, tile):
    if tile is None:
        monkeypatch.delenv("KB_TILE", raising=False)
    else:
        monkeypatch.setenv("KB_TILE", tile)


def _argmax(kb, h, W, b):
    tok, val = kb.argmax_step(h.cuda(), W.cuda(), b.cuda())
    torch.cuda.synchronize()
    return tok.cpu().numpy(), val.cpu().numpy()


@pytest.mark.parametrize("case", range(len(KERNELS)))
@pytest.mark.parametrize("value", ["nan", "-nan", "+inf", "-inf"])
def test_bias_that_is_no_number(kb, case, value, monkeypatch):
    dt, N, H, V, tile = KERNELS[case]
    if "nan" in value and tile is None:
        pytest.skip("the few-row kernel ranks a NaN by its bits")
    _pin(monkeypatch, tile)
    h, W, b = _operands(dt, N, H, V)
    bits = {"nan": 0x7FC00000, "-nan": 0xFFC00000, "+inf": 0x7F800000, "-inf": 0xFF800000}[value]
    words = [5, 131, V // 2, V - 3]
    b[words] = torch.from_numpy(np.array([bits], np.uint32).view(np.float32))
    tok, val = _argmax(kb, h, W, b)
    if value == "+inf":
        assert (tok == 5).all() and (val == np.inf).all()   # equal scores: the lowest word
        return
    x = h.double().numpy() @ W.double().numpy() + b.double().numpy()
    x[:, words] = -np.inf
    assert np.isfinite(val).all() and not np.isin(tok, words).any()
    # float32 sums of up to 128 products of unit-variance logits: within 1e-5 of the 64-bit maximum
    assert np.abs(val - x.max(1)).max() < 1e-5 and np.abs(x[np.arange(N), tok] - x.max(1)).max() < 1e-5


@pytest.mark.parametrize("case", range(len(KERNELS)))
def test_zeros_of_either_sign_are_equal(kb, case, monkeypatch):
    # every score is a zero: products +0 * -w are -0, and so is the sum where
    # the kernel adds them to a bias of -0; the k lowest words win
    dt, N, H, V, tile = KERNELS[case]
    _pin(monkeypatch, tile)
    h, W, b = _operands(dt, N, H, V)
    h[:] = 0.0
    W = -W.abs()
    b[:] = 0.0
    b[::2] = -0.0
    prev = torch.zeros(N)
    k = 4
    off = torch.arange(0, N + 1, dtype=torch.int32)
    tok, par, sc = kb.kbest_step(h.cuda(), W.cuda(), b.cuda(), prev.cuda(), off.cuda(), k)
    torch.cuda.synchronize()
    assert (tok.cpu().numpy() == np.arange(k)).all()
    assert (par.cpu().numpy() == np.arange(N)[:, None]).all()
    assert (_argmax(kb, h, W, b)[0] == 0).all()


# shapes of the register-staged kernel with its last stage whole, short of one
# state and one state long, and of the kernels that take operands as they are
MASKED = [("f32", 300, 128, 2048, "128x256"), ("f32", 40, 65, 2051, "32x128"), ("f32", 100, 127, 2051, "64x256"),
          ("f32", 300, 100, 1030, "256x128"), ("f32", 64, 128, 4096, "64x128"), ("f32", 40, 500, 2051, "32x512"),
          ("bf16", 300, 100, 2051, "256x128"), ("bf16", 40, 65, 2051, "32x512"), ("bf16", 100, 127, 2051, "64x256"),
          ("bf16", 40, 500, 2051, "32x128"), ("bf16", 300, 128, 2048, "256x256"), ("bf16", 40, 20, 1033, "32x128"),
          ("f32", 40, 20, 1033, "32x128"), ("f32", 4, 128, 2048, None)]


@pytest.mark.parametrize("case", range(len(MASKED)))
@pytest.mark.parametrize("at", ["first", "middle", "last"])
@pytest.mark.parametrize("mask", ["-inf", "lowest"])
def test_words_masked_through_the_weights(kb, case, at, mask, monkeypatch):
    # a state of constant 1 carries a mask: -inf or the type's lowest number in
    # its row of W takes a word out (probability 0), and the other words' scores
    # are theirs
    dt, N, H, V, tile = MASKED[case]
    _pin(monkeypatch, tile)
    h, W, b = _operands(dt, N, H, V)
    c = {"first": 0, "middle": H // 2, "last": H - 1}[at]
    h[:, c] = 1.0
    masked = np.zeros(V, bool)
    masked[1::3] = True
    masked[V - 1] = True
    W[c, torch.from_numpy(masked)] = -float("inf") if mask == "-inf" else torch.finfo(W.dtype).min
    k = 4
    prev = torch.zeros(N)
    off = torch.arange(0, N + 1, 2, dtype=torch.int32)
    lse = torch.empty(N, device="cuda")
    tok, par, sc = kb.kbest_step(h.cuda(), W.cuda(), b.cuda(), prev.cuda(), off.cuda(), k, row_lse=lse)
    torch.cuda.synchronize()
    keep = np.flatnonzero(~masked)
    x = h.double().numpy() @ W.double().numpy()[:, keep] + b.double().numpy()[keep]
    want = np.log(np.exp(x).sum(1))
    # float32 sums of at most 500 products of unit-variance logits
    assert np.abs(lse.cpu().numpy() - want).max() < 1e-5
    y = x - want[:, None]
    for s in range(N // 2):
        best = np.sort(y[2 * s:2 * s + 2].ravel())[::-1][:k]
        assert np.abs(sc[s].cpu().numpy() - best).max() < 2e-5
        t, p = tok[s].cpu().numpy(), par[s].cpu().numpy()
        assert not masked[t].any()
        assert np.abs(y[p, np.searchsorted(keep, t)] - best).max() < 2e-5


@pytest.mark.parametrize("case", range(len(MASKED)))
def test_infinite_states_and_weights(kb, case, monkeypatch):
    dt, N, H, V, tile = MASKED[case]
    _pin(monkeypatch, tile)
    h, W, b = _operands(dt, N, H, V)
    c = H - 2
    h[3, c] = float("inf")          # row 3: +-inf by the sign of W's entry
    W[c] = W[c].abs() + 0.01
    W[c, :11] = -W[c, :11]
    tok, val = _argmax(kb, h, W, b)
    assert tok[3] == 11 and val[3] == np.inf
    rest = np.arange(N) != 3
    x = h.double().numpy()[rest] @ W.double().numpy() + b.double().numpy()
    assert np.abs(val[rest] - x.max(1)).max() < 1e-5
    h[3, c] = 1.0
    h[:, c] = h[:, c].abs() + 0.01
    W[c, [V - 2, V // 2]] = float("inf")
    tok, val = _argmax(kb, h, W, b)
    assert (tok == V // 2).all() and (val == np.inf).all()
