"""The register-staged projection kernel at the sizes where it can go wrong,
against the fp64 oracle: states around whole stages (32 in bf16, 16 in
float32) and below one, vocabularies around whole tiles and below one,
operands at odd addresses, and float32 values that the split into bf16 pieces
has to carry exactly."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import kbest_oracle as ko
from synth import workloads as wl
from tests.gpu_util import check, run_step, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1805_09863_amd as kb
    kb.lib()
    return kb


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("H", [1, 7, 15, 16, 17, 31, 32, 33, 63, 65, 127, 129, 200])
def test_state_sizes(kb, dt, H):
    # around one stage, an even and an odd number of them, and whole register sets
    inp = wl.make_step(H=H, V=1033, k=4, rows_per_sentence=[4] * 9 + [3], dtype=dt, seed=4000 + H, name=f"H{H}")
    check(inp, run_step(kb, inp, row_lse=True))


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("V", [1, 3, 17, 127, 128, 129, 255, 257, 511, 513, 769, 1281])
def test_vocabulary_sizes(kb, dt, V):
    # below, at and above one tile of 128, 256 and 512 words: the last tile starts early enough to end at V
    k = min(5, V)
    for rps in ([5] * 2 + [1], [5] * 8, [5] * 45):
        inp = wl.make_step(H=72, V=V, k=k, rows_per_sentence=rps, dtype=dt, seed=4200 + V, name=f"V{V}")
        check(inp, run_step(kb, inp, row_lse=True))


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("tile", ["128x256", "256x128", "32x512", "32x256", "32x128", "64x256"])
def test_operands_at_odd_addresses(kb, dt, tile, monkeypatch):
    # h, W and b one element past a 16-byte boundary: shapes that are otherwise
    # 16-byte loadable, and V odd
    monkeypatch.setenv("KB_TILE", tile)
    for H, V in ((128, 2048), (96, 2051)):
        inp = wl.make_step(H=H, V=V, k=6, rows_per_sentence=[6] * 25, dtype=dt, seed=4400 + V, name=f"odd{V}")
        h, W, b, prev, off = to_dev(inp)

        def moved(x):
            buf = torch.empty(x.numel() + 9, dtype=x.dtype, device="cuda")
            y = buf[1:1 + x.numel()].view(x.shape)
            y.copy_(x)
            return y
        h, W, b = moved(h), moved(W), moved(b)
        assert kb.kbest_plan(kb.KB_BF16 if dt == "bf16" else kb.KB_F32, inp.N, H, V, 6, aligned=False)["kernel"] == "reg"
        out = kb.kbest_step(h, W, b, prev, off, 6)
        torch.cuda.synchronize()
        check(inp, tuple(x.cpu().numpy() for x in out))


@pytest.mark.parametrize("values", ["ordinary", "cut", "small", "largest"])
def test_float32_split_carries_every_bit(kb, values):
    # greedy scores of one-hot states are single products h * w, plus zeros:
    # the pieces' products must give them to float32 rounding, whatever the
    # magnitudes and bits.  Each row of W has its largest entry, the one that is
    # read back, at a random word.
    g = np.random.default_rng(5)
    H, V, N = 64, 1024, 2048
    W = (0.4 * g.random((H, V))).astype(np.float32)
    top = 1.0 + g.random(H)             # 24 random bits
    state = 1.0 + g.random(N)
    if values == "cut":                 # first pieces cut off, not rounded, would leave most behind
        top[:] = 1 + 2.0 ** -7 - 2.0 ** -16
        state[::2] = 1 + 2.0 ** -7 - 2.0 ** -16
    W[np.arange(H), g.integers(0, V, H)] = top
    state = state.astype(np.float32) * np.exp2(g.integers(-20, 20, N)).astype(np.float32)
    W *= np.exp2(g.integers(-20, 20, (H, 1))).astype(np.float32)
    if values == "small":               # weights whose third pieces are subnormal in bf16, the smallest exact ones
        W *= np.float32(2.0 ** -109) / np.exp2(np.floor(np.log2(W.max(1, keepdims=True))))
        state = np.abs(state) * np.float32(2.0 ** 60)
    if values == "largest":             # next to FLT_MAX, whose rounding to bf16 is infinite
        W = (W / W.max(1, keepdims=True) * np.float32(3.4028235e38)).astype(np.float32)
        state = (np.abs(state) * np.float32(2.0 ** -100)).astype(np.float32)
    h = np.zeros((N, H), np.float32)
    h[np.arange(N), np.arange(N) % H] = state
    b = np.zeros(V, np.float32)
    assert kb.kbest_plan(kb.KB_F32, N, H, V, 1)["kernel"] == "dma"
    tok, val = kb.argmax_step(*(torch.from_numpy(x).cuda() for x in (h, W, b)))
    torch.cuda.synchronize()
    col = W.astype(np.float64)[np.arange(N) % H]
    want = state.astype(np.float64) * col.max(1)
    assert np.array_equal(tok.cpu().numpy(), col.argmax(1))
    err = np.abs(val.cpu().numpy() - want) / np.abs(want)
    say(f"{values}: largest relative error {err.max():.2e}")
    # the three products left out are below 2^-24 of the product together; then
    # the float32 rounding of the sum, and those of the five smaller products'
    # sums, together below an eighth of it
    assert err.max() < 2.0 ** -24 * (1 + 1 + 0.125)


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("H,V", [(128, 5000), (100, 5003)])
def test_64_row_tile_of_256_words(kb, dt, H, V, monkeypatch):
    # the DMA pipeline's (aligned bf16) and the register-staged form, over
    # several row tiles, ragged rows and words, k from 1 to 16
    monkeypatch.setenv("KB_TILE", "64x256")
    for k, rps in ((1, [1] * 64), (7, [7] * 21), (12, [12] * 11), (16, [16] * 4 + [1])):
        inp = wl.make_step(H=H, V=V, k=k, rows_per_sentence=rps, dtype=dt, seed=4600 + k, name=f"64x256 k{k}")
        plan = kb.kbest_plan(kb.KB_BF16 if dt == "bf16" else kb.KB_F32, inp.N, H, V, k)
        assert (plan["tile_rows"], plan["tile_words"]) == (64, 256)
        check(inp, run_step(kb, inp, row_lse=True))
