"""The direct projection kernel (fewer than 32 states, vocabularies below a tile
of 128 words or beyond 2^25) at the sizes where it can go wrong, against the
fp64 oracle: states around 16 and 32, words around a tile, every tile it has,
several tiles per split, and vocabularies on both sides of 2^25, where the
register-staged kernel's 32-bit offsets end."""
import pytest
import torch

from synth import workloads as wl
from tests.gpu_util import check, run_step

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1805_09863_amd as kb
    kb.lib()
    return kb


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("tile", ["128x256", "32x512", "32x128"])
@pytest.mark.parametrize("H", [1, 8, 15, 16, 17, 31])
def test_few_states(kb, dt, tile, H, monkeypatch):
    monkeypatch.setenv("KB_TILE", tile)
    for rps, V, k in (([3] * 11, 513, 3), ([9] * 15, 1030, 9), ([16] * 9 + [5], 6007, 16)):
        inp = wl.make_step(H=H, V=V, k=k, rows_per_sentence=rps, dtype=dt, seed=4800 + H, name=f"H{H} V{V} {tile}")
        p = kb.kbest_plan(kb.KB_BF16 if dt == "bf16" else kb.KB_F32, inp.N, H, V, k)
        assert f"{p['tile_rows']}x{p['tile_words']}" == tile
        check(inp, run_step(kb, inp, row_lse=True))


@pytest.mark.parametrize("dt", ["bf16", "f32"])
def test_several_tiles_per_split(kb, dt, monkeypatch):
    # 9 row tiles of 128, so at most 28 splits of the 40 word tiles
    monkeypatch.setenv("KB_TILE", "128x256")
    inp = wl.make_step(H=24, V=10003, k=5, rows_per_sentence=[5] * 230, dtype=dt, seed=4850, name="direct tiles")
    assert kb.kbest_plan(kb.KB_BF16 if dt == "bf16" else kb.KB_F32, inp.N, 24, 10003, 5)["tiles_per_split"] == 2
    check(inp, run_step(kb, inp, row_lse=True))


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("V", [1, 31, 96, 127])
def test_narrow_vocabularies(kb, dt, V):
    # one word tile, states of several loads of 16 and a remainder
    for H, rps in ((256, [4] * 10), (1001, [2] * 33)):
        inp = wl.make_step(H=H, V=V, k=min(4, V), rows_per_sentence=rps, dtype=dt, seed=4870 + V, name=f"V{V} H{H}")
        check(inp, run_step(kb, inp, row_lse=True))


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("V", [(1 << 25) - 3, 1 << 25, (1 << 25) + 5])
def test_widest_vocabularies(kb, dt, V):
    N, H, k = 10, 33, 3
    td = torch.bfloat16 if dt == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(V % 1000)
    h = (torch.randn(N, H, generator=g, device="cuda") * 0.3).to(td)
    W = torch.randn(H, V, generator=g, device="cuda", dtype=td)
    # the best words of all rows at both ends of the vocabulary, where offsets are smallest and largest
    b = torch.zeros(V, device="cuda")
    b[[0, 7, V - 9, V - 1]] = 20.0
    tok, val = kb.argmax_step(h, W, b)
    prev = torch.zeros(N, device="cuda")
    off = torch.arange(0, N + 1, 2, dtype=torch.int32, device="cuda")
    kt, kp, ks = kb.kbest_step(h, W, b, prev, off, k)
    torch.cuda.synchronize()
    x = torch.empty(N, V, dtype=torch.float32, device="cuda")
    for v in range(0, V, 1 << 22):
        x[:, v:v + (1 << 22)] = (h.double() @ W[:, v:v + (1 << 22)].double() + b[v:v + (1 << 22)]).float()
    want, word = x.max(1)
    assert torch.equal(tok.long(), word)
    # a float32 sum of 33 products and a bias, below 64 at every step: 34 roundings of at most 2^-24 * 64
    assert (val - want).abs().max() < 1.3e-4
    lse = torch.cat([torch.logsumexp(x[r:r + 1].double(), 1) for r in range(N)])
    for s in range(N // 2):
        y = torch.cat([x[r].double() - lse[r] for r in (2 * s, 2 * s + 1)])
        best, i = y.topk(k)
        assert torch.equal(kt[s].long(), i % V) and torch.equal(kp[s].long(), i // V + 2 * s)
        assert (ks[s].double() - best).abs().max() < 2.6e-4   # the log-sum-exp's terms are as far off
