"""The fp32 attention and projection kernels at the edges of their blocks, against the float64
oracle: chunks that end on, before and after a 32-key block and a 32-row wave, a resumed chunk whose
keys pass the staged window of 512 pages, decode rows on both sides of the 64-key pass and of
the 256-key split, projections whose eight K slices hold unequal runs (K = 320) or fewer than one
round (K = 64), and caches whose base is only element-aligned."""
import pytest
import torch

from tests.parity import Pair
from workload import Batch, DecodeRow, EmbChunk, ModelConfig, PagedKV, draw_tokens, make_weights

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _need_gpu(request):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"\n[case] {request.node.name}", flush=True)


def config(d, nq, nkv, hd, ff):
    return ModelConfig(n_layers=1, d_model=d, n_q_heads=nq, n_kv_heads=nkv, head_dim=hd, d_ff=ff, vocab=96, dtype="f32")


@pytest.mark.parametrize("cfg,misaligned", [(config(320, 5, 5, 64, 64), False), (config(256, 4, 2, 128, 320), False),
                                            (config(256, 4, 1, 64, 192), True)],
                         ids=["hd64-group1-K320", "hd128-group2", "hd64-group4-misaligned"])
def test_blocks(cfg, misaligned):
    W = make_weights(cfg, 21)
    spans = [(0, 1), (0, 31), (0, 33), (31, 2), (160, 129), (8180, 40)]
    ctx = [0, 15, 63, 64, 255, 256, 300]
    n = len(spans) + len(ctx)
    kv = PagedKV(cfg, sum(-(-(o + c) // 16) for o, c in spans) + sum(c // 16 + 1 for c in ctx) + 3, n, 520, 4)
    for i, (off, c) in enumerate(spans):
        if off:
            kv.fill_random(i, off, 5)
        kv.reserve(i, off + c)
    for j, c in enumerate(ctx):
        if c:
            kv.fill_random(len(spans) + j, c, 6)
        kv.reserve(len(spans) + j, c + 1)
    batch = Batch([EmbChunk(i, off, c, False, "none") for i, (off, c) in enumerate(spans)],
                  [DecodeRow(len(spans) + j, c) for j, c in enumerate(ctx)],
                  draw_tokens(8, 0, sum(c for _, c in spans) + len(ctx), cfg.vocab))
    pair = Pair(cfg, W, kv)
    if misaligned:
        for name in ("k", "v"):
            t = getattr(pair.dkv_e, name)
            room = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
            room[1:].copy_(t.reshape(-1))
            setattr(pair.dkv_e, name, room[1:].view(t.shape))
    pair.workspace(batch.n_tokens, len(spans), len(ctx), 301)
    pair.step(batch)
