"""Decode launches of few work items with long key runs (sixteen waves an item, 256 keys a chunk) against
the float64 oracle: contexts on both sides of a 16-key page, of the 256-key chunk, of a split, and
of the length from which a launch takes this form; every supported query group."""
import pytest
import torch

from tests.parity import Pair
from workload import Batch, DecodeRow, ModelConfig, PagedKV, draw_tokens, make_weights

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _need_gpu(request):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"\n[case] {request.node.name}", flush=True)


@pytest.mark.parametrize("nq,nkv,hd", [(8, 2, 128), (4, 2, 128), (4, 4, 64)])
@pytest.mark.parametrize("ctx", [[383], [384, 0, 15, 16], [255, 256, 511, 512, 700], [1023, 1024, 1500, 2303]])
def test_contexts(nq, nkv, hd, ctx):
    cfg = ModelConfig(n_layers=1, d_model=512, n_q_heads=nq, n_kv_heads=nkv, head_dim=hd, d_ff=512, vocab=64, dtype="bf16")
    kv = PagedKV(cfg, sum(c // 16 + 1 for c in ctx) + 2, len(ctx), 160, 4)
    for j, c in enumerate(ctx):
        if c:
            kv.fill_random(j, c, 6)
        kv.reserve(j, c + 1)
    batch = Batch([], [DecodeRow(j, c) for j, c in enumerate(ctx)], draw_tokens(8, 0, len(ctx), cfg.vocab))
    pair = Pair(cfg, make_weights(cfg, 41), kv)
    pair.workspace(len(ctx), 1, len(ctx), 2400)
    pair.step(batch)
