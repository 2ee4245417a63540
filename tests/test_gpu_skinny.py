"""Steps of at most 16 rows per model through small weights (the projections of gemm_skinny.hip) against
the float64 oracle: 1, 4, 5, 16 rows and, past the rule, 17; head_dim 64 and 128 (two and four
16-dim parts of a rotation half); K that is not a multiple of the waves' 32-deep steps (768) and deep
enough for several rounds of loads (2816); rows the launch norms itself and rows normed before it
(16 rows of a 2048-wide model); prompt rows, embedding rows and decode rows together; a vocabulary
that ends inside a set of 16; two models."""
import pytest
import torch

from tests.parity import Pair
from workload import Batch, DecodeRow, EmbChunk, GenChunk, ModelConfig, PagedKV, draw_tokens, make_weights

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _need_gpu(request):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"\n[case] {request.node.name}", flush=True)


def config(d, nq, nkv, hd, ff, vocab=100):
    return ModelConfig(n_layers=2, d_model=d, n_q_heads=nq, n_kv_heads=nkv, head_dim=hd, d_ff=ff, vocab=vocab, dtype="bf16")


NARROW = config(512, 8, 2, 128, 2816)
ODD = config(768, 12, 12, 64, 768)
WIDE = config(2048, 4, 2, 128, 512)


@pytest.mark.parametrize("cfg,emb,prompt,rows,two", [
    (NARROW, 0, 0, 1, False), (NARROW, 0, 0, 4, False), (NARROW, 7, 4, 5, False), (NARROW, 0, 0, 17, False),
    (ODD, 1, 2, 2, False), (ODD, 6, 0, 10, True), (WIDE, 0, 0, 4, False), (WIDE, 3, 3, 10, False)])
def test_few_rows(cfg, emb, prompt, rows, two):
    W = make_weights(cfg, 31, model_tag=1)
    n0 = (1 if emb else 0)
    n = n0 + (1 if prompt else 0) + rows
    kv = PagedKV(cfg, n * 12 + 4, n, 12, 8)
    gkv = PagedKV(cfg, n * 12 + 4, n, 12, 9) if two else kv
    if emb:
        kv.reserve(0, emb)
    if prompt:
        gkv.fill_random(n0, 21, 3)
        gkv.reserve(n0, 21 + prompt)
    ctx = [(j * 37) % 150 for j in range(rows)]
    first = n - rows
    for j, c in enumerate(ctx):
        if c:
            gkv.fill_random(first + j, c, 4)
        gkv.reserve(first + j, c + 1)
    batch = Batch([EmbChunk(0, 0, emb, True, "mean")] if emb else [], [DecodeRow(first + j, c) for j, c in enumerate(ctx)],
                  draw_tokens(6, 0, emb + prompt + rows, cfg.vocab),
                  gen_chunks=[GenChunk(n0, 21, prompt, True)] if prompt else [])
    pair = Pair(cfg, W, kv, cfg, make_weights(cfg, 32, model_tag=2), gkv) if two else Pair(cfg, W, kv)
    pair.workspace(emb + prompt + rows, 2, rows, 151)
    pair.step(batch)
