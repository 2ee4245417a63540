"""Projections of more than 128 rows (the large kernel's tile shapes) against the float64 oracle, at
row counts on and beside the edges of its tiles: one row past the smallest batch it takes, row
counts that its covers give to 64-, 128- and 192-row tiles, a last row tile of one row, of exactly
64, 128 and of 129 rows, whole tiles, and enough rows for several rounds; with LoRA adapters on part of the rows (ranks 16 and 48,
so that a 32-column step of the update ends inside and past an adapter's block)."""
import numpy as np
import pytest
import torch

from tests.parity import Pair
from workload import Batch, DecodeRow, EmbChunk, ModelConfig, PagedKV, draw_tokens, make_lora, make_weights

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _need_gpu(request):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"\n[case] {request.node.name}", flush=True)


# (rows, rank, d_ff): the wide MLPs have enough column tiles for the two-shape covers (last rows on 128-
# and 64-row tiles, last columns on 192-wide ones)
@pytest.mark.parametrize("rows,rank,ff", [
    (129, 0, 2816), (193, 16, 2816), (257, 0, 2816), (449, 48, 2816), (640, 0, 2816), (832, 0, 2816),
    (897, 0, 2816), (1025, 0, 2816), (1088, 0, 2816), (1152, 16, 2816), (1281, 48, 2816), (1536, 0, 2816),
    (2049, 0, 2816), (300, 0, 28672), (700, 16, 28672), (1025, 0, 28672), (1100, 48, 28672)])
def test_rows(rows, rank, ff):
    cfg = ModelConfig(n_layers=1, d_model=512, n_q_heads=8, n_kv_heads=2, head_dim=128, d_ff=ff, vocab=512,
                      dtype="bf16")
    W = make_weights(cfg, 11)
    if rank:
        W["adapters"] = [make_lora(cfg, 5, rank, tag=i) for i in range(2)]
    n_dec = 3
    lens, left = [], rows - n_dec
    while left:
        lens.append(min(left, 300))
        left -= lens[-1]
    kv = PagedKV(cfg, sum(-(-n // 16) for n in lens) + n_dec * 8 + 4, len(lens) + n_dec, 20, 3)
    for i, n in enumerate(lens):
        kv.reserve(i, n)
    for j in range(n_dec):
        kv.fill_random(len(lens) + j, 40 + j, 9)
        kv.reserve(len(lens) + j, 41 + j)
    batch = Batch([EmbChunk(i, 0, n, True, "mean") for i, n in enumerate(lens)],
                  [DecodeRow(len(lens) + j, 40 + j) for j in range(n_dec)], draw_tokens(7, 0, rows, cfg.vocab),
                  chunk_adapter=[(i % 3) - 1 for i in range(len(lens))] if rank else None)
    pair = Pair(cfg, W, kv)
    pair.workspace(rows, len(lens), n_dec, 64)
    pair.step(batch)
