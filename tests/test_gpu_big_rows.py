"""Projections of more than 128 rows (the large kernel's tile shapes) against the float64 oracle, at
row counts on and beside the edges of its tiles: one row past the smallest batch it takes, row
counts that its covers give to 64-, 128- and 192-row tiles, a last row tile of one row, of exactly
64, 128 and of 129 rows, whole tiles, and enough rows for several rounds; with LoRA adapters on part of the rows (ranks 16 and 48,
so that a 32-column step of the update ends inside and past an adapter's block).  Each case names the K splits
and covers that its four projections take, every cover of the kernel among them: a change of the rules
that loses one shows here.  Beside another model's launches, gate/up where it leaves the large kernel."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2609_25405_amd as P
from tests.parity import Pair
from tests.test_covers import covers
from workload import Batch, DecodeRow, EmbChunk, ModelConfig, PagedKV, draw_tokens, make_lora, make_weights

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _need_gpu(request):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"\n[case] {request.node.name}", flush=True)


# rows, rank, d_model, d_ff, then (K splits, cover) of QKV, o, gate/up and down: the wide MLPs have enough
# column tiles for the two-shape covers (last rows on 128- and 64-row tiles, last columns on 192- and 128-wide
# ones), the 4096-wide models (16 query, 4 key/value heads; 7B-class at qkv 6144) for those with split K
@pytest.mark.parametrize("rows,rank,d,ff,taken", [
    (129, 0, 512, 2816, "1:10 2:10 1:10 4:10"), (193, 16, 512, 2816, "1:10 2:10 1:10 4:10"),
    (257, 0, 512, 2816, "1:10 2:10 1:10 4:10"), (449, 48, 512, 2816, "1:10 2:10 1:8 4:10"),
    (640, 0, 512, 2816, "1:10 2:10 1:8 4:10"), (832, 0, 512, 2816, "1:10 2:10 1:6 4:10"),
    (897, 0, 512, 2816, "1:10 2:10 1:6 4:10"), (1025, 0, 512, 2816, "1:10 2:10 1:3 4:8"),
    (1088, 0, 512, 2816, "1:10 2:10 1:3 4:8"), (1152, 16, 512, 2816, "1:10 2:10 1:3 4:8"),
    (1281, 48, 512, 2816, "1:10 2:10 1:7 4:8"), (1536, 0, 512, 2816, "1:8 2:10 1:5 4:8"),
    (2049, 0, 512, 2816, "1:8 2:8 1:4 4:6"), (300, 0, 512, 28672, "1:10 2:10 1:11 4:10"),
    (700, 16, 512, 28672, "1:10 2:10 1:2 4:10"), (1025, 0, 512, 28672, "1:10 2:10 1:11 4:8"),
    (1100, 48, 512, 28672, "1:10 2:10 1:1 4:8"), (1024, 0, 512, 8192, "1:10 2:10 1:0 4:10"),
    (288, 16, 4096, 512, "2:9 4:6 1:10 1:10"), (512, 48, 4096, 512, "2:3 4:3 1:10 1:10")])
def test_rows(rows, rank, d, ff, taken):
    nq, nkv = (8, 2) if d == 512 else (32, 8)
    plan_big, add_splits, qkv_splits = covers()
    got = []
    for N, K, sw, splits in (((nq + 2 * nkv) * 128, d, False, qkv_splits(rows, (nq + 2 * nkv) * 128, d, False)),
                             (d, nq * 128, False, add_splits(rows, d, nq * 128, 4, False)), (ff, d, True, 1),
                             (d, ff, False, add_splits(rows, d, ff, 4, False))):
        got.append(f"{splits}:{plan_big(rows, N, K, sw, splits, False).shape}")
    assert " ".join(got) == taken
    cfg = ModelConfig(n_layers=1, d_model=d, n_q_heads=nq, n_kv_heads=nkv, head_dim=128, d_ff=ff, vocab=512, dtype="bf16")
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


@pytest.mark.parametrize("rows,rank", [(257, 0), (384, 48), (513, 16), (768, 0)])
def test_rows_beside_a_model(rows, rank):
    """A step of two models whose embedding rows' gate/up takes 192x256 tiles beside the generator's launches: rows
    ending inside a tile and at its end, adapters."""
    on_192 = P.load()["_ZN7orthrus14gate_up_on_192Eiii"]
    on_192.restype, on_192.argtypes = ctypes.c_bool, [ctypes.c_int] * 3
    ff = 14080
    assert on_192(rows, ff, 512)
    cfg = ModelConfig(n_layers=1, d_model=512, n_q_heads=8, n_kv_heads=2, head_dim=128, d_ff=ff, vocab=512, dtype="bf16")
    W, G = make_weights(cfg, 11, model_tag=1), make_weights(cfg, 12, model_tag=2)
    if rank:
        W["adapters"] = [make_lora(cfg, 5, rank, tag=i) for i in range(2)]
    kv, gkv = PagedKV(cfg, rows // 16 + 4, 2, 64, 3), PagedKV(cfg, 12, 3, 4, 4)
    lens = [rows // 2, rows - rows // 2]
    for j, n in enumerate(lens):
        kv.reserve(j, n)
    for j in range(3):
        gkv.fill_random(j, 9 + 16 * j, 5)
        gkv.reserve(j, 10 + 16 * j)
    batch = Batch([EmbChunk(j, 0, n, True, "mean") for j, n in enumerate(lens)], [DecodeRow(j, 9 + 16 * j) for j in range(3)],
                  draw_tokens(8, 0, rows + 3, cfg.vocab), chunk_adapter=[1, -1] if rank else None)
    pair = Pair(cfg, W, kv, cfg, G, gkv)
    pair.workspace(rows + 3, 2, 3, 60)
    pair.step(batch)
