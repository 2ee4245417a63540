"""The one-launch final norm and pooler against the float64 oracle at the edges of its slices of 8
rows: chunks of 1, 7, 8, 9, 16, 17, 64 and 130 rows under every head, first and resumed, beside
each other and beside logits rows (odd and even counts); rows of 256, 4096 and 6144 columns (the
register forms) and of 8448 (the separate launches); a state that does not match its offset."""
import numpy as np
import pytest
import torch

from tests.parity import Pair
from workload import Batch, DecodeRow, EmbChunk, ModelConfig, PagedKV, draw_token_weights, draw_tokens, make_weights
from paper_2609_25405_amd import _abi as A
from paper_2609_25405_amd import runtime as R

pytestmark = pytest.mark.gpu

HEADS = ["mean", "wmean", "last", "cls", "buffer"]


@pytest.fixture(autouse=True)
def _need_gpu(request):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"\n[case] {request.node.name}", flush=True)


def config(d, dtype):
    return ModelConfig(n_layers=1, d_model=d, n_q_heads=4, n_kv_heads=4, head_dim=64, d_ff=256, vocab=40, dtype=dtype)


@pytest.mark.parametrize("d,dtype,n_dec", [(256, "f32", 1), (256, "bf16", 2), (4096, "bf16", 3), (6144, "f32", 0), (8448, "f32", 2)])
def test_slices(d, dtype, n_dec):
    cfg = config(d, dtype)
    lens = [1, 7, 8, 9, 16, 17, 64, 130]
    kv = PagedKV(cfg, 2 * sum(n // 16 + 2 for n in lens) + 4 * n_dec + 8, len(lens) + n_dec, 20, 3)
    for i, n in enumerate(lens):
        kv.reserve(i, 2 * n)
    for j in range(n_dec):
        kv.fill_random(len(lens) + j, 5 + j, 9)
        kv.reserve(len(lens) + j, 8 + j)
    pair = Pair(cfg, make_weights(cfg, 51), kv)
    pair.workspace(sum(lens) + n_dec, len(lens), n_dec, 16)
    heads = [HEADS[i % len(HEADS)] for i in range(len(lens))]
    for step in range(2):
        batch = Batch([EmbChunk(i, step * n, n, step == 1, heads[i]) for i, n in enumerate(lens)],
                      [DecodeRow(len(lens) + j, 5 + j + step) for j in range(n_dec)],
                      draw_tokens(7, step, sum(lens) + n_dec, cfg.vocab),
                      token_weights=draw_token_weights(7, step, sum(lens)), hidden_stride=300)
        pair.step(batch)


@pytest.mark.parametrize("head,n", [("mean", 5), ("mean", 40), ("last", 40), ("buffer", 40)])
def test_state_mismatch(head, n):
    cfg = config(256, "bf16")
    kv = PagedKV(cfg, 20, 2, 10, 3)
    kv.fill_random(0, 32, 1)
    kv.reserve(0, 32 + n)
    kv.reserve(1, 20)
    dm, dkv = R.DeviceModel(cfg, make_weights(cfg, 51)), R.DeviceKV.from_paged(kv)
    ws = R.Workspace(dm, dm, 80, 2, 1, 64)
    S, W = torch.full((2, 256), 3.0, device="cuda"), torch.tensor([31.0, 0.0], device="cuda")
    out = torch.full((2, 256), float("nan"), device="cuda")
    hidden = torch.zeros((2, 100, 256), device="cuda")
    batch = Batch([EmbChunk(0, 32, n, True, head), EmbChunk(1, 0, 20, True, "mean")], [], draw_tokens(7, 0, n + 20, cfg.vocab),
                  hidden_stride=100)
    R.step(dm, dm, batch, dkv, dkv, S, W, None, out, ws, hidden=hidden)
    torch.cuda.synchronize()
    assert ws.device_error() == A.ORTHRUS_DEVERR_ACC
    assert torch.all(S[0] == 3.0) and W.tolist() == [31.0, 20.0] and torch.isnan(out[0]).all()
    np.testing.assert_allclose(float(out[1].norm()), 1.0, rtol=1e-5)
