"""The one-launch final norm and pooler against the float64 oracle at the edges of its slices of 8
rows: chunks of 1, 7, 8, 9, 16, 17, 64 and 130 rows under every head, first and resumed, beside
each other and beside logits rows (odd and even counts); rows of 256, 4096 and 6144 columns (the
register forms) and of 8448 (the separate launches); a state that does not match its offset; chunks
of very uneven lengths (blocks found by search over 1, 2 and more steps of 64 chunks, a block of the
slices' sum taking several chunks), and their cost."""
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


def uneven(lens, heads, d=256):
    cfg = config(d, "bf16")
    kv = PagedKV(cfg, sum(n // 16 + 1 for n in lens) + 2, len(lens), max(lens) // 16 + 1, 3)
    for i, n in enumerate(lens):
        kv.reserve(i, n)
    batch = Batch([EmbChunk(i, 0, n, True, h) for i, (n, h) in enumerate(zip(lens, heads))], [], draw_tokens(7, 0, sum(lens), cfg.vocab),
                  token_weights=draw_token_weights(7, 0, sum(lens)), hidden_stride=max(lens))
    return cfg, kv, batch


@pytest.mark.parametrize("lens,heads", [
    ([300, 1], ["mean"]), ([1] * 70 + [200] + [9, 8, 1] * 20, ["mean"]), ([1] * 70 + [200] + [9, 8, 1] * 20, HEADS),
    ([17] * 65, ["wmean"]), ([1] * 2000 + [100] + [1] * 2200, ["mean"])],
    ids=["two", "131-mean", "131-heads", "65-long", "4201"])
def test_uneven_chunks(lens, heads):
    cfg, kv, batch = uneven(lens, [heads[i % len(heads)] for i in range(len(lens))])
    pair = Pair(cfg, make_weights(cfg, 51), kv)
    pair.workspace(sum(lens), len(lens), 0, 16)
    pair.step(batch)


@pytest.mark.parametrize("d", [2048, 6144])
def test_uneven_chunks_cost_what_their_rows_do(d):
    """One chunk of 1024 rows beside 1024 chunks of one row, against the same rows in 128 equal chunks: the
    launch takes at most four times as long (1.8 measured; 30 with a block per chunk and slice of
    the longest)."""
    times = []
    for lens in ([16] * 128, [1024] + [1] * 1024):
        cfg, kv, batch = uneven(lens, ["mean"] * len(lens), d)
        dm, dkv = R.DeviceModel(cfg, make_weights(cfg, 51)), R.DeviceKV.from_paged(kv)
        ws = R.Workspace(dm, dm, sum(lens), len(lens), 0, 16)
        S, W = torch.zeros((len(lens), d), device="cuda"), torch.zeros(len(lens), device="cuda")
        out = torch.zeros((len(lens), d), device="cuda")
        best = 1e9
        for _ in range(6):
            R.profile_begin(dm)
            R.step(dm, dm, batch, dkv, dkv, S, W, None, out, ws)
            torch.cuda.synchronize()
            best = min(best, R.profile_end(dm)["final_norm_pool"][1])
        times.append(best)
        print(f"{len(lens)} chunks: {best * 1e3:.1f} us", flush=True)
    assert times[1] <= 4 * times[0]
