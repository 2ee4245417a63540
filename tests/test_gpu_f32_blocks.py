"""The fp32 attention and projection kernels at the edges of their blocks, against the float64
oracle: chunks that end on, before and after a 32-key block and a 32-row wave, a resumed chunk whose
keys pass the staged window of 512 pages, decode rows on both sides of the 64-key pass and of
the 256-key split, projections whose eight K slices hold unequal runs (K = 320) or fewer than one
round (K = 64), and caches whose base is only element-aligned; projections of many outputs on two
tiles a wave, and their cost; a page that is not in the pool; a token whose keys and values are not
numbers, which no earlier row of its chunk may see."""
import pytest
import torch

from tests.parity import Pair
from paper_2609_25405_amd import _abi as A
from paper_2609_25405_amd import runtime as R
from workload import Batch, DecodeRow, EmbChunk, ModelConfig, PagedKV, draw_tokens, make_lora, make_weights

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


@pytest.mark.parametrize("nq,nkv,hd", [(4, 4, 64), (4, 2, 128), (4, 1, 64)])
@pytest.mark.parametrize("offset,n,bad", [(0, 70, 1), (0, 70, 31), (13, 100, 57), (40, 33, 32)])
def test_rows_before_a_token_that_is_not_a_number(nq, nkv, hd, offset, n, bad):
    """Rows before the bad token equal a run in which its row of the table is a number (to the order of
    the fp32 sums: 1e-5, as sums of at most 256 products differ): a masked key's weight is zero, and zero
    times its value must not enter the sum.  It and the rows after it are not numbers."""
    cfg = ModelConfig(n_layers=2, d_model=256, n_q_heads=nq, n_kv_heads=nkv, head_dim=hd, d_ff=128, vocab=32, dtype="f32")
    ids = draw_tokens(9, 0, n, 31)
    ids[bad] = 31
    W = make_weights(cfg, 22)
    hidden = []
    for value in (0.5, float("nan")):
        W["tok_emb"][31] = value
        kv = PagedKV(cfg, 40, 1, 20, 4)
        if offset:
            kv.fill_random(0, offset, 5)
        kv.reserve(0, offset + n)
        dm, dkv = R.DeviceModel(cfg, W), R.DeviceKV.from_paged(kv)
        ws = R.Workspace(dm, dm, n, 1, 0, 1)
        S, Wc = torch.zeros((1, 256), device="cuda"), torch.full((1,), float(offset), device="cuda")
        out, h = torch.zeros((1, 256), device="cuda"), torch.zeros((1, 200, 256), device="cuda")
        batch = Batch([EmbChunk(0, offset, n, True, "buffer")], [], ids, hidden_stride=200)
        R.step(dm, dm, batch, dkv, dkv, S, Wc, None, out, ws, hidden=h)
        torch.cuda.synchronize()
        assert ws.device_error() == 0
        hidden.append(h[0, offset:offset + n])
    clean, got = hidden
    assert torch.isfinite(clean).all()
    assert float((got[:bad] - clean[:bad]).abs().max()) <= 1e-5 * float(clean.abs().max())
    assert torch.isnan(got[bad:]).all()


def test_bad_page():
    """A chunk with a page past the pool: flagged; its rows before the page and the other chunk are as in a run
    with the page in place, its other rows leave the page out."""
    cfg = config(256, 4, 2, 128, 128)
    W = make_weights(cfg, 24)
    results = []
    for bad in (False, True):
        kv = PagedKV(cfg, 20, 2, 8, 4)
        kv.reserve(0, 100)
        kv.reserve(1, 50)
        dm, dkv = R.DeviceModel(cfg, W), R.DeviceKV.from_paged(kv)
        bt = kv.block_table.copy()
        if bad:
            bt[0, 3] = kv.n_pages
        dkv.set_block_table(bt)
        ws = R.Workspace(dm, dm, 150, 2, 0, 1)
        S, Wc = torch.zeros((2, 256), device="cuda"), torch.zeros(2, device="cuda")
        out, h = torch.zeros((2, 256), device="cuda"), torch.zeros((2, 100, 256), device="cuda")
        batch = Batch([EmbChunk(0, 0, 100, True, "buffer"), EmbChunk(1, 0, 50, True, "buffer")], [], draw_tokens(9, 0, 150, 96),
                      hidden_stride=100)
        R.step(dm, dm, batch, dkv, dkv, S, Wc, None, out, ws, hidden=h)
        torch.cuda.synchronize()
        assert ws.device_error() == (A.ORTHRUS_DEVERR_PAGE if bad else 0)
        results.append(h)
    good, got = results
    assert torch.isfinite(got).all()
    assert torch.equal(got[1], good[1]) and torch.equal(got[0, :48], good[0, :48])
    assert not torch.equal(got[0, 48:], good[0, 48:])


# Outputs that fill the chip with two tiles a wave (64 x 64 outputs, 64 x 32 for gate/up), rows and columns
# ending inside a tile: gate/up of 280 rows by 8192 and logits of 250 rows by 4001 with one run of eight k
# a wave (K = 64); o and down of 256 rows by 4096 (K = 64) with an adapter on the first 6 rows, logits with K = 4096
@pytest.mark.parametrize("d,ff,vocab,emb,dec,rank", [(64, 8192, 4001, 30, 250, 0), (4096, 64, 4001, 6, 250, 16), (4096, 64, 4001, 6, 243, 0)])
def test_many_outputs(d, ff, vocab, emb, dec, rank):
    cfg = ModelConfig(n_layers=1, d_model=d, n_q_heads=1, n_kv_heads=1, head_dim=64, d_ff=ff, vocab=vocab, dtype="f32")
    W = make_weights(cfg, 23)
    if rank:
        W["adapters"] = [make_lora(cfg, 5, rank, tag=0)]
    kv = PagedKV(cfg, dec + 4, dec + 1, 2, 4)
    kv.reserve(0, emb)
    for j in range(dec):
        kv.fill_random(1 + j, 1 + j % 14, 6)
        kv.reserve(1 + j, 2 + j % 14)
    batch = Batch([EmbChunk(0, 0, emb, True, "mean")], [DecodeRow(1 + j, 1 + j % 14) for j in range(dec)],
                  draw_tokens(8, 0, emb + dec, vocab), chunk_adapter=[0] if rank else None)
    pair = Pair(cfg, W, kv)
    pair.workspace(batch.n_tokens, 1, dec, 20)
    pair.step(batch)


def test_many_outputs_cost():
    """Logits of 256 rows through a 32000 x 4096 head take at most six times those of 32 (4.5 measured; 7.8 on
    one tile a wave, whose loads bound it)."""
    cfg = ModelConfig(n_layers=0, d_model=4096, n_q_heads=1, n_kv_heads=1, head_dim=64, d_ff=64, vocab=32000, dtype="f32")
    W = {"tok_emb": torch.randn(32000, 4096, device="cuda") * 0.02, "lm_head": torch.randn(32000, 4096, device="cuda") * 0.02,
         "final_norm": torch.ones(4096, device="cuda"), "layers": []}
    dm = R.DeviceModel(cfg, W)
    times = []
    for rows in (32, 256):
        kv = PagedKV(cfg, rows + 2, rows, 1, 4)
        for j in range(rows):
            kv.reserve(j, 1)
        dkv = R.DeviceKV.from_paged(kv)
        ws = R.Workspace(dm, dm, rows, 0, rows, 1)
        logits = torch.empty((rows, 32000), device="cuda")
        batch = Batch([], [DecodeRow(j, 0) for j in range(rows)], draw_tokens(8, 0, rows, 32000))
        best = 1e9
        for _ in range(6):
            R.profile_begin(dm)
            R.step(dm, dm, batch, dkv, dkv, None, None, logits, None, ws)
            torch.cuda.synchronize()
            best = min(best, R.profile_end(dm)["lm_head"][1])
        times.append(best)
    print(f"32 rows {times[0] * 1e3:.0f} us, 256 rows {times[1] * 1e3:.0f} us", flush=True)
    assert times[1] <= 6 * times[0]
