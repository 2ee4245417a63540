"""Steps of at most 16 rows per model through small weights (the projections of gemm_skinny.hip) against
the float64 oracle: 1, 4, 5, 16 rows and, past the rule, 17; QKV alone of 17 to 128 rows (tiles of 16: a last tile of
one row, whole ones, pools and models that change inside one; rows it norms itself) and past its rule; head_dim 64 and 128 (two and four
16-dim parts of a rotation half); K that does not divide over the eight waves (768); K of several rounds of
loads, ending inside one (down of 4864: 19 steps a wave, two rounds of 16; QKV of 2304: 9); rows normed in the launch (K
of 256 to 1024: one to four steps a wave, up to 8192 values in all), with the gather (layer 0), and by a launch of
their own (past that, and before gate/up where an o projection whose weights are too large leaves partial sums); prompt rows,
embedding rows and decode rows together; a vocabulary that ends inside a set of 16; two models; a
row whose page is not in the pool."""
import pytest
import torch

from paper_2609_25405_amd import _abi as A
from paper_2609_25405_amd import runtime as R
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
DEEP = config(512, 8, 2, 128, 4864)
WIDEST = config(2304, 2, 1, 128, 256)
NORMED = config(1024, 4, 2, 128, 512)
SMALL = config(256, 4, 4, 64, 512)
LARGE_O = config(512, 64, 16, 128, 256)     # o: 8 MB of weights, too much for more than 4 rows


@pytest.mark.parametrize("cfg,emb,prompt,rows,two", [
    (NARROW, 0, 0, 1, False), (NARROW, 0, 0, 4, False), (NARROW, 7, 4, 5, False), (NARROW, 0, 0, 17, False),
    (ODD, 1, 2, 2, False), (ODD, 6, 0, 10, True), (WIDE, 0, 0, 4, False), (WIDE, 3, 3, 10, False),
    (DEEP, 0, 0, 4, False), (DEEP, 1, 0, 2, False), (WIDEST, 0, 0, 3, False), (WIDEST, 3, 2, 2, False),
    (LARGE_O, 0, 0, 7, False), (NARROW, 0, 0, 33, False), (NARROW, 30, 50, 48, False), (NARROW, 0, 0, 129, False),
    (ODD, 20, 10, 11, False), (ODD, 70, 5, 31, True), (ODD, 17, 0, 64, True), (NORMED, 0, 0, 8, False),
    (NORMED, 3, 2, 4, True), (NORMED, 0, 0, 9, False), (SMALL, 0, 0, 16, False), (SMALL, 5, 3, 40, False)])
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


@pytest.mark.parametrize("ahead", [0, 17])
def test_bad_page(ahead):
    """The launch that appends flags the row whose page is past the pool and writes nothing for it; the other
    rows and every other slot are as in a run with its page in place."""
    cfg = NARROW
    W = make_weights(cfg, 31)
    ctx = [7] * ahead + [40, 33, 7]
    n, row = len(ctx), ahead + 1
    results = []
    for bad in (False, True):
        kv = PagedKV(cfg, 20 + ahead, n, 4, 8)
        for j, c in enumerate(ctx):
            kv.fill_random(j, c, 4)
            kv.reserve(j, c + 1)
        dm, dkv = R.DeviceModel(cfg, W), R.DeviceKV.from_paged(kv)
        bt = kv.block_table.copy()
        own = int(bt[row, 2])
        if bad:
            bt[row, 2] = kv.n_pages
        dkv.set_block_table(bt)
        before = [dkv.k.clone(), dkv.v.clone()]
        ws = R.Workspace(dm, dm, n, 0, n, 64)
        logits = torch.zeros((n, cfg.vocab), device="cuda")
        R.step(dm, dm, Batch([], [DecodeRow(j, c) for j, c in enumerate(ctx)], draw_tokens(6, 0, n, cfg.vocab)), dkv, dkv, None, None,
               logits, None, ws)
        torch.cuda.synchronize()
        assert ws.device_error() == (A.ORTHRUS_DEVERR_PAGE if bad else 0)
        results.append((logits, dkv.k, dkv.v, before))
    (good_l, good_k, good_v, _), (bad_l, bad_k, bad_v, before) = results
    assert torch.isfinite(bad_l).all()
    others_l = [j for j in range(n) if j != row]
    assert torch.equal(good_l[others_l], bad_l[others_l])
    bits = lambda t: t.view(torch.int16)
    others = [pg for pg in range(good_k.shape[1]) if pg != own]
    assert torch.equal(bits(good_k[:, others]), bits(bad_k[:, others])) and torch.equal(bits(good_v[:, others]), bits(bad_v[:, others]))
    assert torch.equal(bits(before[0][:, own]), bits(bad_k[:, own])) and torch.equal(bits(before[1][:, own]), bits(bad_v[:, own]))


@pytest.mark.parametrize("rows", [17, 128])
def test_rotation_is_no_launch_of_its_own(rows):
    cfg = NARROW
    kv = PagedKV(cfg, rows + 2, rows, 1, 8)
    for j in range(rows):
        kv.reserve(j, 1)
    dm, dkv = R.DeviceModel(cfg, make_weights(cfg, 31)), R.DeviceKV.from_paged(kv)
    ws = R.Workspace(dm, dm, rows, 0, rows, 2)
    R.profile_begin(dm)
    R.step(dm, dm, Batch([], [DecodeRow(j, 0) for j in range(rows)], draw_tokens(6, 0, rows, cfg.vocab)), dkv, dkv, None, None,
           torch.zeros((rows, cfg.vocab), device="cuda"), None, ws)
    torch.cuda.synchronize()
    names = R.profile_end(dm)
    assert "gemm_qkv_rope" in names and "rope_append" not in names, names


@pytest.mark.parametrize("cfg,rows,launches", [(NARROW, 4, 1), (NARROW, 16, 3), (NORMED, 8, 1), (NORMED, 9, 4), (WIDE, 1, 4)])
def test_norms_in_the_launch_where_rows_are_short(cfg, rows, launches):
    """Launches of norms in two layers and after them: the gather's alone where the projections norm their rows
    (gate and up of 16 rows of the 512-wide model are too large)."""
    kv = PagedKV(cfg, rows + 2, rows, 1, 8)
    for j in range(rows):
        kv.reserve(j, 1)
    dm, dkv = R.DeviceModel(cfg, make_weights(cfg, 31)), R.DeviceKV.from_paged(kv)
    ws = R.Workspace(dm, dm, rows, 0, rows, 2)
    R.profile_begin(dm)
    R.step(dm, dm, Batch([], [DecodeRow(j, 0) for j in range(rows)], draw_tokens(6, 0, rows, cfg.vocab)), dkv, dkv, None, None,
           torch.zeros((rows, cfg.vocab), device="cuda"), None, ws)
    torch.cuda.synchronize()
    names = R.profile_end(dm)
    assert sum(names[n][0] for n in names if "rmsnorm" in n or n == "gather_norm") == launches, names
