"""Prefill of more than 16 tokens runs the many-row kernels; up to 16 it runs
the verify passes' kernels, which the oracle tests cover.  Both must leave the
same bits: a prompt taken at once against the same prompt taken in pieces of
at most 16 tokens, on the pages of a permuted pool, compared on the logits, the
next token and the whole KV pool."""
import ctypes

import numpy as np
import pytest

import lede_inputs as li
from lede_inputs.configs import TINY, shrink
from tests import wide_host
from tests.parity import say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BF16_64 = shrink(TINY, name="bf16-hd64", dtype="bf16")
BF16_128 = shrink(TINY, name="bf16-hd128", n_layers=3, d_model=512, n_heads=4, n_kv_heads=4, head_dim=128,
                  ffn_dim=1376, vocab=4096, dtype="bf16", qnet_hidden=64, exits=(1, 2, 3))
GQA_64 = shrink(TINY, name="bf16-gqa-hd64", n_layers=2, d_model=544, n_heads=6, n_kv_heads=2, head_dim=64,
                ffn_dim=1000, vocab=2048, dtype="bf16", qnet_hidden=32, exits=(1, 2))
GQA_128_F32 = shrink(TINY, name="f32-gqa-hd128", n_layers=2, d_model=512, n_heads=8, n_kv_heads=2, head_dim=128,
                     ffn_dim=704, vocab=1024, dtype="f32", qnet_hidden=32, exits=(1, 2))
GQA_8 = shrink(TINY, name="bf16-gqa8-hd128", n_layers=1, d_model=1024, n_heads=16, n_kv_heads=2, head_dim=128,
               ffn_dim=1376, vocab=1024, dtype="bf16", qnet_hidden=32, exits=(1,))
GQA_64_F = shrink(GQA_64, name="bf16-gqa-hd64-f1024", ffn_dim=1024)
MODELS = [TINY, BF16_64, BF16_128, GQA_64, GQA_128_F32, GQA_8]
# (tokens already cached, new tokens): one past a group, edges of row tiles and
# pages, ragged ends, several page groups behind the rows
SIZES = [(0, 17), (0, 64), (5, 65), (30, 127), (0, 129), (70, 300)]


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    return wide_host.load(tmp_path_factory.mktemp("wide_host"))


def _shapes(host, m, n):
    """Output tiles of n rows' linear kernels: QKV, output projection and down,
    gate-up (0: k_wide; 1 to 4: k_wide_lds of 128 x 64, 64 x 64, 96 x 128, 128 x 128)."""
    dt = int(m.dtype == "bf16")
    return tuple(host.linear_shape(dt, g // 16, n) for g in (m.q_dim + 2 * m.kv_dim, m.d_model, 2 * m.ffn_dim))


def _split(host, m, max_ctx, ctx, n):
    """How the attention of n rows behind ctx positions is split (0: not, 1:
    partials of pages, 2: of the combine's groups), mode 1's pages per block,
    and where the partials lie (0: the 16-row passes', 1: the normalised rows',
    2: the activations' region)."""
    pages, at = ctypes.c_int(), ctypes.c_int()
    mode = host.attn_split(m.n_heads, m.n_kv_heads, m.head_dim, m.d_model, m.ffn_dim, max_ctx, n, ctx + n,
                           ctypes.byref(pages), ctypes.byref(at))
    return mode, pages.value if mode == 1 else 0, at.value if mode else None


def _state(eng):
    sl, pend, table = eng.lede_get_kv_state()
    return sl, pend, table, eng.kv.cpu().numpy(), eng.logits(0)


def _engine(model, max_ctx, seed):
    from paper_2606_03113_amd import Engine
    eng = Engine(model, max_ctx=max_ctx, k_max=8)
    eng.kv.fill_(0xFF)  # NaNs in every slot that has not been written
    eng.load_weights(li.weights(model), li.qnet_weights(model))
    eng.lede_set_options(0, 1)
    eng.lede_set_free_list(np.random.default_rng(seed).permutation(-(-max_ctx // 64)))
    return eng


def _check(model, max_ctx, ctx, n, piece=16):
    toks = li.uniform_int(1, 20, ctx + n, 0, model.vocab - 1)
    got = []
    for step in (n, piece):
        eng = _engine(model, max_ctx, ctx + n)
        for i in range(0, ctx, piece):
            eng.lede_prefill(toks[i:min(ctx, i + piece)])
        for i in range(ctx, ctx + n, step):
            eng.lede_prefill(toks[i:min(ctx + n, i + step)])
        got.append(_state(eng))
        eng.close()
    (sl, pend, table, kv, z), (sl2, pend2, table2, kv2, z2) = got
    assert (sl, pend, table) == (sl2, pend2, table2)
    assert np.isfinite(z).all() and np.array_equal(z, z2)
    assert np.array_equal(kv, kv2)


@pytest.mark.parametrize("ctx,n", SIZES)
@pytest.mark.parametrize("model", MODELS, ids=lambda m: m.name)
def test_prefill_at_once_equals_pieces(model, ctx, n):
    say("wide prefill", model.name, ctx, n)
    _check(model, 448, ctx, n)


@pytest.mark.parametrize("model", [BF16_64, GQA_64, TINY], ids=lambda m: m.name)
def test_prefill_of_several_passes(model):
    """More rows than one pass takes, ending in a ragged pass."""
    say("wide prefill, several passes", model.name)
    _check(model, 2400, 40, 2201)


# every staged kernel with every epilogue, widths and row counts that end
# inside a tile
STAGED = shrink(TINY, name="bf16-staged", n_layers=1, d_model=4064, n_heads=33, n_kv_heads=11, head_dim=64,
                ffn_dim=2008, vocab=512, dtype="bf16", qnet_hidden=32, exits=(1,))
STAGED_F32 = shrink(STAGED, name="f32-staged", d_model=2080, n_heads=11, n_kv_heads=11, ffn_dim=1048, dtype="f32")


@pytest.mark.parametrize("model,n,shape", [(STAGED, 947, 1), (STAGED, 441, 2), (STAGED, 1299, 3), (STAGED, 1793, 4),
                                           (STAGED_F32, 1250, 1)], ids=lambda v: getattr(v, "name", v))
def test_prefill_staged_kernels(host, model, n, shape):
    assert _shapes(host, model, n) == (shape, shape, shape)
    say("wide prefill, staged kernel", shape, model.name, n)
    _check(model, 1856, 0, n)


@pytest.mark.parametrize("model,n,split", [(GQA_64, 400, (0, 0, None)), (GQA_64, 130, (2, 0, 0)), (GQA_64_F, 130, (2, 0, 2))],
                         ids=lambda v: getattr(v, "name", v))
def test_prefill_past_128_pages(host, model, n, split):
    """Contexts longer than one round of the page combine's eight groups,
    walked by one block per row block, and split over the groups."""
    assert _split(host, model, 8640, 8190, n) == split
    say("wide prefill, 128 pages", model.name, n)
    _check(shrink(model, n_layers=1, exits=(1,)), 8640, 8190, n)


@pytest.mark.parametrize("model,ctx,n,split", [(GQA_8, 1300, 30, (1, 1, 2)), (GQA_8, 2130, 130, (2, 0, 2)),
                                               (BF16_128, 1980, 17, (1, 1, 2)), (GQA_64_F, 1500, 260, (2, 0, 2)),
                                               (GQA_64, 1500, 130, (2, 0, 1)), (GQA_64, 2000, 17, (1, 1, 1))],
                         ids=lambda v: getattr(v, "name", v))
def test_prefill_behind_many_pages(host, model, ctx, n, split):
    """Few rows behind many pages: the pages are split over blocks, with
    partials of pages or of the combine's groups, in the activations' region or,
    where the feed-forward width leaves a tile partly empty, another."""
    assert _split(host, model, 2400, ctx, n) == split
    say("wide prefill, many pages", model.name, ctx, n)
    _check(model, 2400, ctx, n)


@pytest.mark.parametrize("ctx,n,split", [(33, 40, (0, 0, None)), (33, 200, (0, 0, None)), (1000, 40, (1, 3, 2))])
def test_prefill_at_full_width(host, ctx, n, split):
    """One layer at the Llama-2-7B widths (the last with blocks of three pages)."""
    from lede_inputs.configs import WORKLOADS
    m = shrink(WORKLOADS["llama2-7b"].model, n_layers=1, exits=(1,))
    assert _split(host, m, 512 if ctx < 512 else 1100, ctx, n) == split
    say("wide prefill, 7B widths", ctx, n)
    _check(m, 512 if ctx < 512 else 1100, ctx, n)


# widths of a single K tile (32 bf16 or 16 fp32 columns), with enough rows and
# columns for the staged kernel: gate-up, then down, with the tile full and
# partly filled
K1 = dict(n_layers=2, n_heads=2, n_kv_heads=1, head_dim=64, vocab=512, qnet_hidden=32, exits=(1, 2))
K1_MODELS = [(shrink(TINY, name="bf16-d32", d_model=32, ffn_dim=1376, dtype="bf16", **K1), 600),
             (shrink(TINY, name="bf16-f32", d_model=4096, ffn_dim=32, dtype="bf16", **K1), 420),
             (shrink(TINY, name="bf16-f8", d_model=4096, ffn_dim=8, dtype="bf16", **K1), 420),
             (shrink(TINY, name="f32-f16", d_model=4096, ffn_dim=16, dtype="f32", **K1), 700)]


@pytest.mark.parametrize("model,n", K1_MODELS, ids=lambda v: getattr(v, "name", v))
def test_prefill_of_one_k_tile(host, model, n):
    assert _shapes(host, model, n)[2 if model.d_model == 32 else 1] > 0
    say("wide prefill, one K tile", model.name, n)
    _check(model, 768, 0, n)


@pytest.mark.parametrize("heads,n,split", [(2, 40, 1), (32, 60, 0)], ids=["split", "unsplit"])
def test_page_of_overflowed_scores(host, heads, n, split):
    """Cached keys so large that every score of a page overflows to -inf: the
    page has no weight, as in the 16-row kernels.  Every query has a large
    element in a slowly rotating dimension, in which the second page's keys
    hold -3e38."""
    from paper_2606_03113_amd import Engine
    hd, ctx = 64, 128
    m = shrink(TINY, name="overflow", n_layers=2, n_heads=heads, n_kv_heads=1, head_dim=hd, ffn_dim=256, dtype="bf16",
               qnet_hidden=32, exits=(1, 2))
    assert _split(host, m, 256, ctx, n)[0] == split
    bf16 = lambda x: int(np.float32(x).view(np.uint32) >> 16)  # noqa: E731
    w = li.weights(m)
    w["embed"][:, 0] = bf16(0.08)
    for layer in w["layers"]:
        layer["wq"][hd // 2 - 1::hd, 0] = bf16(60.0)
    toks = li.uniform_int(1, 20, ctx + n, 0, m.vocab - 1)
    got = []
    for step in (n, 16):
        say("wide prefill, overflowed scores", heads, step)
        eng = Engine(m, max_ctx=256, k_max=8)
        eng.kv.zero_()
        eng.load_weights(w, li.qnet_weights(m))
        eng.lede_set_options(0, 1)
        eng.lede_prefill(toks[:ctx])
        page = eng.lede_get_kv_state()[2][1]
        keys = eng.kv[:eng.region_bytes[1] // 2].view(torch.int16)[:2 * eng.cfg.n_pages * 64 * hd].view(2, -1, 64, hd)
        keys[0, page] = 0
        keys[0, page, :, hd // 2 - 1] = bf16(-3e38) - (1 << 16)
        torch.cuda.synchronize()
        for i in range(ctx, ctx + n, step):
            eng.lede_prefill(toks[i:min(ctx + n, i + step)])
        got.append(_state(eng))
        eng.close()
    assert np.isfinite(got[1][4]).all()
    assert np.array_equal(got[0][4], got[1][4]) and np.array_equal(got[0][3], got[1][3])


# query heads, cached, new tokens, the bad one, rows before it that must be
# clean, and how the pages are split: a token in a later group of 16 rows than
# the clean ones; and one in the same group, which crosses a page, with the
# clean rows on the page before
@pytest.mark.parametrize("heads,ctx,n,bad,clean,split", [(2, 0, 100, 57, 48, 0), (2, 52, 40, 66, 64, 0), (2, 128, 40, 153, 144, 1),
                                                         (2, 180, 40, 194, 192, 1), (8, 1972, 40, 1986, 1984, 2)])
def test_overflowed_value_stays_with_its_rows(host, heads, ctx, n, bad, clean, split):
    """A token whose value overflows to infinity: the rows that do not see it,
    of earlier groups of 16 in its page and of earlier pages in its group, keep
    the bits they have in 16-row passes (a weight of 0 would make infinity a
    NaN)."""
    from paper_2606_03113_amd import Engine
    max_ctx = 2048 if ctx > 256 else 256
    m = shrink(TINY, name="overflow-v", n_layers=2, n_heads=heads, n_kv_heads=1, head_dim=64, ffn_dim=256, dtype="bf16",
               qnet_hidden=32, exits=(1, 2))
    assert _split(host, m, max_ctx, ctx, n)[0] == split
    bf16 = lambda x: int(np.float32(x).view(np.uint32) >> 16)  # noqa: E731
    toks = li.uniform_int(1, 20, ctx + n, 0, m.vocab - 2)
    toks[bad] = m.vocab - 1
    w = li.weights(m)
    w["embed"][:, 1] = 0
    w["embed"][m.vocab - 1, 1] = bf16(2.0)
    w["layers"][0]["wv"][:, 1] = bf16(3e38)
    got = []
    for step in (n, 16):
        say("wide prefill, overflowed value", heads, ctx, step)
        eng = Engine(m, max_ctx=max_ctx, k_max=8)
        eng.kv.zero_()
        eng.load_weights(w, li.qnet_weights(m))
        if ctx:
            eng.lede_prefill(toks[:ctx])
        for i in range(ctx, ctx + n, step):
            eng.lede_prefill(toks[i:min(ctx + n, i + step)])
        half, slots = eng.region_bytes[1] // 2, eng.cfg.n_pages * 64
        got.append([eng.kv[h:h + 2 * slots * 64 * 2].view(torch.bfloat16).view(2, slots, 64).float().cpu().numpy()
                    for h in (0, half)])
        eng.close()
    assert np.isinf(got[0][1][0, bad]).all()
    for at_once, pieces in zip(*got):
        assert np.isfinite(pieces[:, :clean]).all()
        assert np.array_equal(at_once[:, :clean], pieces[:, :clean])


@pytest.mark.parametrize("model", [TINY, BF16_128], ids=lambda m: m.name)
def test_smaller_workspaces(model):
    """Workspaces that hold fewer rows of a prefill pass, in the end none: the
    same bits (other pass sizes, and 16-row passes)."""
    toks = li.uniform_int(1, 20, 440, 0, model.vocab - 1)
    min_bytes = {"tiny": 500992, "bf16-hd128": 1207552}[model.name]
    got = []
    for share in (1.0, 0.5, 0.3, 0.0):
        eng = _engine(model, 448, 1)
        size = min_bytes + int(share * (eng.region_bytes[2] - min_bytes))
        say("wide prefill, workspace of", size, "of", eng.region_bytes[2])
        eng.L.lede_destroy(eng.ctx)
        ctx = ctypes.c_void_p()
        wb, kvb, _ = eng.region_bytes
        eng.ws.fill_(0xFF)
        assert eng.L.lede_create(ctypes.byref(eng.cfg), eng.weights.data_ptr(), wb, eng.kv.data_ptr(), kvb,
                                 eng.ws.data_ptr(), size, ctypes.byref(ctx)) == 0
        eng.ctx = ctx
        eng.lede_set_options(0, 1)
        eng.lede_prefill(toks[:300])
        eng.lede_prefill(toks[300:])
        got.append(_state(eng))
        assert (eng.ws[size:] == 0xFF).all()
        eng.close()
    for state in got[1:]:
        assert state[:3] == got[0][:3]
        assert np.array_equal(state[3], got[0][3]) and np.array_equal(state[4], got[0][4])
