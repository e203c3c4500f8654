"""The bf16 prefill in blocks of up to 2048 rows: 256 x 256 projection tiles, masked attention over the paged cache with the
keys of a block shared by its rows (split and merged again where there are few rows), the head for the last row only.
Sizes where that can go wrong: one row past a row tile, ragged tails, blocks that continue a cached prefix off a page or
tile boundary, few rows behind many keys, head counts that do not fill a workgroup, both head widths.  Against the
oracle's cache-free causal forward, with the bounds of test_gpu_prefill.py."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2603_02599_amd import binding as sun, workloads as wl
from test_gpu_prefill import PREFILL_ABS_TOL, _one_request_case, _prefill, _written_mask

pytestmark = pytest.mark.gpu

G1 = dataclasses.replace(wl.SMALL128, name="small_g1", n_q_heads=4, n_kv_heads=4)
G3 = dataclasses.replace(wl.SMALL128, name="small_g3", n_q_heads=6, n_kv_heads=2)


@pytest.fixture(scope="module")
def H():
    import gpu_harness
    assert torch.cuda.is_available(), "these tests need the MI355X"
    sun.lib()
    return gpu_harness


@pytest.mark.parametrize("shape,T,cuts", [
    (wl.SMALL128, 257, []), (wl.SMALL128, 700, [40, 641]), (wl.SMALL128, 450, [1, 33, 47]), (wl.SMALL_G5, 330, [300]),
    (wl.TINY_Q, 290, [5]), (G1, 300, [270]), (G3, 100, [31])],
    ids=["g4-257", "g4-few-rows-behind-640-keys", "g4-off-tile", "g5-330", "d64-g2-290", "g1-300", "g3-100"])
def test_prefill_blocks_equal_the_causal_forward(H, shape, T, cuts):
    H.say(f"prefill blocks {shape.name} T={T} cuts={cuts}")
    case, rng = _one_request_case(H, shape, "bf16", T, seed=700 + T)
    toks = rng.integers(0, shape.vocab, size=T).astype(np.int32)
    before = H.to_np(case.pool_mem).copy()
    st, table = H.layout_strides(case.lay), case.work.page_tables[0]
    logits, K, V = H.orc.full_forward(H.orc.make_cfg(shape), case.oracle_params(), toks, round_kv=True, want_kv=True)
    expect = before.copy()
    H.orc.kv_ingest(expect, st, H.orc.bf16_bits(K), H.orc.bf16_bits(V), 0, table)
    for a, b in zip([0] + cuts, cuts + [T]):
        got, nxt = _prefill(case, toks[a:b], a, 1)
        H.check_logits(got[None], logits[b - 1][None], "bf16")
        H.check_next_tokens(np.array([nxt]), logits[b - 1][None], 2e-2)
    after = H.to_np(case.pool_mem).copy()
    mask = _written_mask(H, st, after.size, shape.n_layers, shape.n_kv_heads, shape.head_dim, table, 0, T)
    H.check_appended_kv(after, expect, before, mask, "bf16", abs_tol=PREFILL_ABS_TOL, max_off_frac=0.6)


def test_prefill_takes_a_workspace_sized_for_256_tokens(H):
    """A workspace that serves 256 rows serves a longer prompt, with the same result up to rounding; a smaller one is refused.
    (This shape's 600 rows need no more; shorter blocks are chosen in the test of a middle-sized workspace.)"""
    T = 600
    case, rng = _one_request_case(H, wl.SMALL128, "bf16", T, seed=741)
    toks = torch.from_numpy(rng.integers(0, wl.SMALL128.vocab, size=T).astype(np.int32)).cuda()
    row = case.tables[0].contiguous()
    full, least = (sun.sun_prefill_workspace_bytes(case.cfg, n, row.numel()) for n in (T, 256))
    assert least <= full
    got = []
    for nbytes in (full, least):
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        logits = torch.full((wl.SMALL128.vocab,), float("nan"), device="cuda")
        sun.sun_prefill(case.pool, case.weights, toks, row, 0, 0, logits, None, ws, flags=sun.SUN_VALIDATE)
        torch.cuda.synchronize()
        got.append(logits.cpu().numpy())
    H.check_logits(got[1][None], got[0][None], "bf16")
    with pytest.raises(sun.SunError) as e:
        sun.sun_prefill(case.pool, case.weights, toks, row, 0, 0, logits, None, ws[:least - 256], flags=0)
    assert e.value.status == 4


@pytest.mark.parametrize("bad_at,T", [(20, 50), (0, 33), (63, 300)])
def test_a_row_that_is_not_finite_reaches_later_rows_only(H, bad_at, T):
    """A prompt token whose embedding is NaN: the entries before it are those of the prompt without it, bit for bit in the
    first layer and finite in all, the entries after it and the logits are NaN (it is attended to by every later row)."""
    shape = wl.SMALL128
    case, rng = _one_request_case(H, shape, "bf16", T, seed=750 + bad_at)
    toks = rng.integers(1, shape.vocab, size=T).astype(np.int32)
    clean, _ = _prefill(case, toks, 0, 0)
    ok = H.to_np(case.pool_mem).copy()
    case.w["embed"][0] = float("nan")
    toks[bad_at] = 0
    got, _ = _prefill(case, toks, 0, 0)
    after = H.to_np(case.pool_mem).copy()
    case.w["embed"][0] = 0.0
    st, table = H.layout_strides(case.lay), case.work.page_tables[0]
    sizes = (after.size, shape.n_layers, shape.n_kv_heads, shape.head_dim, table)
    early = _written_mask(H, st, *sizes, 0, bad_at) if bad_at else np.zeros(after.size, bool)
    late = _written_mask(H, st, *sizes, bad_at, T - bad_at)
    assert np.isfinite(clean).all() and np.isnan(got).all()
    value = lambda bits: (bits.astype(np.uint32) << 16).view(np.float32)
    assert np.array_equal(after[early], ok[early])      # every operation of an earlier row is the same one
    layer = np.zeros(after.size, bool)
    layer[int(st["k_layer"]):] = True                   # from the second layer on; in the first only the token's own entry is NaN
    assert np.isnan(value(after[late & layer])).all()


@pytest.mark.parametrize("rows", [129, 200, 256])
def test_wide_vocabulary_projection(H, rows):
    """The vocabulary projection above 128 rows (256 x 256 tiles, a ragged last column tile) against float64."""
    shape = dataclasses.replace(wl.SMALL128, name="small_wide", vocab=81920 + 96)
    cfg = sun.make_cfg(shape, "bf16")
    w = wl.make_weights(shape, "bf16", H.DEV, 77)
    W = sun.sun_weights_create(cfg, w)
    x = torch.randn((rows, shape.hidden), device=H.DEV, generator=torch.Generator(device=H.DEV).manual_seed(rows))
    out = torch.full((rows, shape.vocab), float("nan"), device=H.DEV)
    ws = torch.empty(sun.sun_workspace_bytes(cfg, rows, 1), dtype=torch.uint8, device=H.DEV)
    sun.sun_linear(W, 0, 4, x, out, ws)
    torch.cuda.synchronize()
    want = x.double() @ w["wlm"].double().t()
    assert ((out.double() - want).abs() <= 2e-4 + 1e-5 * want.abs()).all()


@pytest.mark.parametrize("rows", [129, 256])
@pytest.mark.parametrize("hidden,vocab", [(512, 65536), (512, 65568), (512, 81632), (512, 81664), (2048, 73440), (2048, 73472), (4096, 65568)])
def test_vocabulary_projection_on_both_sides_of_the_wide_rule(H, hidden, vocab, rows):
    """One round of 256 column tiles, just past it, and the last column count of the strip kernel and the first of the wide one
    behind it (319 / 320 tiles, from hidden 2048 on 287 / 288, from 4096 on any), against float64."""
    shape = dataclasses.replace(wl.SMALL128, name="small_head", n_layers=1, hidden=hidden, vocab=vocab)
    cfg = sun.make_cfg(shape, "bf16")
    w = wl.make_weights(shape, "bf16", H.DEV, 81)
    W = sun.sun_weights_create(cfg, w)
    x = torch.randn((rows, hidden), device=H.DEV, generator=torch.Generator(device=H.DEV).manual_seed(rows))
    out = torch.full((rows, vocab), float("nan"), device=H.DEV)
    ws = torch.empty(sun.sun_workspace_bytes(cfg, rows, 1), dtype=torch.uint8, device=H.DEV)
    sun.sun_linear(W, 0, 4, x, out, ws)
    torch.cuda.synchronize()
    want = x.double() @ w["wlm"].double().t()
    assert ((out.double() - want).abs() <= 2e-4 + 1e-5 * want.abs()).all()


def _expect(H, case, shape, toks, before):
    st, table = H.layout_strides(case.lay), case.work.page_tables[0]
    logits, K, V = H.orc.full_forward(H.orc.make_cfg(shape), case.oracle_params(), toks, round_kv=True, want_kv=True)
    pool = before.copy()
    H.orc.kv_ingest(pool, st, H.orc.bf16_bits(K), H.orc.bf16_bits(V), 0, table)
    return logits, pool, _written_mask(H, st, before.size, shape.n_layers, shape.n_kv_heads, shape.head_dim, table, 0, len(toks))


@pytest.mark.parametrize("shape,T,cuts", [(wl.SMALL128, 2400, [203]), (wl.SMALL_G5, 1536, [])],
                         ids=["blocks-of-1280-and-917-behind-203-keys", "g5-shares-of-14-14-12-stages"])
def test_prefill_in_several_wide_blocks(H, shape, T, cuts):
    """Two blocks of more than 256 rows in one call, the second at a workspace layout of its own and behind the first one's
    keys, off a page and a tile boundary; and a split along k whose last share is shorter."""
    H.say(f"wide blocks {shape.name} T={T} cuts={cuts}")
    case, rng = _one_request_case(H, shape, "bf16", T, seed=760 + T)
    toks = rng.integers(0, shape.vocab, size=T).astype(np.int32)
    before = H.to_np(case.pool_mem).copy()
    logits, expect, mask = _expect(H, case, shape, toks, before)
    for a, b in zip([0] + cuts, cuts + [T]):
        got, nxt = _prefill(case, toks[a:b], a, 1)
        H.check_logits(got[None], logits[b - 1][None], "bf16")
        H.check_next_tokens(np.array([nxt]), logits[b - 1][None], 2e-2)
    H.check_appended_kv(H.to_np(case.pool_mem).copy(), expect, before, mask, "bf16", abs_tol=PREFILL_ABS_TOL, max_off_frac=0.6)


def test_prefill_in_the_blocks_that_a_middle_sized_workspace_holds(H):
    """1600 tokens in one block, and in the least workspace in blocks of 1024 and 576 rows."""
    T = 1600
    shape = dataclasses.replace(wl.SMALL128, name="small_wide_down", n_layers=1, hidden=1024, ffn=4096)
    case, rng = _one_request_case(H, shape, "bf16", T, seed=770)
    toks = rng.integers(0, shape.vocab, size=T).astype(np.int32)
    before = H.to_np(case.pool_mem).copy()
    logits, expect, mask = _expect(H, case, shape, toks, before)
    d_tok, row = torch.from_numpy(toks).cuda(), case.tables[0].contiguous()
    full, least = (sun.sun_prefill_workspace_bytes(case.cfg, n, row.numel()) for n in (T, 256))
    assert least < full
    for nbytes in (full, full - 256, least):
        case.pool_mem.copy_(torch.from_numpy(before.view(np.int16)).view(torch.bfloat16))
        got = torch.full((shape.vocab,), float("nan"), device="cuda")
        sun.sun_prefill(case.pool, case.weights, d_tok, row, 0, 0, got, None, torch.empty(nbytes, dtype=torch.uint8, device="cuda"),
                        flags=sun.SUN_VALIDATE)
        torch.cuda.synchronize()
        H.check_logits(got.cpu().numpy()[None], logits[T - 1][None], "bf16")
        H.check_appended_kv(H.to_np(case.pool_mem).copy(), expect, before, mask, "bf16", abs_tol=PREFILL_ABS_TOL, max_off_frac=0.6)


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("first,bad_at,rows", [(43, 40, 20), (1003, 1000, 40), (1003, 100, 40), (1003, 1000, 300)],
                         ids=["one-split-same-tile", "split-keys-same-tile", "split-keys-earlier-tile", "a-wide-block"])
def test_a_value_that_is_not_finite_reaches_the_rows_that_see_it(H, value, first, bad_at, rows):
    """A cached position with a finite K and a V that is not finite, in the 32 keys of the block's first rows (whose products
    leave it out and mark the rows instead) or before them: every row of the block sees it, so all of a row's entries
    after the first layer and the logits are not numbers; the first layer's entries are those of the clean cache bit for bit."""
    shape = wl.SMALL128
    T = first + rows
    case, rng = _one_request_case(H, shape, "bf16", T, seed=780 + bad_at + rows)
    toks = rng.integers(0, shape.vocab, size=T).astype(np.int32)
    _prefill(case, toks[:first], 0, 0)
    cached = case.pool_mem.clone()
    clean, _ = _prefill(case, toks[first:], first, 0)
    ok = H.to_np(case.pool_mem).copy()
    case.pool_mem.copy_(cached)
    st, table = H.layout_strides(case.lay), case.work.page_tables[0]
    at = int(st["v_off"]) + int(table[bad_at // 16]) * int(st["v_page"]) + (bad_at % 16) * int(st["v_token"])   # layer 0, head 0
    case.pool_mem[at + 7 * int(st["v_dim"])] = value
    got, _ = _prefill(case, toks[first:], first, 0)
    after = H.to_np(case.pool_mem).copy()
    new = _written_mask(H, st, after.size, shape.n_layers, shape.n_kv_heads, shape.head_dim, table, first, rows)
    deeper = np.zeros(after.size, bool)
    deeper[int(st["k_layer"]):] = True
    assert np.isfinite(clean).all() and np.isnan(got).all()
    assert np.array_equal(after[new & ~deeper], ok[new & ~deeper])
    assert np.isnan((after[new & deeper].astype(np.uint32) << 16).view(np.float32)).all()


@pytest.mark.parametrize("first,rows", [(0, 37), (0, 300), (45, 9), (1003, 40)])
def test_slots_past_the_prompt_may_hold_anything(H, first, rows):
    """K and V of the positions behind the prompt, in its last page and the table's following ones, are not numbers: the same
    logits and entries bit for bit."""
    shape = wl.SMALL128
    T = first + rows
    case, rng = _one_request_case(H, shape, "bf16", T, seed=790 + T, extra=70)
    toks = rng.integers(0, shape.vocab, size=T).astype(np.int32)
    st, table = H.layout_strides(case.lay), case.work.page_tables[0]
    sizes = (case.pool_mem.numel(), shape.n_layers, shape.n_kv_heads, shape.head_dim, table)
    behind = torch.from_numpy(_written_mask(H, st, *sizes, T, 70)).cuda()
    own = _written_mask(H, st, *sizes, 0, T)
    if first:
        _prefill(case, toks[:first], 0, 0)
    cached, got = case.pool_mem.clone(), []
    for fill in (0.0, float("nan")):
        case.pool_mem.copy_(cached)
        case.pool_mem[behind] = fill
        logits, _ = _prefill(case, toks[first:], first, 0)
        got.append((logits, H.to_np(case.pool_mem).copy()[own]))
    assert np.isfinite(got[0][0]).all()
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])


@pytest.mark.parametrize("hidden,heads,ffn", [(256, (64, 32), 7040), (256, (56, 28), 8192), (512, (72, 36), 16256), (512, (42, 42), 18816), (512, (52, 26), 13568)],
                         ids=["qkv-8-gate-up-6", "qkv-6-gate-up-8", "qkv-7-gate-up-6", "qkv-6-gate-up-7", "qkv-5-gate-up-5"])
def test_column_tiles_of_other_widths(H, hidden, heads, ffn):
    """Widths for which q/k/v and gate/up take workgroups of five to eight 32-column strips (the last workgroup ragged), three row
    tiles of which the last holds eight rows."""
    shape = dataclasses.replace(wl.SMALL128, name="narrow", hidden=hidden, n_q_heads=heads[0], n_kv_heads=heads[1], ffn=ffn)
    test_prefill_blocks_equal_the_causal_forward(H, shape, 520, [])


@pytest.mark.parametrize("rows,slabs", [(520, 3), (1024, 2), (1536, 3), (2048, 1)])
def test_the_split_along_k_does_not_follow_the_tile_width(H, rows, slabs):
    """How many slabs the sums of q/k/v (6144 x 4096) have, read from V: its weights are 2^30, then ones, then -2^30, and the inputs
    ones, so that of each row's 4096 products those of the first slab are lost beside the 2^30 (64 is half of what it resolves there, a
    matrix instruction adds 16) and those of the others stay.  The tiles are six or seven strips wide."""
    shape = dataclasses.replace(wl.SHAPES["llama8b"], name="one_layer", n_layers=1, ffn=128, vocab=64)
    cfg = sun.make_cfg(shape, "bf16")
    w = wl.make_weights(shape, "bf16", H.DEV, 91)
    w["embed"].fill_(1.0)
    w["g1"][0].fill_(1.0)
    w["wv"][0].fill_(1.0)
    w["wv"][0][:, 0] = 2.0 ** 30
    w["wv"][0][:, -1] = -(2.0 ** 30)
    W = sun.sun_weights_create(cfg, w)
    n_pages = (rows + 15) // 16
    mem = torch.zeros(sun.sun_kv_pool_bytes(cfg, n_pages) // 2, dtype=torch.bfloat16, device=H.DEV)
    pool = sun.sun_kv_pool_create(cfg, mem, 16, 1)
    lay = pool.layout()
    table = torch.arange(n_pages, dtype=torch.int32, device=H.DEV)
    ws = torch.empty(sun.sun_prefill_workspace_bytes(cfg, rows, n_pages), dtype=torch.uint8, device=H.DEV)
    logits, nxt = torch.empty(shape.vocab, device=H.DEV), torch.empty(1, dtype=torch.int32, device=H.DEV)
    sun.sun_prefill(pool, W, torch.zeros(rows, dtype=torch.int32, device=H.DEV), table, 0, 0, logits, nxt, ws)
    torch.cuda.synchronize()
    v = mem.as_strided((n_pages, shape.n_kv_heads, shape.head_dim, 16), (lay.v_page, lay.v_head, lay.v_dim, lay.v_token), lay.v_off)
    v = v.permute(0, 3, 1, 2).reshape(n_pages * 16, -1)[:rows].float()
    stages = shape.hidden // 32
    first = -(-stages // slabs) * 32
    # the last slab and each sum with a slab behind the first round to a multiple of 64, V to 2^-9 of itself
    assert float(v.min()) == float(v.max()) and abs(float(v[0, 0]) - (shape.hidden - first)) <= 32 * slabs + 8


@pytest.mark.parametrize("rows", [129, 160, 161, 192, 193, 224, 225])
def test_wide_vocabulary_projection_leaves_out_row_blocks(H, rows):
    """Five to eight of the eight 32-row blocks of a tile hold rows: a wave with both of its blocks, with one, with none."""
    test_wide_vocabulary_projection(H, rows)
