"""A decode step at the sizes where the fp32 kernels, the step's first launch and the argmax can go wrong: widths that are
not a multiple of four or do not start on 16 bytes, row counts around the eight of a wave, head widths and group sizes,
more requests than a thread of the plan sums up, vocabularies that leave ragged slices, ties across slices.  Against the
oracle, with the bounds of the other parity tests."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2603_02599_amd import binding as sun, workloads as wl

pytestmark = pytest.mark.gpu

ODD = dataclasses.replace(wl.TINY, name="odd", ffn=689, vocab=1031)
WIDE = dataclasses.replace(wl.TINY, name="wide", n_q_heads=8, n_kv_heads=1, head_dim=128, vocab=5000)


@pytest.fixture(scope="module")
def H():
    import gpu_harness
    assert torch.cuda.is_available(), "these tests need the MI355X"
    sun.lib()
    return gpu_harness


@pytest.mark.parametrize("shape,dtype,batch,lo,hi,quant", [
    (ODD, "f32", 1, 5, 5, None), (ODD, "f32", 9, 1, 70, None), (WIDE, "f32", 7, 60, 300, None), (WIDE, "f32", 8, 1, 17, None),
    (wl.TINY_Q, "f32", 17, 1, 40, "asym"), (wl.TINY, "f32", 65, 200, 700, None), (wl.SMALL128, "bf16", 255, 1, 60, None),
    (wl.TINY_QWEN, "f32", 3, 15, 33, None)],
    ids=["odd-1", "odd-9", "g8-d128-7", "g8-d128-8", "w4-17", "65-full-chunks", "bf16-255", "head-norm-3"])
def test_step_at_the_edges(H, shape, dtype, batch, lo, hi, quant):
    work = wl.make_workload("cfg1", shape=shape, dtype=dtype, batch=batch, seed=900 + batch)
    rng = np.random.default_rng(batch)
    work.seq_lens = rng.integers(lo, hi + 1, size=batch).astype(np.int32)
    work.page_tables, work.n_pages = wl.deal_page_tables(work.seq_lens, rng)
    case = H.GpuCase(work, quant_mode=quant)
    ref = H.run_oracle(case, list(range(batch)))
    for host_lens in (True, False):
        case.logits.fill_(float("nan"))
        case.step(flags=sun.SUN_VALIDATE, host_lens=host_lens)
        H.check_logits(case.logits.cpu().numpy(), ref["logits"], dtype)
        H.check_next_tokens(case.next.cpu().numpy(), ref["logits"], 1e-4 if dtype == "f32" else 2e-2)


def test_f32_weights_that_do_not_start_on_16_bytes(H):
    """The same matrices behind pointers that are four bytes off a 16-byte boundary: the same logits up to fp32 sums."""
    work = wl.make_workload("cfg1", seed=950)
    case = H.GpuCase(work)
    case.step()
    want = case.logits.cpu().numpy()

    def off(t):
        buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
        buf[1:] = t.reshape(-1)
        return buf[1:].view(t.shape)
    w = {k: [off(t) for t in v] if isinstance(v, list) else off(v) if isinstance(v, torch.Tensor) else v for k, v in case.w.items()}
    assert w["wq"][0].data_ptr() % 16 == 4
    case.weights = sun.sun_weights_create(case.cfg, w)
    case.step()
    assert np.abs(case.logits.cpu().numpy() - want).max() <= 2e-5   # two fp32 sums of 688 terms, a fifth of the parity bar


@pytest.mark.parametrize("vocab,dtype", [(1024, "f32"), (5001, "f32"), (4100, "f32"), (8224, "bf16")])
def test_argmax_takes_the_lowest_index_of_a_tie(H, vocab, dtype):
    shape = dataclasses.replace(wl.TINY if dtype == "f32" else wl.TINY_Q, name="tie", vocab=vocab)
    work = wl.make_workload("cfg1", shape=shape, dtype=dtype, seed=960)
    case = H.GpuCase(work)
    case.step()
    best = int(case.next.cpu()[0])
    wlm = case.w["wlm"].clone()
    for places in ([best, 7, 8], [vocab - 1, best], [0, vocab // 2, vocab - 1], [vocab - 2, vocab - 1]):
        w = dict(case.w)
        w["wlm"] = wlm.clone()
        w["wlm"][best] = 0.0
        w["wlm"][places] = wlm[best]
        case.weights = sun.sun_weights_create(case.cfg, w)
        case.step()
        row = case.logits.cpu().numpy()[0]
        assert int(case.next.cpu()[0]) == min(places) == int(np.argmax(row))


@pytest.mark.parametrize("rows", [1, 8, 9, 16, 17, 33, 65, 97, 150, 161, 256])
def test_w4_projections_at_the_edges_of_row_tiles(H, rows):
    """One row more or less than an octet of the scaled rows or a 32-row tile; an odd number of tiles.  Against float64 of the
    dequantised matrices, with the bound of a 4-bit projection (its activations are rounded to 16 bits a group)."""
    shape = wl.SMALL128
    cfg = sun.make_cfg(shape, "bf16")
    w = wl.make_weights(shape, "bf16", H.DEV, 78)
    quant = {k: [sun.sun_quantize_w4(m, 128, "asym") for m in w[k]] for k in sun.QUANT_KEYS}
    W = sun.sun_qweights_create(cfg, w, quant)

    def dense(q, s, z):
        codes = torch.stack([q & 15, q >> 4], 2).view(q.shape[0], -1, 128).double()
        return ((codes - z.double().unsqueeze(2)) * s.double().unsqueeze(2)).view(q.shape[0], -1)
    mats = {0: ["wq", "wk", "wv"], 1: ["wo"], 3: ["wd"]}
    ws = torch.empty(sun.sun_workspace_bytes(cfg, rows, 1), dtype=torch.uint8, device=H.DEV)
    for mat, keys in mats.items():
        M = torch.cat([dense(*quant[k][1]) for k in keys])
        x = torch.randn((rows, M.shape[1]), device=H.DEV, generator=torch.Generator(device=H.DEV).manual_seed(rows + mat))
        out = torch.full((rows, M.shape[0]), float("nan"), device=H.DEV)
        sun.sun_linear(W, 1, mat, x, out, ws)
        torch.cuda.synchronize()
        want = x.double() @ M.t()
        assert ((out.double() - want).abs() <= 1e-3 + 1e-4 * want.abs()).all(), mat


@pytest.mark.parametrize("rows,full", [(66, 128), (96, 128), (129, 256), (150, 256), (225, 256)])
def test_w4_rows_do_not_depend_on_the_rows_beside_them(H, rows, full):
    """The split along k goes with the class of the row count, so the rows of a smaller batch are those of the full one, bit
    for bit, also where fewer row tiles are launched."""
    shape = dataclasses.replace(wl.SMALL128, name="w4_rows", n_layers=1, hidden=4096, n_q_heads=32, n_kv_heads=8)
    cfg = sun.make_cfg(shape, "bf16")
    w = wl.make_weights(shape, "bf16", H.DEV, 79)
    W = sun.sun_qweights_create(cfg, w, {k: [sun.sun_quantize_w4(m, 128, "asym") for m in w[k]] for k in sun.QUANT_KEYS})
    x = torch.randn((full, 4096), device=H.DEV, generator=torch.Generator(device=H.DEV).manual_seed(rows))
    got = []
    for n in (rows, full):
        out = torch.full((n, 4096), float("nan"), device=H.DEV)
        sun.sun_linear(W, 0, 1, x[:n], out, torch.empty(sun.sun_workspace_bytes(cfg, n, 1), dtype=torch.uint8, device=H.DEV))
        torch.cuda.synchronize()
        got.append(out.cpu().numpy())
    assert np.isfinite(got[0]).all() and np.array_equal(got[0], got[1][:rows])


@pytest.mark.parametrize("ffn", [13184, 13312, 16512], ids=["206-workgroups", "208-workgroups", "ragged-strips"])
@pytest.mark.parametrize("batch", [1, 33, 64])
def test_gate_up_on_both_sides_of_the_fused_epilogue(H, ffn, batch):
    """Below 208 workgroups of columns the gate/up sums go through slabs and a SwiGLU kernel, from there on through the
    projection's epilogue; 1032 strips leave waves of the last workgroup without columns."""
    shape = dataclasses.replace(wl.SMALL128, name="ffn", ffn=ffn)
    work = wl.make_workload("cfg1", shape=shape, dtype="bf16", batch=batch, seed=970 + batch)
    rng = np.random.default_rng(batch)
    work.seq_lens = rng.integers(1, 40, size=batch).astype(np.int32)
    work.page_tables, work.n_pages = wl.deal_page_tables(work.seq_lens, rng)
    case = H.GpuCase(work)
    ref = H.run_oracle(case, list(range(batch)))
    case.logits.fill_(float("nan"))
    case.step(flags=sun.SUN_VALIDATE)
    H.check_logits(case.logits.cpu().numpy(), ref["logits"], "bf16")
    H.check_next_tokens(case.next.cpu().numpy(), ref["logits"], 2e-2)


@pytest.mark.parametrize("tokens,first", [(4096, 5), (4097, 5), (4133, 0)], ids=["through-the-caches", "streamed", "streamed-aligned"])
def test_ingest_on_both_sides_of_the_streaming_rule(H, tokens, first):
    """A hand-over of more than 32 MB (8 KB a token here) streams past the caches: the pool bit for bit as the oracle's."""
    shape = dataclasses.replace(wl.LLAMA_8B, name="ingest", n_layers=2)
    cfg = sun.make_cfg(shape, "bf16")
    n_pages = (tokens + first + 15) // 16 + 3
    mem = torch.empty(sun.sun_kv_pool_bytes(cfg, n_pages) // 2, dtype=torch.bfloat16, device="cuda")
    wl.fill_kv_pool(mem, 62)
    pool = sun.sun_kv_pool_create(cfg, mem, 16, 1)
    host = H.to_np(mem).copy()
    row = np.random.default_rng(tokens).permutation(n_pages).astype(np.int32)
    k = torch.randn((2, tokens, shape.n_kv_heads, shape.head_dim), device="cuda").to(torch.bfloat16)
    v = torch.randn_like(k)
    sun.sun_kv_pool_ingest(pool, 0, k, v, first, torch.from_numpy(row).cuda(), flags=sun.SUN_VALIDATE)
    H.orc.kv_ingest(host, H.layout_strides(pool.layout()), H.to_np(k), H.to_np(v), first, row)
    torch.cuda.synchronize()
    assert np.array_equal(H.to_np(mem), host)


def test_chunks_are_merged_in_groups_of_eight(H):
    """The merge of a request's chunks adds them in token order under a running maximum that moves once per eight chunks, for
    one chunk, ragged groups and more than a wave's 64.  The inputs make every chunk's maximum, sum (1) and output exact (one
    key per chunk counts, with a bf16 score and value), so the sums can be repeated bit for bit; an order of its own (one
    maximum for all chunks, say) agrees in about two outputs of three."""
    shape, B = wl.SMALL128, 64
    rng = np.random.default_rng(980)
    lens = rng.integers(1, 3000, size=B).astype(np.int32)
    lens[:4] = [1, 64, 17 * 1024 + 40, 66 * 256]
    cfg = sun.make_cfg(shape, "bf16")
    tables, n_pages = wl.deal_page_tables(lens - 1, rng)
    n_pages += 1
    D, Hkv, G = shape.head_dim, shape.n_kv_heads, shape.n_q_heads // shape.n_kv_heads
    bf = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).to(torch.bfloat16)
    host = np.zeros(sun.sun_kv_pool_bytes(cfg, n_pages) // 2, np.uint16)
    mem = torch.empty(host.size, dtype=torch.bfloat16, device=H.DEV)
    pool = sun.sun_kv_pool_create(cfg, mem, 16, 1)
    st = H.layout_strides(pool.layout())
    chunks = []
    for b, n in enumerate(lens):
        full = max(int(n) // 256 - 1, 0)       # the chunk grid from 64 requests up
        starts = [256 * i for i in range(full)] + list(range(256 * full, int(n), 64))
        ends = starts[1:] + [int(n)]
        keys = [int(rng.integers(a, z)) for a, z in zip(starts, ends)]
        K = np.zeros((shape.n_layers, n, Hkv, D), np.float32)
        V = np.zeros_like(K)
        K[..., 0] = -30000.0
        K[0, keys, :, 0] = bf(rng.normal(0, 3, (len(keys), Hkv))).float().numpy()
        V[0, keys] = bf(rng.normal(0, 1, (len(keys), Hkv, D))).float().numpy()
        H.orc.kv_ingest(host, st, H.to_np(bf(K)), H.to_np(bf(V)), 0, tables[b])
        chunks.append((K[0, keys, :, 0], V[0, keys]))
    mem.copy_(torch.from_numpy(host.view(np.int16)).view(torch.bfloat16))
    scale = np.float32(1.4426950408889634) / np.sqrt(np.float32(D))
    x = np.float32(1) / scale                  # the query whose scaled value is exactly 1
    x = next(c for c in (x, np.nextafter(x, np.float32(0)), np.nextafter(x, np.float32(99))) if c * scale == 1)
    q = np.zeros((B, shape.n_q_heads, D), np.float32)
    q[:, :, 0] = x
    out = torch.full((B, shape.q_dim), float("nan"), device=H.DEV)
    ws = torch.empty(sun.sun_workspace_bytes(cfg, B, tables.shape[1]), dtype=torch.uint8, device=H.DEV)
    sun.sun_paged_attention(pool, 0, torch.from_numpy(q.reshape(B, -1)).to(H.DEV), torch.from_numpy(tables).to(H.DEV),
                            torch.from_numpy(lens).to(H.DEV), out, ws)
    got = out.cpu().numpy().reshape(B, Hkv, G, D)
    exp2 = lambda a: torch.exp2(torch.from_numpy(np.asarray(a, np.float32)).to(H.DEV)).cpu().numpy()
    fma = lambda a, c, d: (a.astype(np.float64) * c + d).astype(np.float32)
    same = 0
    for b, (m, o) in enumerate(chunks):
        M, num, den = np.full(Hkv, -np.inf, np.float32), np.zeros((Hkv, D), np.float32), np.zeros(Hkv, np.float32)
        for c0 in range(0, len(m), 8):
            Mn = np.maximum(M, m[c0:c0 + 8].max(0))
            sc, w, M = exp2(M - Mn), exp2(m[c0:c0 + 8] - Mn), Mn
            num, den = num * sc[:, None], den * sc
            for i in range(len(w)):
                den = fma(w[i], 1.0, den)
                num = fma(w[i][:, None], o[c0 + i], num)
        want = (num / den[:, None])[:, None]
        assert np.abs(got[b] - want).max() <= 1e-5 * np.abs(o).max()
        same += int((got[b] == want).sum())
    assert same >= 0.999 * got.size, same / got.size   # what is left: sums rounded twice, and exponentials an ulp apart


@pytest.mark.parametrize("rows", [1, 32, 33, 64])
def test_projections_on_both_sides_of_the_streaming_rule(H, rows):
    """A model of more than 256 MB of weights streams them past the caches, a smaller one loads them plainly: the same sums bit
    for bit, and those of float64."""
    small = dataclasses.replace(wl.SMALL128, name="below", n_layers=1, hidden=1024, vocab=4096)
    large = dataclasses.replace(small, name="above", vocab=131072)
    w = wl.make_weights(large, "bf16", H.DEV, 80)
    x = torch.randn((rows, 1024), device=H.DEV, generator=torch.Generator(device=H.DEV).manual_seed(rows))
    got = {}
    for shape in (small, large):
        cfg = sun.make_cfg(shape, "bf16")
        assert (sun.sun_weights_pack_bytes(cfg) > 256 << 20) == (shape is large)
        W = sun.sun_weights_create(cfg, {**w, "embed": w["embed"][:shape.vocab], "wlm": w["wlm"][:shape.vocab].contiguous()})
        ws = torch.empty(sun.sun_workspace_bytes(cfg, rows, 1), dtype=torch.uint8, device=H.DEV)
        for mat, n in ((0, shape.q_dim + 2 * shape.kv_dim), (2, shape.ffn), (4, shape.vocab)):
            out = torch.full((rows, n), float("nan"), device=H.DEV)
            sun.sun_linear(W, 0, mat, x, out, ws)
            torch.cuda.synchronize()
            got[shape.name, mat] = out
    for mat in (0, 2, 4):
        a, b = got["below", mat], got["above", mat]
        assert torch.equal(a, b[:, :a.shape[1]]), mat
    want = x.double() @ w["wlm"].double().t()
    assert ((got["above", 4].double() - want).abs() <= 2e-4 + 1e-5 * want.abs()).all()


@pytest.mark.parametrize("heads", [(2, 2), (8, 2), (10, 2), (8, 1)], ids=lambda h: f"{h[0]}on{h[1]}")
def test_k_through_the_caches_and_past_them(H, heads):
    """The K of a step that fits the memory-side cache is read through it, a larger one past it.  Without the lengths on the host the tables
    and the pool count (20 requests of up to 16 000 positions, 328 MB of K), with them the tokens (4 MB): the same bits, the oracle's logits.
    Attention alone reads a small K as its operand lies: the same bits again."""
    shape = dataclasses.replace(wl.SMALL128, name="k", hidden=128 * heads[0], n_q_heads=heads[0], n_kv_heads=heads[1])
    work = wl.make_workload("cfg1", shape=shape, dtype="bf16", batch=20, seed=996)
    rng = np.random.default_rng(7)
    work.seq_lens = rng.integers(0, 200, size=20).astype(np.int32)
    work.page_tables, _ = wl.deal_page_tables(work.seq_lens, rng)
    work.page_tables = np.pad(work.page_tables, ((0, 0), (0, 1000 - work.page_tables.shape[1])), constant_values=-1)
    work.n_pages = 20000 // heads[1]
    case = H.GpuCase(work)
    ref = H.run_oracle(case, list(range(20)))
    pool0, got = case.pool_mem.clone(), []
    for host_lens in (True, False):
        case.pool_mem.copy_(pool0)
        case.logits.fill_(float("nan"))
        case.step(host_lens=host_lens)
        got.append((case.logits.clone(), case.pool_mem.clone()))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    H.check_logits(got[0][0].cpu().numpy(), ref["logits"], "bf16")
    q, n = torch.randn((20, 128 * heads[0]), device=H.DEV), case.lens + 1
    outs = [torch.full_like(q, float("nan")) for _ in range(2)]
    for out, host in zip(outs, (n.cpu().numpy(), None)):
        sun.sun_paged_attention(case.pool, 1, q, case.tables, n, out, case.ws, n_tokens_host=host)
    torch.cuda.synchronize()
    assert torch.equal(*outs) and bool(torch.isfinite(outs[0]).all())


@pytest.mark.parametrize("rows", [1, 32, 33])
@pytest.mark.parametrize("hidden,vocab", [(256, 114656), (256, 128256), (1024, 152064), (1024, 256000), (3072, 256000)])
def test_vocabulary_projection_on_both_sides_of_the_rule_for_its_waves(H, hidden, vocab, rows):
    """From 3584 strips of 32 columns on the waves of a workgroup are chosen by the activation tile that each stages again: four instead of six
    at 128 256 columns of 256, seven instead of five at 152 064 of 1024, seven instead of four at 256 000; up to 32 rows,
    with k of 3072 or more, a workgroup keeps the four that its start and end ask for.  114 656 columns are a strip below the rule.  Workgroups of seven
    leave the last one ragged.  Against float64 (about 1e-6 of a logit from the sums; the bound of the other projections)."""
    shape = dataclasses.replace(wl.SMALL128, name="vocab", n_layers=1, hidden=hidden, vocab=vocab, ffn=128)
    cfg = sun.make_cfg(shape, "bf16")
    w = wl.make_weights(shape, "bf16", H.DEV, 83)
    W = sun.sun_weights_create(cfg, w)
    x = torch.randn((rows, hidden), device=H.DEV, generator=torch.Generator(device=H.DEV).manual_seed(rows))
    out = torch.full((rows, vocab), float("nan"), device=H.DEV)
    ws = torch.empty(sun.sun_workspace_bytes(cfg, rows, 1), dtype=torch.uint8, device=H.DEV)
    sun.sun_linear(W, 0, 4, x, out, ws)
    torch.cuda.synchronize()
    want = x.double() @ w["wlm"].double().t()
    assert ((out.double() - want).abs() <= 2e-4 + 1e-5 * want.abs()).all()


def test_activations_are_rounded_to_nearest_even(H):
    """Every lower half of a float under signs, exponents and mantissas of all kinds, through a projection by the unit matrix: its input is
    split into two bf16 planes, whose sum, exact in fp32, is that of torch's rounding."""
    shape = dataclasses.replace(wl.SMALL128, name="rounding", n_layers=1, hidden=1024, n_q_heads=8, n_kv_heads=8)
    cfg = sun.make_cfg(shape, "bf16")
    w = wl.make_weights(shape, "bf16", H.DEV, 85)
    w["wo"][0].copy_(torch.eye(1024))
    W = sun.sun_weights_create(cfg, w)
    rng = np.random.default_rng(85)
    ws = torch.empty(sun.sun_workspace_bytes(cfg, 64, 1), dtype=torch.uint8, device=H.DEV)
    for upper in rng.integers(0, 1 << 16, size=(4, 1 << 16)):
        upper = (upper & 0x807F) | (64 + (upper >> 7 & 127)) << 7     # exponents 64 to 190: the lower plane is normal too
        bits = (upper.astype(np.uint32) << 16) | rng.permutation(1 << 16).astype(np.uint32)
        x = torch.from_numpy(bits.view(np.float32).reshape(64, 1024)).to(H.DEV)
        out = torch.full_like(x, float("nan"))
        sun.sun_linear(W, 0, 1, x, out, ws)
        torch.cuda.synchronize()
        high = x.bfloat16().float()
        assert torch.equal(out, high + (x - high).bfloat16().float())


@pytest.mark.parametrize("rows", [1, 32])
@pytest.mark.parametrize("ffn", [57344, 58368, 65536])
def test_wide_4_bit_gate_up_is_not_split_along_k(H, ffn, rows):
    """The rule for a vocabulary's waves does not reach a gate/up pair as wide as a vocabulary, whose split along k sets the order of its
    sums.  An up column's 16 groups add up to 15 * 2^22, about 1 each, -15 * 2^22: 1 is lost beside the first (fp32 resolves 4 there), so one
    slab sums to what the first was rounded by, 2 at most, and what a second one holds (by that rule 58 368 and 65 536 columns have two and
    three) stays, 4 or more.  The gate is 16."""
    shape = dataclasses.replace(wl.SMALL128, name="gate_up", n_layers=1, hidden=2048, n_q_heads=2, n_kv_heads=1, ffn=ffn, vocab=64)
    cfg = sun.make_cfg(shape, "bf16")
    w = wl.make_weights(shape, "bf16", H.DEV, 84)

    def codes(n, k, scales):   # code 15, zero point 0
        s = torch.tensor(scales, dtype=torch.float16, device=H.DEV)[None].expand(n, k // 128).contiguous()
        return torch.full((n, k // 2), 0xFF, dtype=torch.uint8, device=H.DEV), s, torch.zeros_like(s)

    dims = {"wq": (256, 2048), "wk": (128, 2048), "wv": (128, 2048), "wo": (2048, 256), "wg": (ffn, 2048), "wu": (ffn, 2048), "wd": (2048, ffn)}
    one = 1 / (15 * 128)
    quant = {k: [codes(n, c, [one] * (c // 128))] for k, (n, c) in dims.items()}
    quant["wu"] = [codes(ffn, 2048, [2.0 ** 15] + [one] * 14 + [-(2.0 ** 15)])]
    W = sun.sun_qweights_create(cfg, w, quant)
    x = torch.ones((rows, shape.hidden), device=H.DEV)
    out = torch.full((rows, ffn), float("nan"), device=H.DEV)
    sun.sun_linear(W, 0, 2, x, out, torch.empty(sun.sun_workspace_bytes(cfg, rows, 1), dtype=torch.uint8, device=H.DEV))
    torch.cuda.synchronize()
    assert float(out.abs().max()) <= 16 * 2.1


@pytest.mark.parametrize("hidden,ffn,batch", [(256, 688, 3), (256, 688, 95), (256, 688, 96), (512, 1024, 17), (1024, 1000, 9), (1024, 1000, 2),
                                              (2048, 4104, 5), (4096, 300, 1)])
def test_f32_step_on_both_sides_of_its_rules(H, hidden, ffn, batch):
    """The norm inside the projections or in a launch of its own, two or eight rows a wave, one or four steps along k in flight:
    row counts that leave ragged groups of two and eight, against the oracle."""
    shape = dataclasses.replace(wl.TINY, name="f32", n_layers=1, hidden=hidden, ffn=ffn, vocab=1100)
    work = wl.make_workload("cfg1", shape=shape, dtype="f32", batch=batch, seed=990 + batch)
    rng = np.random.default_rng(batch)
    work.seq_lens = rng.integers(1, 30, size=batch).astype(np.int32)
    work.page_tables, work.n_pages = wl.deal_page_tables(work.seq_lens, rng)
    case = H.GpuCase(work)
    ref = H.run_oracle(case, list(range(batch)))
    case.logits.fill_(float("nan"))
    case.step(flags=sun.SUN_VALIDATE)
    H.check_logits(case.logits.cpu().numpy(), ref["logits"], "f32")
    H.check_next_tokens(case.next.cpu().numpy(), ref["logits"], 1e-4)


def test_f32_step_refuses_a_hidden_width_its_norm_does_not_hold(H):
    """More than 16384 columns are refused, as in the bf16 step."""
    shape = dataclasses.replace(wl.TINY, name="too_wide", n_layers=1, hidden=16392, ffn=128, vocab=64)
    case = H.GpuCase(wl.make_workload("cfg1", shape=shape, dtype="f32", batch=1, seed=995))
    with pytest.raises(sun.SunError):
        case.step()


@pytest.mark.parametrize("shift", [0, 64, -64])
def test_f32_gate_up_may_write_over_its_input(H, shift):
    """Gate/up with the output over the input (the same start, or a part of it): the result of separate buffers."""
    shape, batch = wl.TINY, 9
    cfg = sun.make_cfg(shape, "f32")
    W = sun.sun_weights_create(cfg, wl.make_weights(shape, "f32", H.DEV, 82))
    ws = torch.empty(sun.sun_workspace_bytes(cfg, batch, 1), dtype=torch.uint8, device=H.DEV)
    x = torch.randn((batch, shape.hidden), device=H.DEV, generator=torch.Generator(device=H.DEV).manual_seed(1))
    want = torch.empty((batch, shape.ffn), device=H.DEV)
    sun.sun_linear(W, 0, 2, x, want, ws)
    buf = torch.zeros(batch * shape.ffn + 128, device=H.DEV)
    at_x, at_out = 64, 64 + shift
    xin, out = buf[at_x:at_x + x.numel()].view_as(x), buf[at_out:at_out + want.numel()].view_as(want)
    xin.copy_(x)
    sun.sun_linear(W, 0, 2, xin, out, ws)
    torch.cuda.synchronize()
    assert torch.equal(out, want)


@pytest.mark.parametrize("tokens,first", [(4096, 0), (4097, 3)], ids=["stores-through-the-caches", "stores-streamed"])
def test_ingest_on_both_sides_of_the_rule_for_its_stores(H, tokens, first):
    """Above 256 MB of source (64 KB a token here) the stores stream as well: the pool bit for bit as the oracle's."""
    shape = dataclasses.replace(wl.LLAMA_8B, name="ingest", n_layers=16)
    cfg = sun.make_cfg(shape, "bf16")
    n_pages = (tokens + first + 15) // 16 + 1
    mem = torch.zeros(sun.sun_kv_pool_bytes(cfg, n_pages) // 2, dtype=torch.bfloat16, device="cuda")
    pool = sun.sun_kv_pool_create(cfg, mem, 16, 1)
    host = H.to_np(mem).copy()
    row = np.random.default_rng(tokens).permutation(n_pages).astype(np.int32)
    k = torch.randn((16, tokens, shape.n_kv_heads, shape.head_dim), device="cuda").to(torch.bfloat16)
    v = torch.randn_like(k)
    sun.sun_kv_pool_ingest(pool, 0, k, v, first, torch.from_numpy(row).cuda(), flags=sun.SUN_VALIDATE)
    H.orc.kv_ingest(host, H.layout_strides(pool.layout()), H.to_np(k), H.to_np(v), first, row)
    torch.cuda.synchronize()
    assert np.array_equal(H.to_np(mem), host)


SHORT = 384   # positions of the longest table whose attention is one launch; many or wide query heads make it shorter
G4, G2_D128, G1_D128 = (dataclasses.replace(wl.TINY, name=n, n_q_heads=q, n_kv_heads=2, head_dim=d)
                        for n, q, d in (("g4", 8, 64), ("g2_d128", 4, 128), ("g1_d128", 2, 128)))


@pytest.mark.parametrize("shape,lens,extra", [
    (wl.TINY, [0], 0), (wl.TINY, [15, 16, 62, 63, 64, 127, 128, 255, 382], 0), (wl.TINY, [383], 0), (wl.TINY, [383, 5], 1),
    (WIDE, [0, 63, 200, 383], 0), (wl.TINY_BIAS, [17, 64, 300], 0), (wl.TINY_QWEN, [17, 64, 300], 0), (wl.TINY, list(range(310, 375)), 0),
    (WIDE, [0, 15, 62, 63], -20), (WIDE, [0, 63, 64, 79], -19), (G4, [0, 63, 191, 255], -8), (G4, [0, 63, 256, 271], -7),
    (G2_D128, [5, 127, 255], -8), (G1_D128, [0, 64, 383], 0)],
    ids=["empty", "edges", "whole", "beyond", "g8-d128-beyond", "bias", "head-norm", "65-full-chunks", "g8-d128", "g8-d128-one-page-more", "g4-d64",
         "g4-d64-one-page-more", "g2-d128", "g1-d128"])
def test_short_tables_take_one_launch_for_attention(H, shape, lens, extra):
    """Bit for bit what the separate launches give (SUN_PROFILE asks for them): logits and every slot of the cache."""
    work = wl.make_workload("cfg1", shape=shape, dtype="f32", batch=len(lens), seed=980 + len(lens))
    work.seq_lens = np.asarray(lens, np.int32)
    work.page_tables, work.n_pages = wl.deal_page_tables(work.seq_lens, np.random.default_rng(3))
    wide = np.full((len(lens), SHORT // 16 + extra), -1, np.int32)
    wide[:, :work.page_tables.shape[1]] = work.page_tables
    work.page_tables = wide
    case = H.GpuCase(work)
    pool0 = case.pool_mem.clone()
    ref = H.run_oracle(case, list(range(len(lens))))
    got = []
    for flags in (0, sun.SUN_PROFILE):
        case.pool_mem.copy_(pool0)
        case.ws.fill_(0xFF)
        case.step(flags=flags)
        H.check_logits(case.logits.cpu().numpy(), ref["logits"], "f32")
        got.append((case.logits.clone(), case.pool_mem.clone()))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1].view(torch.int16), got[1][1].view(torch.int16))
