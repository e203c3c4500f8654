"""A step of few requests runs all layers in one launch.  Checked where that can go wrong: row counts around the eight that a wave
each finishes and the largest taken, one row beyond it, lengths around chunk and page boundaries, matrices with fewer
column blocks than compute units, more layers than one launch takes, head norm, biases, both 4-bit layouts.  Against the oracle, and
against a launch per operation (which SUN_PROFILE asks for)."""
import ctypes
import dataclasses
import threading

import numpy as np
import pytest
import torch

from paper_2603_02599_amd import binding as sun, workloads as wl

pytestmark = pytest.mark.gpu

# more layers than one launch takes, every matrix split along k
DEEP = dataclasses.replace(wl.SMALL128, name="deep", n_layers=50, hidden=512, n_q_heads=4, n_kv_heads=1, ffn=512, vocab=512)
DEEP_W4 = dataclasses.replace(DEEP, name="deep_w4", hidden=1024, n_q_heads=8, ffn=1024)
SMALL, SMALL_G5, SMALL_BIAS = (dataclasses.replace(s, n_layers=7) for s in (wl.SMALL128, wl.SMALL_G5, wl.SMALL_BIAS))   # deep enough for it
NORM = dataclasses.replace(SMALL, name="norm", qk_norm=True)
ONE_KV = dataclasses.replace(SMALL, name="one_kv", hidden=384, n_q_heads=8, n_kv_heads=1, ffn=640)
EDGES = [0, 1, 15, 16, 17, 62, 63, 64, 65, 127, 128, 129, 255, 256, 300, 511]


@pytest.fixture(scope="module")
def H():
    import gpu_harness
    assert torch.cuda.is_available(), "these tests need the MI355X"
    sun.lib()
    return gpu_harness


def make_case(H, shape, lens, quant=None, seed=700, spare=0):
    work = wl.make_workload("cfg1", shape=shape, dtype="bf16", batch=len(lens), seed=seed + len(lens))
    work.seq_lens = np.asarray(lens, dtype=np.int32)
    work.page_tables, work.n_pages = wl.deal_page_tables(work.seq_lens, np.random.default_rng(seed))
    work.n_pages += spare
    return H.GpuCase(work, quant_mode=quant)


def bits(t):
    return t.clone().view(torch.int16)


def takes_one_launch(case):
    """Whether a step takes the launch: one whose first wait gives up at once has no result."""
    mem = case.pool_mem.clone()
    case.step(flags=sun.SUN_WAIT_POLLS(0))
    case.pool_mem.copy_(mem)
    return bool((case.next == -1).all())


def check_against_oracle(H, case, rows, extracted, quant):
    """Every new entry of every layer and the logits, the oracle going on from the entries that it accepts (a rounding step apart)."""
    ref = H.oracle_step_next_to_gpu_cache(case, rows, extracted, case.pool_pages_now(extracted[3]), quant=quant is not None)
    H.check_logits(case.logits.cpu().numpy()[rows], ref["logits"], "bf16")


def rel(a, b):
    a, b = a.double(), b.double()
    return float((a - b).norm() / b.norm())


# Two correct sums of these products differ by 1e-5 (bf16) and 3e-4 (4-bit: 16 bits a group) of the logits.  Where a new cache entry
# falls on the other side of a bf16 rounding it differs by up to 2^-8 of itself, and for a request of one position
# that is an element of attention's output: ten such among the 256 of a row's K or V are 2^-8 sqrt(10 / 256) = 8e-4 of the row.
# Twice that, for each layer by itself, and for 4-bit weights ten times their 3e-4 beside it.
@pytest.mark.parametrize("shape,lens,quant", [
    (SMALL, [300], None), (SMALL, [0], "asym"), (SMALL, EDGES[:8], None), (SMALL, EDGES[8:], "asym"),
    (SMALL, EDGES[7:], None), (SMALL, EDGES, None), (SMALL, EDGES + [40], None), (SMALL_G5, EDGES[5:8], None),
    (SMALL_G5, EDGES[9:13], "sym_noz"), (ONE_KV, [1200, 31, 640], None), (ONE_KV, [1200, 31, 640], "asym"),
    (NORM, EDGES[3:8], None), (NORM, EDGES[3:8], "asym"), (SMALL_BIAS, [70, 5, 257], None), (SMALL_BIAS, [70, 5, 257], "asym")],
    ids=lambda v: v.name if hasattr(v, "name") else f"{len(v)}rows" if isinstance(v, list) else str(v))
def test_all_layers_in_one_launch(H, shape, lens, quant):
    case = make_case(H, shape, lens, quant)
    assert takes_one_launch(case) == (len(lens) <= 16)
    pool0 = case.pool_mem.clone()
    ref = H.run_oracle(case, list(range(len(lens))))
    got = []
    for flags, host_lens in ((0, True), (0, False), (sun.SUN_PROFILE, True)):
        case.pool_mem.copy_(pool0)
        case.ws.fill_(0xFF)              # NaN everywhere: nothing is taken from the call before
        case.logits.fill_(float("nan"))
        case.step(flags=flags, host_lens=host_lens)
        got.append((case.logits.clone(), case.pool_mem.clone()))
        H.check_logits(case.logits.cpu().numpy(), ref["logits"], "bf16")
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    bound = (5e-3 if quant else 2e-3) * shape.n_layers ** 0.5
    assert rel(got[0][0], got[2][0]) <= bound
    # the same slots of the pool, with values a rounding step of bf16 apart at most (a few steps where they nearly cancel)
    a, b, o = (t.view(torch.int16) for t in (got[0][1], got[2][1], pool0))
    assert torch.equal(a != o, b != o) or int(((a != o) != (b != o)).sum()) <= 2   # a new entry may equal the old content
    assert rel(got[0][1], got[2][1]) <= 2e-3


@pytest.mark.parametrize("rows,layers,quant,taken", [(1, 1, None, False), (1, 2, None, True), (8, 2, None, False), (8, 3, None, True), (12, 3, None, False), (12, 4, None, True),
                                                     (16, 6, None, False), (16, 7, None, True), (17, 48, None, False), (1, 2, "asym", False), (1, 3, "asym", True),
                                                     (5, 3, "asym", False), (5, 4, "asym", True), (8, 6, "asym", False), (8, 7, "asym", True), (9, 48, "asym", False)])
def test_few_layers_take_a_launch_per_operation(H, rows, layers, quant, taken):
    """Where the one launch costs more than its layers save: then bit for bit the launches that SUN_PROFILE asks for."""
    case = make_case(H, dataclasses.replace(DEEP, name="rule", n_layers=layers), [40] * rows, quant)
    assert takes_one_launch(case) == taken
    if not taken:
        pool0, got = case.pool_mem.clone(), []
        for flags in (0, sun.SUN_PROFILE):
            case.pool_mem.copy_(pool0)
            case.step(flags=flags)
            got.append((case.logits.clone(), case.pool_mem.clone().view(torch.int16)))
        assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


def test_a_row_does_not_depend_on_the_rows_beside_it(H):
    """Same row index and row count; every other row replaced."""
    case = make_case(H, SMALL, EDGES)
    pool0 = case.pool_mem.clone()
    case.step()
    base = case.logits.clone()
    rng = np.random.default_rng(5)
    for keep in (0, 11, 15):
        toks, lens = case.work.tokens.copy(), case.work.seq_lens.copy()
        for i in range(len(lens)):
            if i != keep:
                toks[i], lens[i] = rng.integers(0, SMALL.vocab), rng.integers(0, lens[i] + 1)
        case.pool_mem.copy_(pool0)
        case.step(tokens=torch.from_numpy(toks).to(H.DEV), lens=torch.from_numpy(lens).to(H.DEV))
        assert torch.equal(case.logits[keep], base[keep])


@pytest.mark.parametrize("shape,lens,quant", [(DEEP, [33, 64], None), (DEEP_W4, [33, 64], "asym")], ids=["bf16", "w4"])
def test_more_layers_than_one_launch_takes(H, shape, lens, quant):
    case, rows = make_case(H, shape, lens, quant), [0, 1]
    assert takes_one_launch(case)
    extracted = H.case_extract_pool(case, rows)
    case.step()
    check_against_oracle(H, case, rows, extracted, quant)
    # a gain of the layer that the second launch begins with taken from the layer before it, in the oracle: noticed
    case.w["g1"][48] = case.w["g1"][47]
    with pytest.raises(AssertionError):
        check_against_oracle(H, case, rows, extracted, quant)


@pytest.mark.parametrize("quant", [None, "asym"])
def test_tiles_that_are_written_again(H, quant):
    """A stack so deep that its tiles do not all fit: against the oracle layer by layer, twice in a row the same, and the workspace that
    is asked for is the one that is used."""
    shape = dataclasses.replace(DEEP_W4 if quant else DEEP, name="deeper", n_layers=90)
    case = make_case(H, shape, EDGES[3:11] if quant else EDGES, quant)
    assert takes_one_launch(case)
    pool0 = case.pool_mem.clone()
    need = case.ws.numel()
    guard = torch.full((need + 4096,), 0xA5, dtype=torch.uint8, device=H.DEV)
    case.ws = guard[:need]
    rows, got = [0, 5, 7] if quant else [0, 7, 8, 15], []
    extracted = H.case_extract_pool(case, rows)
    for _ in range(2):
        case.pool_mem.copy_(pool0)
        case.step()
        got.append((case.logits.clone(), bits(case.pool_mem)))
    assert all(torch.equal(a, b) for a, b in zip(*got)) and bool((guard[need:] == 0xA5).all())
    check_against_oracle(H, case, rows, extracted, quant)


@pytest.mark.parametrize("lens,layers,quant", [([1500], 2, None), (EDGES, 7, None), ([900, 3, 64, 2000, 255], 4, "asym")], ids=["1-bf16", "16-bf16", "5-w4"])
def test_widths_of_the_8b_shape(H, lens, layers, quant):
    """Units of every phase as the 8B shape has them; the bf16 weights exceed 256 MB, so they stream past the caches (a kernel of
    its own)."""
    shape = dataclasses.replace(wl.LLAMA_8B, name="8b_widths", n_layers=layers, vocab=2048)
    case = make_case(H, shape, lens, quant)
    assert quant or sun.sun_weights_pack_bytes(case.cfg) > 256 << 20
    assert takes_one_launch(case)
    rows = sorted({0, len(lens) // 2, len(lens) - 1})
    extracted = H.case_extract_pool(case, rows)
    case.step()
    check_against_oracle(H, case, rows, extracted, quant)


@pytest.mark.parametrize("lens", [[40], EDGES[4:11], EDGES[6:14]], ids=lambda v: f"{len(v)}rows")
def test_more_4_bit_gate_up_blocks_than_workgroups(H, lens):
    """272 blocks of every other strip, so that sixteen workgroups finish two; one row, seven, and the eight whose planes fill an operand."""
    shape = dataclasses.replace(DEEP_W4, name="wide_ffn", n_layers=7, ffn=17408)
    case = make_case(H, shape, lens, "asym")
    assert takes_one_launch(case)
    rows = sorted({0, len(lens) // 2, len(lens) - 1})
    extracted = H.case_extract_pool(case, rows)
    case.step()
    check_against_oracle(H, case, rows, extracted, "asym")


def test_under_capture_a_step_takes_a_launch_per_operation(H):
    case = make_case(H, SMALL, [5, 100, 300])
    pool0 = case.pool_mem.clone()
    case.step(flags=sun.SUN_PROFILE)
    want = case.logits.clone()
    case.step(host_lens=True)             # everything is loaded before the capture
    lens = case.lens.cpu().numpy()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sun.sun_decode_step(case.pool, case.weights, case.tokens, case.tables, case.lens, case.ids, case.logits, case.next, case.ws,
                            seq_lens_host=lens)
    for _ in range(3):
        case.pool_mem.copy_(pool0)
        case.logits.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(case.logits, want)
        case.step()                       # an eager step between the replays


@pytest.mark.parametrize("words,one", [([0xFFFFFFFF] * 8, True), ([0xFFFFFFFF] * 4 + [0] * 4, False), ([0xFFFFFFFE] + [0xFFFFFFFF] * 7, False)],
                         ids=["all", "half", "all-but-one"])
def test_a_stream_confined_to_some_compute_units_takes_a_launch_per_operation(H, words, one):
    """The launch needs a workgroup on every compute unit, which such a stream cannot give it."""
    case = make_case(H, SMALL, [5, 100, 300])
    pool0 = case.pool_mem.clone()
    case.step(flags=0 if one else sun.SUN_PROFILE)
    want, pool = case.logits.clone(), bits(case.pool_mem)
    case.pool_mem.copy_(pool0)
    case.logits.fill_(float("nan"))
    lens = case.lens.cpu().numpy()
    torch.cuda.synchronize()
    hip, stream = ctypes.CDLL("libamdhip64.so"), ctypes.c_void_p()
    hip.hipExtStreamCreateWithCUMask.argtypes = [ctypes.POINTER(ctypes.c_void_p), ctypes.c_uint32, ctypes.POINTER(ctypes.c_uint32)]
    hip.hipStreamSynchronize.argtypes = hip.hipStreamDestroy.argtypes = [ctypes.c_void_p]
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(stream), 8, (ctypes.c_uint32 * 8)(*words)) == 0
    try:
        sun.sun_decode_step(case.pool, case.weights, case.tokens, case.tables, case.lens, case.ids, case.logits, case.next, case.ws,
                            seq_lens_host=lens, stream=stream.value)
        assert hip.hipStreamSynchronize(stream) == 0
        assert torch.equal(case.logits, want) and torch.equal(bits(case.pool_mem), pool)
    finally:
        hip.hipStreamDestroy(stream)


def test_steps_on_two_streams_from_two_threads(H):
    """Two such launches do not fit the chip together: they run one behind the other, each with counters in its own workspace."""
    cases = [make_case(H, SMALL, EDGES[:8], seed=s) for s in (710, 720)]
    pools = [c.pool_mem.clone() for c in cases]
    want = []
    for c in cases:
        c.step()
        torch.cuda.synchronize()
        want.append(c.logits.clone())
    got, streams = [[], []], [torch.cuda.Stream(), torch.cuda.Stream()]

    def work(i):
        with torch.cuda.stream(streams[i]):
            for _ in range(10):
                c = cases[i]
                c.pool_mem.copy_(pools[i])
                sun.sun_decode_step(c.pool, c.weights, c.tokens, c.tables, c.lens, c.ids, c.logits, c.next, c.ws, seq_lens_host=lens)
                got[i].append(c.logits.clone())

    lens = np.asarray(EDGES[:8], dtype=np.int32)
    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert [len(g) for g in got] == [10, 10]
    for w, g in zip(want, got):
        assert all(torch.equal(w, x) for x in g)


@pytest.mark.parametrize("shape,quant", [(SMALL, None), (SMALL, "asym"), (DEEP, None)], ids=["small", "small-w4", "two-launches"])
def test_a_wait_that_gives_up_is_reported(H, shape, quant):
    """The wait made to give up after few polls, which some workgroups then do and some do not: either the step is the usual one, or it has no
    result (next -1, logits not-a-numbers) and every cache entry is the old one or the right one; the next step on the same
    workspace is the usual one again."""
    case = make_case(H, shape, EDGES[2:8], quant)
    pool0 = case.pool_mem.clone()
    case.step()
    torch.cuda.synchronize()
    logits, nxt, pool = case.logits.clone(), case.next.clone(), bits(case.pool_mem)
    for polls in (0, 1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 32, 48, 64, 0):
        case.pool_mem.copy_(pool0)
        case.logits.fill_(7.0)
        case.next.fill_(-7)
        case.step(flags=sun.SUN_WAIT_POLLS(polls))
        torch.cuda.synchronize()
        lost = bool((case.next == -1).all())
        assert lost or torch.equal(case.next, nxt)
        assert lost or polls > 0
        assert bool(torch.isnan(case.logits).all()) if lost else torch.equal(case.logits, logits)
        after = bits(case.pool_mem)
        assert bool(((after == pool) | (after == bits(pool0))).all())
        case.pool_mem.copy_(pool0)
        case.step()
        torch.cuda.synchronize()
        assert torch.equal(case.logits, logits) and torch.equal(case.next, nxt) and torch.equal(bits(case.pool_mem), pool)


@pytest.mark.parametrize("polls", [0, 4, 20])
def test_a_run_goes_on_behind_a_step_without_a_result(H, polls):
    lens0, steps = [3, 15, 60, 100], 6
    case = make_case(H, SMALL, lens0, seed=730, spare=6)
    pool0, got = case.pool_mem.clone(), []
    for flags in (0, sun.SUN_WAIT_POLLS(polls)):
        case.pool_mem.copy_(pool0)
        tok, tab, ln = case.tokens.clone(), torch.full((4, 12), -1, dtype=torch.int32, device=H.DEV), case.lens.clone()
        tab[:, :case.tables.shape[1]] = case.tables
        free = torch.arange(case.work.n_pages - 6, case.work.n_pages, dtype=torch.int32, device=H.DEV)
        start = (tok.clone(), tab.clone(), ln.clone())
        head, status = torch.zeros(1, dtype=torch.int32, device=H.DEV), torch.full((1,), 9, dtype=torch.int32, device=H.DEV)
        out = torch.full((steps, 4), -7, dtype=torch.int32, device=H.DEV)
        ws = torch.empty(sun.sun_workspace_bytes(case.cfg, 4, 12), dtype=torch.uint8, device=H.DEV)
        sun.sun_decode_run(case.pool, case.weights, steps, tok, tab, ln, case.ids, free, head, status, out, case.logits, ws, flags=flags)
        torch.cuda.synchronize()
        got.append((out.cpu(), int(status), ln.cpu(), tok.cpu(), tab.cpu(), int(head), bits(case.pool_mem)))
    (want, ok, *_), (out, status, ln, tok, tab, head, pool) = got
    lost = (out == -1).all(1)
    done = int((~lost).sum())
    assert ok & 4 == 0 and bool((want >= 0).all())
    assert torch.equal(out[~lost], want[:done]) and bool(((out == -1).any(1) == lost).all())
    assert (status & 4 != 0) == bool(lost.any())
    if polls == 0:
        assert done == 0 and head == 0
        for a, b in zip((tok, tab, ln), start):
            assert torch.equal(a, b.cpu())
    assert bool(((pool == got[0][6]) | (pool == bits(pool0))).all())


def test_serving_goes_on_behind_steps_without_a_result(H):
    from test_gpu_serve import _Setup
    S = _Setup(H, SMALL, "bf16", 4, [5, 30, 64, 1, 17], [4, 7, 3, 5, 6], 12, 8, seed=21)
    got = []
    for lose in (False, True):
        S.case.pool_mem.copy_(torch.from_numpy(S.before.view(np.int16)).cuda().view(torch.bfloat16))
        state = sun.ServeTensors(S.slots, S.cols, S.waiting, S.ring, S.n_pages, S.idle)
        ws = torch.empty(sun.sun_serve_workspace_bytes(S.case.cfg, S.slots, S.cols), dtype=torch.uint8, device=H.DEV)

        def serve(n, flags):
            toks, reqs = (torch.full((n, S.slots), -7, dtype=torch.int32, device=H.DEV) for _ in range(2))
            sun.sun_decode_serve(S.case.pool, S.case.weights, n, state, toks, reqs, S.case.logits, ws, flags=flags)
            torch.cuda.synchronize()
            return toks, reqs
        if lose:
            toks, reqs = serve(3, sun.SUN_SERVE_RESET | sun.SUN_WAIT_POLLS(0))
            assert bool((toks == -1).all()) and bool((reqs == -1).all())
            c = state.counters.cpu().numpy()
            assert c[3] == 4 and c[4] == 0 and c[6] == 0 and c[7] == 3
        toks, reqs = serve(6, 0 if lose else sun.SUN_SERVE_RESET)
        got.append((toks, reqs, state.seq_lens.clone(), state.page_tables.clone(), state.counters.clone(), bits(S.case.pool_mem)))
    for i in (0, 1, 2, 3, 5):
        assert torch.equal(got[0][i], got[1][i])
    a, b = (g[4].cpu().numpy() for g in got[:2])
    assert list(a[[0, 1, 2, 4, 5, 6]]) == list(b[[0, 1, 2, 4, 5, 6]]) and b[3] == a[3] | 4 and b[7] == a[7] + 3
