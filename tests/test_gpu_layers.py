"""A step of few requests runs all layers in one launch.  Checked where that can go wrong: row counts around the eight that a wave
each finishes and the largest taken, one row beyond it, lengths around chunk and page boundaries, matrices with fewer
column blocks than compute units, more layers than one launch takes, head norm, biases, both 4-bit layouts.  Against the oracle, and
against a launch per operation (which SUN_PROFILE asks for)."""
import dataclasses
import threading

import numpy as np
import pytest
import torch

from paper_2603_02599_amd import binding as sun, workloads as wl

pytestmark = pytest.mark.gpu

DEEP = dataclasses.replace(wl.SMALL128, name="deep", n_layers=50, hidden=256, n_q_heads=2, n_kv_heads=1, ffn=256, vocab=512)
NORM = dataclasses.replace(wl.SMALL128, name="norm", qk_norm=True)
ONE_KV = dataclasses.replace(wl.SMALL128, name="one_kv", hidden=384, n_q_heads=8, n_kv_heads=1, ffn=640)
EDGES = [0, 1, 15, 16, 17, 62, 63, 64, 65, 127, 128, 129, 255, 256, 300, 511]


@pytest.fixture(scope="module")
def H():
    import gpu_harness
    assert torch.cuda.is_available(), "these tests need the MI355X"
    sun.lib()
    return gpu_harness


def make_case(H, shape, lens, quant=None, seed=700):
    work = wl.make_workload("cfg1", shape=shape, dtype="bf16", batch=len(lens), seed=seed + len(lens))
    work.seq_lens = np.asarray(lens, dtype=np.int32)
    work.page_tables, work.n_pages = wl.deal_page_tables(work.seq_lens, np.random.default_rng(seed))
    return H.GpuCase(work, quant_mode=quant)


def rel(a, b):
    a, b = a.double(), b.double()
    return float((a - b).norm() / b.norm())


# Two correct sums of these products differ by 1e-5 (bf16) and 3e-4 (4-bit: 16 bits a group) of the logits.  Where a new cache entry
# falls on the other side of a bf16 rounding it differs by up to 2^-8 of itself, and for a request of one position
# that is an element of attention's output: ten such among the 256 of a row's K or V are 2^-8 sqrt(10 / 256) = 8e-4 of the row.
# Twice that, and for 4-bit weights ten times their 3e-4 beside it.
@pytest.mark.parametrize("shape,lens,quant", [
    (wl.SMALL128, [300], None), (wl.SMALL128, [0], "asym"), (wl.SMALL128, EDGES[:8], None), (wl.SMALL128, EDGES[8:], "asym"),
    (wl.SMALL128, EDGES[7:], None), (wl.SMALL128, EDGES, None), (wl.SMALL128, EDGES + [40], None), (wl.SMALL_G5, EDGES[5:8], None),
    (wl.SMALL_G5, EDGES[9:13], "sym_noz"), (ONE_KV, [1200, 31, 640], None), (ONE_KV, [1200, 31, 640], "asym"),
    (NORM, EDGES[3:8], None), (NORM, EDGES[3:8], "asym"), (wl.SMALL_BIAS, [70, 5, 257], None), (wl.SMALL_BIAS, [70, 5, 257], "asym"),
    (DEEP, [33, 64], None)],
    ids=lambda v: v.name if hasattr(v, "name") else f"{len(v)}rows" if isinstance(v, list) else str(v))
def test_all_layers_in_one_launch(H, shape, lens, quant):
    case = make_case(H, shape, lens, quant)
    pool0 = case.pool_mem.clone()
    ref = H.run_oracle(case, list(range(len(lens)))) if shape is not DEEP else None
    got = []
    for flags, host_lens in ((0, True), (0, False), (sun.SUN_PROFILE, True)):
        case.pool_mem.copy_(pool0)
        case.ws.fill_(0xFF)              # NaN everywhere: nothing is taken from the call before
        case.logits.fill_(float("nan"))
        case.step(flags=flags, host_lens=host_lens)
        got.append((case.logits.clone(), case.pool_mem.clone()))
        if ref is not None:
            H.check_logits(case.logits.cpu().numpy(), ref["logits"], "bf16")
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    bound = 5e-3 if quant else 2e-3
    assert rel(got[0][0], got[2][0]) <= (bound if shape is not DEEP else 20 * bound)   # rounded entries travel through 50 layers
    # the same slots of the pool, with values a rounding step of bf16 apart at most (a few steps where they nearly cancel)
    a, b, o = (t.view(torch.int16) for t in (got[0][1], got[2][1], pool0))
    assert torch.equal(a != o, b != o) or int(((a != o) != (b != o)).sum()) <= 2   # a new entry may equal the old content
    assert rel(got[0][1], got[2][1]) <= 2e-3


def test_a_row_does_not_depend_on_the_rows_beside_it(H):
    """Same row index and row count; every other row replaced."""
    case = make_case(H, wl.SMALL128, EDGES)
    pool0 = case.pool_mem.clone()
    case.step()
    base = case.logits.clone()
    rng = np.random.default_rng(5)
    for keep in (0, 11, 15):
        toks, lens = case.work.tokens.copy(), case.work.seq_lens.copy()
        for i in range(len(lens)):
            if i != keep:
                toks[i], lens[i] = rng.integers(0, wl.SMALL128.vocab), rng.integers(0, lens[i] + 1)
        case.pool_mem.copy_(pool0)
        case.step(tokens=torch.from_numpy(toks).to(H.DEV), lens=torch.from_numpy(lens).to(H.DEV))
        assert torch.equal(case.logits[keep], base[keep])


@pytest.mark.parametrize("quant", [None, "asym"])
def test_tiles_that_are_written_again(H, quant):
    """A stack so deep that its tiles do not all fit: the same as a launch per operation, twice in a row, and the workspace that is
    asked for is the one that is used."""
    shape = dataclasses.replace(DEEP, name="deeper", n_layers=90)
    case = make_case(H, shape, EDGES[3:11] if quant else EDGES, quant)
    pool0 = case.pool_mem.clone()
    need = case.ws.numel()
    guard = torch.full((need + 4096,), 0xA5, dtype=torch.uint8, device=H.DEV)
    case.ws = guard[:need]
    got = []
    for flags in (0, 0, sun.SUN_PROFILE):
        case.pool_mem.copy_(pool0)
        case.step(flags=flags)
        got.append(case.logits.clone())
    assert torch.equal(got[0], got[1]) and bool((guard[need:] == 0xA5).all())
    assert rel(got[0], got[2]) <= 40 * (5e-3 if quant else 2e-3)   # rounded entries travel through 90 layers


def test_under_capture_a_step_takes_a_launch_per_operation(H):
    case = make_case(H, wl.SMALL128, [5, 100, 300])
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


def test_steps_on_two_streams_from_two_threads(H):
    """Two such launches do not fit the chip together: they run one behind the other, each with counters in its own workspace."""
    cases = [make_case(H, wl.SMALL128, EDGES[:8], seed=s) for s in (710, 720)]
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
