"""What the compiler makes of device code whose correctness it cannot see: requests from memory straight into LDS are
written as inline assembly, and waits for them are counted by hand.  The sources are compiled to assembly here (no GPU) and read."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2603_02599_amd", "csrc")


def assembly(src, out):
    """kernel name -> its instructions, one string each, labels included"""
    from paper_2603_02599_amd.build import FLAGS
    flags = [f for f in FLAGS if f != "-fPIC"]
    subprocess.run(["hipcc", *flags, "--offload-device-only", "-S", str(src), "-o", str(out)], check=True, capture_output=True)
    return instructions(out)


def instructions(out):
    kernels, name = {}, None
    for line in open(out):
        line = line.split(";")[0].strip()
        m = re.fullmatch(r"(_Z\w+):", line)
        if m:
            name = m.group(1)
            kernels[name] = []
        elif line.startswith(".Lfunc_end"):
            name = None
        elif name and line and not line.startswith("."):
            kernels[name].append(line)
        elif name and re.fullmatch(r"\.LBB\w+:", line):
            kernels[name].append(line)
    return kernels


PROBE = r"""
#include "common.hpp"
using namespace sun;
typedef __attribute__((address_space(3))) unsigned lds_t;
typedef __attribute__((address_space(1))) const void* global_t;
__global__ void probe_m0(const unsigned* a, const unsigned* b, unsigned* out) {
    __shared__ unsigned buf[1024];
    const int lane = threadIdx.x & 63;
    lds_t* l = (lds_t*)buf;
    __builtin_amdgcn_global_load_lds((global_t)(a + lane), l, 4, 0, 0);
    REQUEST(b, lane * 4, (uint32_t)(uintptr_t)l + 2048);
    __builtin_amdgcn_global_load_lds((global_t)(a + 64 + lane), l, 4, 256, 0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    out[lane] = buf[lane] + buf[lane + 64] + buf[lane + 512];
}
"""


@pytest.mark.parametrize("request_fn", ["lds_dma4", "lds_dma16"])
def test_a_request_into_lds_owns_m0(tmp_path, request_fn):
    """The statement overwrites m0: code around it that uses m0 has to set it again."""
    src = tmp_path / "probe.hip"
    src.write_text(PROBE.replace('"common.hpp"', f'"{CSRC}/common.hpp"').replace("REQUEST", request_fn))
    code = next(v for n, v in assembly(src, tmp_path / "probe.s").items() if "probe_m0" in n)
    uses = [i for i, s in enumerate(code) if s.startswith("global_load_lds")]
    sets = [i for i, s in enumerate(code) if re.match(r"s_\w+ m0\b", s)]
    assert len(uses) == 3
    for a, b in zip([-1] + uses, uses):
        assert any(a < i < b for i in sets), "a request without m0 of its own"


def registers(operand):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]|s(\d+)", operand)
    return set() if not m else {int(m[3])} if m[3] else set(range(int(m[1]), int(m[2]) + 1))


def late_writers(code):
    """Requests into LDS whose base a vector instruction wrote fewer than five wait states before, on any path."""
    label = {s[:-1]: i for i, s in enumerate(code) if s.endswith(":")}
    before = [[] for _ in code]
    for i, s in enumerate(code):
        if s.startswith(("s_branch", "s_cbranch")):
            before[label[s.split()[1]]].append(i)
        if i + 1 < len(code) and not s.startswith(("s_branch", "s_endpgm")):
            before[i + 1].append(i)
    found = []
    for i, s in enumerate(code):
        if not s.startswith("global_load_lds"):
            continue
        base = registers(re.split(r"[ ,]+", s)[2])
        assert len(base) == 2, s
        todo = [(p, 0, frozenset(base)) for p in before[i]]
        while todo:
            j, states, need = todo.pop()
            t = code[j]
            if not t.endswith(":"):
                operands = re.split(r"[ ,]+", t)[1:]
                written = operands[:2] if "_co_" in t.split()[0] else operands[:1]   # a carry is the second result
                if t.startswith("v_") and any(need & registers(o) for o in written):
                    found.append((t, s, states))
                    continue
                if t.startswith("s_") and operands:
                    need = need - registers(operands[0])
                states += int(operands[0]) + 1 if t.startswith("s_nop") else 1
            if need and states < 5:
                todo += [(p, states, need) for p in before[j]]
    return found


@pytest.mark.parametrize("source", ["proj.hip", "attention.hip"])
def test_requests_into_lds_read_a_base_that_is_there(source, projection_code, attention_code):
    """Five wait states lie between a vector instruction that writes a scalar register and a vector memory instruction that
    reads it; in front of assembly the compiler inserts none, so the kernels' requests have to take their base from
    scalar instructions (or far enough from a lane read)."""
    code = projection_code if source == "proj.hip" else attention_code
    requests = sum(s.startswith("global_load_lds") for v in code.values() for s in v)
    assert requests >= 10
    for name, v in code.items():
        assert not late_writers(v), name
    # the reading itself: a lane read right before a request is noticed, one five states earlier is not
    assert late_writers(["v_readfirstlane_b32 s5, v1", "s_mov_b32 m0, s2", "s_nop 0", "global_load_lds_dword v0, s[4:5]"])
    assert not late_writers(["v_readfirstlane_b32 s5, v1", "s_mov_b32 m0, s2", "s_nop 3", "global_load_lds_dword v0, s[4:5]"])
    assert not late_writers(["v_readfirstlane_b32 s5, v1", "s_mov_b64 s[4:5], s[6:7]", "global_load_lds_dword v0, s[4:5]"])


def fewest_loads_between_waits(code, wait):
    """Over every path from a hand-counted wait (and its barrier) to the next one: the fewest vector loads that follow the
    path's last request into LDS.  None where no path leads from one wait to another."""
    label = {s[:-1]: i for i, s in enumerate(code) if s.endswith(":")}
    at = {i for i, s in enumerate(code) if s == wait and code[i + 1] == "s_barrier"}
    assert at, wait
    fewest = None
    for start in at:
        todo, best = [(start + 2, 0)], {}
        while todo:
            i, n = todo.pop()
            if i >= len(code) or best.get(i, 1 << 30) <= n:
                continue
            best[i] = n
            s = code[i]
            if i in at:
                fewest = n if fewest is None else min(fewest, n)
                continue
            if s.startswith("global_load_lds"):
                n = 0
            elif re.match(r"(global|buffer|flat|scratch)_load", s):
                n += 1
            if s.startswith("s_endpgm"):
                continue
            if s.startswith("s_branch"):
                todo.append((label[s.split()[1]], n))
                continue
            if s.startswith("s_cbranch"):
                todo.append((label[s.split()[1]], n))
            todo.append((i + 1, n))
    return fewest


@pytest.mark.parametrize("waves", [4, 5, 6, 7])
def test_the_4_bit_kernel_waits_for_the_stage_it_reads(projection_code, waves):
    """Its wait counts what is requested behind a stage's fragments: three vector loads (codes and scales), the next stage's
    requests, three loads more.  Were the compiler to merge or move those loads, the wait would be too short: so every way
    round the loop has to hold three of them behind its requests into LDS."""
    per = -(-9 // waves)       # nine requests a stage, shared by the waves
    wait = f"s_waitcnt vmcnt({3 + per + 3})"
    kernels = [v for n, v in projection_code.items() if f"proj_w4_kernelILi{waves}E" in n]
    assert len(kernels) == 3
    for code in kernels:
        assert fewest_loads_between_waits(code, wait) >= 3
        assert not any(s.startswith("scratch_") for s in code)
        loads = [i for i, s in enumerate(code) if s.startswith("global_load_dword") and i > code.index(wait)]
        assert fewest_loads_between_waits(code[:loads[1]] + ["s_nop 0"] + code[loads[1] + 1:], wait) < 3


@pytest.fixture(scope="module")
def projection_code(tmp_path_factory):
    return assembly(os.path.join(CSRC, "proj.hip"), tmp_path_factory.mktemp("asm") / "proj.s")


@pytest.mark.parametrize("epilogue", [0, 1, 2])
@pytest.mark.parametrize("rows,ahead,norm", [(2, 4, 0), (2, 4, 1), (8, 4, 0), (8, 4, 1), (8, 1, 0), (8, 1, 1)])
def test_the_fp32_projection_has_a_step_of_loads_in_flight(projection_code, rows, ahead, norm, epilogue):
    """A step along k is `ahead` times a weight (gate and up: two), the rows' values and the norm's gain, with nothing asked between their
    loads (but whether the last of four lies within k): a question whether the weights are 4-bit, asked at each weight, made a step as many
    round trips as it has of them."""
    found = [v for n, v in projection_code.items() if f"proj_f32_kernelILi{rows}ELi{ahead}ELb{norm}ELi{epilogue}E" in n]
    if (norm, epilogue) == (1, 1):
        assert not found   # the sum behind attention and down has no norm in front
        return
    code, = found
    most = n = 0
    for s in code:
        n = 0 if s.endswith(":") or s.startswith(("s_cbranch", "s_branch")) else n + bool(re.match(r"(global|flat)_load_dword ", s))
        most = max(most, n)
    assert most >= max(1, ahead - 1) * (rows + (2 if epilogue == 2 else 1) + norm)


@pytest.fixture(scope="module")
def attention_file(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm") / "attention.s"
    assembly(os.path.join(CSRC, "attention.hip"), out)
    return out


@pytest.fixture(scope="module")
def attention_code(attention_file):
    return instructions(attention_file)


def test_the_kernel_of_all_layers_keeps_its_registers(tmp_path):
    """It takes nearly the whole register file (one workgroup of eight waves a compute unit): what does not fit would go through
    memory in every layer."""
    kernels = {n: v for n, v in assembly(os.path.join(CSRC, "layers.hip"), tmp_path / "layers.s").items() if "layers_kernel" in n}
    assert len(kernels) == 3
    for name, code in kernels.items():
        assert not any(s.startswith("scratch_") for s in code), name


@pytest.mark.parametrize("dims", [64, 128])
def test_the_short_attention_leaves_room_for_a_second_workgroup(attention_registers, dims):
    """More requests x KV heads than compute units are two workgroups of eight waves on one: four waves a SIMD, 128 of its 512 registers each."""
    (used, spilled), = [v for n, v in attention_registers.items() if f"attn_short_f32_kernelILi{dims}E" in n]
    assert used <= 128 and spilled == 0


@pytest.mark.parametrize("heads", [1, 4, 8])
def test_attention_streams_v_always_and_k_where_it_is_told(attention_code, heads):
    """Sixteen loads of a page pair: eight of K, eight of V; those past the caches are marked."""
    def share(k_read):   # streamed, rows through the caches, in place through the caches
        code, = [v for n, v in attention_code.items() if f"attn_split_kernelILi128ELi{heads}ELNS_5KReadE{k_read}E" in n]
        loads = [s for s in code if s.startswith("global_load_dwordx4") and "lds" not in s]
        return sum(s.endswith(" nt") for s in loads), len(loads)
    streamed, rows, in_place = share(0), share(1), share(2)
    assert streamed[1] == rows[1] == in_place[1] and streamed[0] == 2 * rows[0] == 2 * in_place[0] > 0


@pytest.fixture(scope="module")
def attention_registers(attention_file):
    """kernel name -> its vector registers, how many of them are kept in memory"""
    text = open(attention_file).read()
    found = re.findall(r"\.name:\s+(_Z\w+)\n(?:(?!\.name:).)*?\.vgpr_count:\s+(\d+)\n\s+\.vgpr_spill_count:\s+(\d+)", text, re.S)
    return {n: (int(a), int(b)) for n, a, b in found}
