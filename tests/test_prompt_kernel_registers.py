"""The prompt GEMM requests its LDS fragments in inline assembly and waits for them in separate statements, so the compiler
takes a fragment's registers as written while the read is still in flight.  That is sound only as long as the compiled code
leaves those registers alone until the wait: no copy, spill, reuse or second request, on any path (the stage loop's back edge
above all).  This test compiles the kernels for gfx950 (no GPU needed) and follows every such read through the control flow.

LDS reads of a wave return in the order of their issue and s_waitcnt lgkmcnt(n) leaves at most n outstanding, so a read has
arrived at a wait whose n is at most the number of LDS operations issued after it.  Scalar loads count in lgkmcnt too; leaving
them out can only make the check stricter."""
import os
import re
import subprocess

import pytest

from paper_2503_08524_amd import build as d3_build

VGPR = re.compile(r"\bv(?:\[(\d+):(\d+)\]|(\d+)\b)")
WAIT = re.compile(r"lgkmcnt\((\d+)\)")


def registers(text):
    out = set()
    for lo, hi, one in VGPR.findall(text):
        out |= {int(one)} if one else set(range(int(lo), int(hi) + 1))
    return out


def blocks_of(lines):
    """[(label, [(line number, instruction, inside inline assembly)])] of one function, in layout order."""
    blocks, asm = [("entry", [])], False
    for no, raw in lines:
        if "#ASMSTART" in raw or "#ASMEND" in raw:
            asm = "#ASMSTART" in raw
            continue
        text = raw.split(";")[0].strip()
        if text.endswith(":"):
            blocks.append((text[:-1], []))
        elif text and not text.startswith("."):
            blocks[-1][1].append((no, text, asm))
    return blocks


def faults(lines):
    """Uses of registers that an inline-assembly LDS read may still be writing."""
    blocks = blocks_of(lines)
    index = {label: i for i, (label, _) in enumerate(blocks)}
    entry = [None] * len(blocks)                       # per block: register -> fewest LDS operations issued after the read that writes it
    entry[0] = {}
    work, found, n_reads = [0], {}, set()

    def flow(to, state):
        old = entry[to]
        new = dict(state) if old is None else {r: min(old.get(r, 99), state.get(r, 99)) for r in old.keys() | state.keys()}
        if new != old:
            entry[to] = new
            work.append(to)

    while work:
        i = work.pop()
        state, falls = dict(entry[i]), True
        for no, text, asm in blocks[i][1]:
            op = text.split()[0]
            wait = WAIT.search(text)
            if op == "s_waitcnt" and wait:
                state = {r: k for r, k in state.items() if k < int(wait.group(1))}
                continue
            hit = registers(text) & state.keys()
            if hit:
                found[no] = f"line {no}: `{text}` touches v{sorted(hit)} in flight"
            if op.startswith("ds_"):
                state = {r: min(k + 1, 99) for r, k in state.items()}
                if asm and op.startswith("ds_read"):
                    n_reads.add(no)
                    state.update({r: 0 for r in registers(text.split(",")[0])})
            if op.startswith("s_cbranch") or op == "s_branch":
                flow(index[text.split()[1]], state)
                falls = op != "s_branch"
            if op == "s_endpgm":
                falls = False
            if not falls:
                break
        if falls and i + 1 < len(blocks):
            flow(i + 1, state)
    return list(found.values()), len(n_reads)


def listing(text):
    return list(enumerate(text.strip().splitlines(), 1))


READ = ";#ASMSTART\nds_read_b128 v[{0}:{1}], v9 offset:0\n;#ASMEND\n"


@pytest.mark.parametrize("text,n_faults", [
    (READ.format(0, 3) + "s_waitcnt lgkmcnt(0)\nv_mov_b32 v20, v1\ns_endpgm", 0),
    (READ.format(0, 3) + "v_mov_b32 v20, v1\ns_waitcnt lgkmcnt(0)\ns_endpgm", 1),                          # read too early
    (READ.format(0, 3) + "v_mov_b32 v2, v20\ns_waitcnt lgkmcnt(0)\ns_endpgm", 1),                          # overwritten
    (READ.format(0, 3) + READ.format(4, 7) + "s_waitcnt lgkmcnt(1)\nv_mov_b32 v20, v1\ns_endpgm", 0),      # the older one is there ...
    (READ.format(0, 3) + READ.format(4, 7) + "s_waitcnt lgkmcnt(1)\nv_mov_b32 v20, v5\ns_endpgm", 1),      # ... the newer one is not
    (READ.format(0, 3) + READ.format(3, 6) + "s_waitcnt lgkmcnt(0)\ns_endpgm", 1),                         # two reads into one register
    (READ.format(6, 9) + READ.format(0, 3) + "s_waitcnt lgkmcnt(0)\ns_endpgm", 1),                         # an address still in flight
    (".L1:\ns_waitcnt lgkmcnt(0)\nv_mov_b32 v20, v1\n" + READ.format(0, 3) + "s_cbranch_scc1 .L1\ns_waitcnt lgkmcnt(0)\ns_endpgm", 0),
    (".L1:\nv_mov_b32 v20, v1\ns_waitcnt lgkmcnt(0)\n" + READ.format(0, 3) + "s_cbranch_scc1 .L1\ns_waitcnt lgkmcnt(0)\ns_endpgm", 1),   # over the back edge
    (READ.format(0, 3) + "s_cbranch_scc0 .L2\ns_waitcnt lgkmcnt(0)\n.L2:\nv_mov_b32 v20, v1\ns_endpgm", 1),                              # one path waits
    (READ.format(0, 3) + "s_cbranch_scc0 .L2\n" + READ.format(4, 7) + ".L2:\ns_waitcnt lgkmcnt(1)\nv_mov_b32 v20, v1\ns_endpgm", 1),     # fewer reads behind it on one
])
def test_the_check_itself(text, n_faults):
    assert len(faults(listing(text))[0]) == n_faults


@pytest.fixture(scope="module")
def compiled(tmp_path_factory):
    """(lines of the compiled file, {kernel: its lines})."""
    out = str(tmp_path_factory.mktemp("prompt") / "gemm_prompt.s")
    src = os.path.join(d3_build.CSRC, "gemm_prompt.hip")
    r = subprocess.run([d3_build.HIPCC] + d3_build.FLAGS + ["-x", "hip", "--cuda-device-only", "-S", src, "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    lines = listing(open(out).read())
    starts = [(i, raw.split(":")[0]) for i, (_, raw) in enumerate(lines) if re.match(r"_Z\w+:", raw)]
    kernels = {name: lines[i + 1:end] for (i, name), end in zip(starts, [i for i, _ in starts[1:]] + [len(lines)])}
    kernels = {n: [ln for ln in body] for n, body in kernels.items() if "gemm_prompt_kernel" in n or "mfma_yardstick_kernel" in n}
    assert len(kernels) == 7
    return lines, kernels


def test_yardstick_issues_the_planes_of_an_accumulator_back_to_back(compiled):
    # the order that the prompt kernel uses and that draws least power: a bound for it has to be measured in that order
    for name, body in compiled[1].items():
        if "mfma_yardstick" not in name:
            continue
        issued = [re.search(r"v_mfma\S+ (\S+), \S+, \S+, (\S+)", raw) for _, raw in body]
        issued = [m.groups() for m in issued if m]
        assert len(issued) == 64, name
        assert all(hi[0] == lo[1] for hi, lo in zip(issued[::2], issued[1::2])), name


def test_fragments_in_flight_are_left_alone(compiled):
    lines, kernels = compiled
    for name, body in kernels.items():
        end = next(i for i, (_, raw) in enumerate(body) if raw.strip().startswith(".section"))
        found, n_reads = faults(body[:end])
        print(name, n_reads, "reads")
        assert n_reads >= (100 if "gemm_prompt" in name else 12), name
        assert not found, f"{name}:\n" + "\n".join(found)
    text = "\n".join(raw for _, raw in lines)
    for what in ("vgpr_spill_count", "sgpr_spill_count", "private_segment_fixed_size"):
        assert set(re.findall(rf"\.{what}:\s+(\d+)", text)) == {"0"}, what


def step_loops(lines):
    """The innermost loops that multiply: (lines of the body)."""
    labels = {raw.split(":")[0]: i for i, (_, raw) in enumerate(lines) if re.match(r"\.LBB\w+:", raw)}
    loops = []
    for i, (_, raw) in enumerate(lines):
        m = re.search(r"s_c?branch\w* (\.LBB\w+)", raw)
        if m and labels.get(m.group(1), i) < i:
            loops.append([t for _, t in lines[labels[m.group(1)]:i]])
    loops = [b for b in loops if any("v_mfma" in t for t in b)]
    return [b for b in loops if not any(len(o) < len(b) and set(o) <= set(b) for o in loops)]


def test_fragments_in_flight_are_left_alone_in_the_kernel_of_the_larger_tiles(tmp_path):
    # the same for the tiles of 256 columns: four steps of 16 reads each are written out (the last one of 6), and the first reads of a tile.  No vector register is spilled, but
    # all of them are taken and scalars (buffer descriptors, the plan of the next tile) are kept in lanes of a few of them: between tiles, and in the loop over steps only QKV's
    # descriptors of three matrices, four times each way in 128 MFMAs
    out = str(tmp_path / "gemm_prompt_256.s")
    src = os.path.join(d3_build.CSRC, "gemm_prompt_256.hip")
    r = subprocess.run([d3_build.HIPCC] + d3_build.FLAGS + ["-x", "hip", "--cuda-device-only", "-S", src, "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    text = open(out).read()
    lines = listing(text)
    starts = [(i, raw.split(":")[0]) for i, (_, raw) in enumerate(lines) if re.match(r"_Z\w+gemm_prompt_256_kernel\w+:", raw)]
    assert len(starts) == 3
    for i, name in starts:
        end = next(k for k in range(i + 1, len(lines)) if lines[k][1].strip().startswith(".section"))
        found, n_reads = faults(lines[i + 1:end])
        print(name, n_reads, "reads")
        assert n_reads >= 60, name
        assert not found, f"{name}:\n" + "\n".join(found)
        loops = step_loops(lines[i + 1:end])
        assert len(loops) == 1 and sum("v_mfma" in t for t in loops[0]) == 128, name
        lanes = sum("v_readlane" in t or "v_writelane" in t for t in loops[0])
        assert lanes <= (8 if "ILi3E" in name else 0), f"{name}: {lanes}"
    for what in ("vgpr_spill_count", "private_segment_fixed_size"):
        assert set(re.findall(rf"\.{what}:\s+(\d+)", text)) == {"0"}, what
