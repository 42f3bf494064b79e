"""Checks of the gfx950 code that hipcc generates from the kernel sources: what the kernels rely on and the compiler does
not check in hand-written instructions."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2603_11564_amd import build


LDS_BYTES = {}  # of a kernel, without what its launch adds
REGISTERS = {}  # vector and accumulation registers of a kernel


def compile_device(src, out):
    """Compiles one translation unit for the device; returns its assembly (one list of lines per kernel or function) and how
    many vector registers each kernel spills."""
    r = subprocess.run([build._hipcc(), *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, src), "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    functions, current, spills, kernel = {}, None, {}, None
    for line in open(out):
        entry = re.match(r"\s+\.(symbol|vgpr_count|vgpr_spill_count):\s+(\S+)", line)    # of the kernel descriptors at the end
        if entry and entry.group(1) == "symbol":
            kernel = entry.group(2)
            LDS_BYTES[kernel] = lds
        elif entry and entry.group(1) == "vgpr_count":
            REGISTERS[kernel] = int(entry.group(2))
        elif entry:
            spills[kernel] = int(entry.group(2))
        size = re.match(r"\s+\.group_segment_fixed_size:\s+(\d+)", line)     # (stands before the symbol)
        if size:
            lds = int(size.group(1))
        line = line.split(";")[0].split("//")[0].rstrip()
        label = re.match(r"(_Z\w+):", line)
        if label:
            current = functions.setdefault(label.group(1), [])
        elif current is not None and line.strip():
            current.append(line.strip())
    return functions, spills


@pytest.fixture(scope="module")
def units(tmp_path_factory):
    folder = tmp_path_factory.mktemp("device_code")
    with ThreadPoolExecutor(max_workers=6) as pool:
        jobs = {src: pool.submit(compile_device, src, str(folder / (src + ".s"))) for src in build.SOURCES}
        return {src: job.result() for src, job in jobs.items()}


def scalar_registers(operand):
    """The scalar registers that an operand names: "s5", "s[4:5]", "vcc"."""
    operand = operand.strip().strip("-|")
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.fullmatch(r"s(\d+)", operand)
    return {int(m.group(1))} if m else {operand[:3]} if operand in ("vcc", "vcc_lo", "vcc_hi") else set()


def early_reads_of_vector_written_scalars(lines):
    """Vector instructions that read a scalar register (as a carry, a mask or a value) fewer than two wait states after a vector
    instruction wrote it: gfx950 needs two there, and does not check."""
    written, clock, found = {}, 0, []
    for line in lines:
        if line.endswith(":") or line.startswith("."):
            continue
        op, _, rest = line.partition(" ")
        operands = re.findall(r"s\[\d+:\d+\]|v\[\d+:\d+\]|a\[\d+:\d+\]|[^,\s]+", rest)
        clock += 1 if op != "s_nop" else int(operands[0], 0) + 1
        if not op.startswith("v_"):
            if op.startswith("s_") and operands:    # (a scalar write takes the register over)
                for r in scalar_registers(operands[0]):
                    written.pop(r, None)
            continue
        two_results = re.match(r"v_(add|sub|subrev|addc|subb|subbrev)_co_|v_div_scale|v_mad_[ui]64", op) is not None
        n = 2 if two_results else 1
        for operand in operands[n:]:
            if any(clock - written.get(r, -9) <= 2 for r in scalar_registers(operand)):
                found.append(line)
        for operand in operands[:n]:
            for r in scalar_registers(operand):
                written[r] = clock
    return found


def test_the_scan_itself():
    cmp, use = "v_cmp_lt_u32_e32 vcc, s2, v2", "v_addc_co_u32_e32 v0, vcc, v0, v0, vcc"
    assert early_reads_of_vector_written_scalars([cmp, use]) == [use]
    assert early_reads_of_vector_written_scalars([cmp, "s_nop 0", use]) == [use]
    assert early_reads_of_vector_written_scalars([cmp, "s_nop 1", use]) == []
    assert early_reads_of_vector_written_scalars([cmp, "v_mov_b32_e32 v1, v2", "v_mov_b32_e32 v1, v3", use]) == []
    assert early_reads_of_vector_written_scalars(["v_cmp_lt_u32_e64 s[4:5], v1, v2", "v_cndmask_b32_e64 v0, 0, 1, s[4:5]"]) != []
    assert early_reads_of_vector_written_scalars(["v_readfirstlane_b32 s4, v1", "v_add_u32_e32 v0, s4, v0"]) != []
    assert early_reads_of_vector_written_scalars(["v_readfirstlane_b32 s4, v1", "s_mov_b32 s4, 0", "v_add_u32_e32 v0, s4, v0"]) == []


def test_vector_written_scalars_are_read_two_wait_states_later(units):
    """The compiler inserts these waits for its own instructions, not inside inline assembly or around it."""
    early = {f"{src}: {name}": lines[:4] for src, (fs, _) in units.items() for name, body in fs.items()
             if (lines := early_reads_of_vector_written_scalars(body))}
    assert not early, early


def test_no_kernel_spills_vector_registers(units):
    """The waits of the key rings count vector memory operations in the order they were issued: a spilled register's store or
    reload is one more of them, and a reload waits for all that are in flight."""
    spills = {f"{src}: {name}": n for src, (_, kernels) in units.items() for name, n in kernels.items()}
    assert len(spills) > 40 and any("score_wave_pass1_kernel" in name for name in spills)
    assert not {name: n for name, n in spills.items() if n}


def test_waves_of_a_score_walk_have_a_simd_to_themselves(units):
    """A SIMD has 512 registers: two waves fit one from 256 down, and would sit there while other SIMDs have none."""
    walks = {name: n for name, n in REGISTERS.items() if re.search(r"score_(wave_pass[12]|fused)_kernel", name)}
    assert len(walks) > 60 and any("score_fused_kernelILi2E" in name for name in walks)
    assert not {name: n for name, n in walks.items() if n <= 256}


def test_four_workgroups_of_a_large_tile_call_fit_a_compute_unit(units):
    """Calls of more tiles than compute units live from several workgroups to each (make_score_plan): four of 128 keys, with the column
    sums of eight row blocks in pass 2.  (With those of the largest tiles in its static part three fitted: pass 2 of a ragged batch, two
    layers, 32 rows, 80751 keys 68.2 -> 72.6 us, and half of that back with four.)"""
    tile = 128 * 256
    for kernel, launch in (("score_tile_pass1_kernelILb0E", tile), ("score_tile_pass2_kernelILb0ELb0E", tile + 8 * 128 * 4)):
        static, = (n for name, n in LDS_BYTES.items() if kernel in name)
        assert 4 * (static + launch) <= 160 * 1024, (kernel, static)


def basic_blocks(lines):
    """The basic blocks of a function's text: instructions, and the numbers of the blocks that can follow."""
    starts, labels, blocks = [0], {}, []
    for i, line in enumerate(lines):
        if line.endswith(":"):
            starts.append(i)
        elif line.startswith(("s_branch", "s_cbranch", "s_endpgm", "s_setpc")):
            starts.append(i + 1)
    starts = sorted({i for i in starts if i < len(lines)})
    for n, (at, end) in enumerate(zip(starts, starts[1:] + [len(lines)])):
        if lines[at].endswith(":"):
            labels[lines[at][:-1]] = n
        blocks.append([line for line in lines[at:end] if not line.endswith(":") and not line.startswith(".")])
    follow = []
    for n, block in enumerate(blocks):
        last = block[-1] if block else ""
        assert not last.startswith("s_setpc"), "a jump to an address that the text does not name"
        to = [labels[last.split()[1]]] if last.startswith(("s_branch", "s_cbranch")) else []
        if not last.startswith(("s_branch", "s_endpgm")) and n + 1 < len(blocks):
            to.append(n + 1)
        follow.append(to)
    return blocks, follow


def transfers_before_reads_are_done(lines):
    """Transfers from memory into LDS that are issued while reads of LDS may still be queued, on any way through the function: a block
    begins with as many queued as any of the blocks before it may leave."""
    blocks, follow = basic_blocks(lines)

    def run(block, queued, found=None):
        for line in block:
            wait = re.search(r"lgkmcnt\((\d+)\)", line)
            if line.startswith("ds_read"):
                queued = min(queued + 1, 64)
            elif line.startswith("s_waitcnt") and wait:
                queued = min(queued, int(wait.group(1)))
            elif queued and found is not None and re.match(r"(buffer_load|global_load)\w* .*\blds\b|global_load_lds", line):
                found.append(line)
        return queued

    begin, todo = [0] * len(blocks), list(range(len(blocks)))
    while todo:
        n = todo.pop()
        queued = run(blocks[n], begin[n])
        for to in follow[n]:
            if queued > begin[to]:
                begin[to] = queued
                todo.append(to)
    found = []
    for block, queued in zip(blocks, begin):
        run(block, queued, found)
    return found


def test_the_order_scan_itself():
    read, load, wait = "ds_read_b128 v[0:3], v4", "buffer_load_dwordx4 v1, s[0:3], s4 offen lds", "s_waitcnt lgkmcnt(0)"
    assert transfers_before_reads_are_done([read, load]) == [load]
    assert transfers_before_reads_are_done([read, wait, load]) == []
    assert transfers_before_reads_are_done([read, read, "s_waitcnt lgkmcnt(1)", load]) == [load]
    # the reads at the end of a loop body, the transfer at its start
    loop = ["a:", load, read, "s_cbranch_scc1 a", "s_endpgm"]
    assert transfers_before_reads_are_done(loop) == [load]
    assert transfers_before_reads_are_done(["a:", wait] + loop[1:]) == []
    # a block behind a jump, entered from one with reads queued and from one without
    assert transfers_before_reads_are_done([read, "s_cbranch_vccz b", wait, "s_branch c", "b:", load, "c:", "s_endpgm"]) == [load]
    assert transfers_before_reads_are_done([read, wait, "s_cbranch_vccz b", read, "s_branch c", "b:", load, "c:", "s_endpgm"]) == []


# Transfers that the scan finds because reads of another area may be queued, the queries', which no transfer overwrites while they are
# read: the keys of the pseudo tokens' own block (8 to a sub-block), and the first tiles of a decode step (16 transfers before the row count is known, 16 after it).
BESIDE_READS_OF_QUERIES = {"score_pseudo_kernelILb0E": 8, "decode_attention_kernel": 32}


def test_ring_slots_are_refilled_after_their_reads(units):
    """A transfer past the end of its source fetches nothing, and its zeros are in LDS before reads that were issued just before it."""
    for src in ("qproj.hip", "score.hip", "decode.hip"):
        bodies = units[src][0]
        assert any(re.match(r"buffer_load.* lds|global_load_lds", line) for body in bodies.values() for line in body), src
        for name, body in bodies.items():
            known = sum(n for kernel, n in BESIDE_READS_OF_QUERIES.items() if kernel in name)
            early = transfers_before_reads_are_done(body)
            assert len(early) <= known, (name, early[:2])
