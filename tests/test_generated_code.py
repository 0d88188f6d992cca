"""Checks on the machine code hipcc generates for the tree-attention sweep (no GPU needed: the kernels are only
compiled).  Two properties that correctness or speed depend on and that a compiler update could silently break:
  - the LDS address register M0 is written by the kernel's own assembly (direct-to-LDS loads) and the compiler was
    not told; so no compiler-generated instruction may use M0;
  - in the steady-state loop of every sweep instantiation the only waits on the vector-memory counter are the
    kernel's own, one per tile, next to its barrier: an additional compiler-placed wait would make the LDS reads of
    the tile being computed wait for the loads of the next tile (bf16 prefix: two-tile loop of a double buffer; fp8
    prefix and small bf16 launches: four-tile loop of a four-stage ring)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2409_10644_amd.build import COMMON, CSRC, SOURCES

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def sweep_asm(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("hipcc not available")
    out = tmp_path_factory.mktemp("asm") / "tree_attention.s"
    # with the flags of the build itself: what they do to the kernels (arguments preloaded into registers, say) is in what ships
    cmd = [HIPCC, *COMMON, *SOURCES["tree_attention.hip"], "-S", "--cuda-device-only", "-o", str(out),
           os.path.join(CSRC, "tree_attention.hip")]
    subprocess.run(cmd, check=True, capture_output=True)
    return out.read_text().split("\n")


def _functions(lines):
    starts = [(i, l.split(":")[0]) for i, l in enumerate(lines) if re.match(r"^_Z\w+:", l)]
    for (i0, name), (i1, _) in zip(starts, starts[1:] + [(len(lines), "")]):
        yield name, lines[i0:i1]


def test_m0_is_only_touched_by_the_kernels_own_assembly(sweep_asm):
    inside, seen = False, 0
    for l in sweep_asm:
        if "#ASMSTART" in l:
            inside = True
        elif "#ASMEND" in l:
            inside = False
        elif re.search(r"\bm0\b", l.split(";")[0]):
            assert inside, f"compiler-generated use of M0: {l.strip()}"
            seen += 1
    assert seen > 0


def test_steady_state_loops_wait_for_memory_once_per_tile(sweep_asm):
    checked = 0
    for name, body in _functions(sweep_asm):
        if "tree_attn_bf16_kernel" not in name and "tree_attn_bf16_short_kernel" not in name:
            continue
        labels = {m.group(1): i for i, l in enumerate(body) if (m := re.match(r"^(\.LBB\d+_\d+):", l))}
        loops = []
        for i, l in enumerate(body):
            m = re.search(r"s_c?branch\w*\s+(\.LBB\d+_\d+)", l)
            if m and m.group(1) in labels and labels[m.group(1)] < i:
                loop = body[labels[m.group(1)]:i + 1]
                if any("global_load_lds" in x for x in loop) and any("v_mfma" in x for x in loop):
                    loops.append(loop)
        assert loops, f"no streaming loop found in {name}"
        D, QBP, NS, F8 = (int(x) for x in re.search(r"ILi(\d+)ELi(\d+)ELi(\d+)ELb(\d)E", name).groups())
        if NS == 2:
            # the loop of two full tiles: all it requests are full tiles (a tile that is not takes an address per lane, "off"), two
            # of them non-temporally, and block placement may put backward jumps inside it: the innermost that spans all of it
            alone = D == 128 and QBP == 1 and "short" not in name          # (has the compute unit to itself: waits for halves)
            keys = {1: 128, 2: 64, 4: 64}[QBP]
            loads_per_half = keys * D * 2 // 1024 // 4
            code = [[y.split(";")[0] for y in x] for x in loops]
            full = [x for x in code if sum(bool(re.search(r"global_load_lds.*\bnt\b", y)) for y in x) == 4 * loads_per_half
                    and not any(re.search(r"global_load_lds\S* v\[\d+:\d+\], off", y) for y in x) and sum("s_barrier" in y for y in x) == (4 if alone else 2)]
            assert full, f"{name}: no loop of two full tiles found"
            code = min(full, key=len)
            waits = [int(x) for y in code for x in re.findall(r"vmcnt\((\d+)\)", y)]
            assert waits == ([2 * loads_per_half] * 4 if alone else [0, 0]), f"{name}: {waits}"
        else:
            # four-stage ring, four tiles per trip; a step waits for all loads but those of the two, one or zero tiles
            # requested after its own (three alternative instructions), right before its barrier, and nowhere else
            # (of the backward branches that span exactly the ring's four barriers the one with the fewest waits, the
            # longest of those: block placement adds backward jumps from the kernel's epilogue whose spans hold the
            # loop plus the waits before and after it; a wait the compiler added inside the loop is in every span)
            four = [x for x in loops if sum("s_barrier" in y.split(";")[0] for y in x) == 4]
            assert four, f"{name}: no four-tile loop found"
            loop = min(four, key=lambda x: (sum("vmcnt" in y.split(";")[0] for y in x), -len(x)))
            code = [x.split(";")[0] for x in loop if x.split(";")[0].strip() and not x.strip().startswith(".")]
            wait_at = [i for i, x in enumerate(code) if "vmcnt" in x]
            barrier_at = [i for i, x in enumerate(code) if "s_barrier" in x]
            assert len(barrier_at) == 4 and len(wait_at) == 12, f"{name}: {len(wait_at)} waits, {len(barrier_at)} barriers"
            for i in wait_at:
                assert any(0 < b - i <= 16 for b in barrier_at), f"{name}: a wait on vector memory away from the barriers"
            row_bytes = D if F8 else 2 * D                     # 64-key tiles: 2 (K, V) x 64 rows / rows per 1 KiB load / 4 wavefronts
            loads_per_tile = 2 * 64 * row_bytes // 1024 // 4
            assert sorted(set(int(re.search(r"vmcnt\((\d+)\)", code[i]).group(1)) for i in wait_at)) == \
                [0, loads_per_tile, 2 * loads_per_tile], name
        assert not any("scratch_" in x for x in code), f"{name}: register spills inside the streaming loop"
        checked += 1
    # head_dim 64 / 128 x 1, 2, 4 query blocks with two stages, x 2, 4 query blocks with four; fp8 prefix: head_dim 128 x 2, 4;
    # and those of two stages and of the fp8 prefix once more, with fp32 partial results (short prefixes)
    assert checked == 12 + 8


def test_the_loop_of_a_workgroup_alone_waits_for_halves(sweep_asm):
    """Grids of pairs: the loop of two tiles with two waits and barriers each leaves exactly two half tiles' loads under way."""
    checked = 0
    for name, body in _functions(sweep_asm):
        if "tree_attn_bf16_ragged_kernel" not in name:
            continue
        D, QBP = (int(x) for x in re.search(r"ILi(\d+)ELi(\d+)ELi2ELb0E", name).groups())
        labels = {m.group(1): i for i, l in enumerate(body) if (m := re.match(r"^(\.LBB\d+_\d+):", l))}
        spans = [body[labels[m.group(1)]:i + 1] for i, l in enumerate(body)
                 if (m := re.search(r"s_c?branch\w*\s+(\.LBB\d+_\d+)", l)) and labels.get(m.group(1), i) < i]
        four = [x for x in spans if sum("s_barrier" in y.split(";")[0] for y in x) == 4 and any(re.search(r"global_load_lds.*\bnt\b", y) for y in x)]
        assert four, f"{name}: no such loop found"
        code = [x.split(";")[0] for x in min(four, key=len)]
        keys = {1: 128, 2: 64}[QBP]
        loads_per_half = keys * D * 2 // 1024 // 4
        assert [int(x) for y in code for x in re.findall(r"vmcnt\((\d+)\)", y)] == [2 * loads_per_half] * 4, name
        assert not any("scratch_" in x for x in code), name
        checked += 1
    assert checked == 3                                         # 64 columns x 1, 2 query blocks, 128 x 2


def test_masked_scores_cost_two_instructions(sweep_asm):
    """A bit spread over a register and a blend per score; comparing and selecting takes twice as many."""
    checked = 0
    for name, body in _functions(sweep_asm):
        if "tree_attn_bf16_" not in name or "merge" in name:
            continue
        QBP = int(re.search(r"ILi\d+ELi(\d+)E", name).group(1))
        code = [x.split(";")[0] for x in body]
        spread = [x for x in code if re.search(r"v_bfe_i32 v\d+, v\d+, \d+, 1\s*$", x)]
        assert spread and len(spread) % (16 * (2 if QBP == 4 else 1)) == 0, f"{name}: {len(spread)}"
        assert not any(re.search(r"v_and_b32\w* v\d+, 0x(100|200|400|800|10000|20000|40000|80000), v", x) for x in code), name
        assert not any("scratch_" in x for x in code), f"{name}: spills"
        checked += 1
    assert checked == 12 + 8 + 3


def test_hidden_networks_read_a_batch_while_the_one_before_is_multiplied(tmp_path):
    """Matrix instructions stand between the reads of a batch's weights from LDS and the wait for them."""
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("hipcc not available")
    out = tmp_path / "decision.s"
    subprocess.run([HIPCC, *COMMON, *SOURCES["decision.hip"], "-S", "--cuda-device-only", "-o", str(out), os.path.join(CSRC, "decision.hip")],
                   check=True, capture_output=True)
    kinds = {"ds_read_b128": "r", "v_mfma_f32_4x4x1": "m", "lgkmcnt(0)": "w"}
    checked = 0
    for name, body in _functions(out.read_text().split("\n")):
        if "decision_hidden_kernel" not in name:
            continue
        labels = {m.group(1): i for i, l in enumerate(body) if (m := re.match(r"^(\.LBB\d+_\d+):", l))}
        spans = [[x.split(";")[0] for x in body[labels[m.group(1)]:i + 1]] for i, l in enumerate(body)
                 if (m := re.search(r"s_c?branch\w*\s+(\.LBB\d+_\d+)", l)) and labels.get(m.group(1), i) < i]
        loops = [x for x in spans if sum("v_mfma" in y for y in x) == 32]                # two batches per trip
        assert loops, f"{name}: no loop of two batches"
        for loop in loops:
            events = "".join(v for x in loop for k, v in kinds.items() if k in x)
            assert events.count("r") == 8 and "rw" not in events, f"{name}: {events}"
            checked += 1
    assert checked >= 2


def test_the_checked_code_takes_its_leading_arguments_in_registers(sweep_asm):
    """The compile above is the shipped one: its kernels say how many argument registers are preloaded."""
    preloaded = [int(m.group(1)) for l in sweep_asm if (m := re.match(r"\s*\.amdhsa_user_sgpr_kernarg_preload_length\s+(\d+)", l))]
    assert preloaded and max(preloaded) > 0
