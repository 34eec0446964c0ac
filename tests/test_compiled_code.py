"""Properties of the compiled kernels that a run does not show, or shows only as time: read from the assembly that the
package's own compiler flags give."""
import functools
import os
import re
import subprocess

import pytest

from paper_2605_16360_amd import build


@functools.lru_cache(maxsize=None)
def kernels(source):
    """(name, assembly) of every kernel of a source file"""
    r = subprocess.run([build._hipcc(), *build.FLAGS, "-x", "hip", "--cuda-device-only", "-S", os.path.join(build.CSRC, source),
                        "-o", "-"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return re.findall(r"^(_ZN\w*):(.*?)^\.Lfunc_end", r.stdout, re.M | re.S)


def test_every_topk_pass_waits_for_its_adds_before_the_ticket():
    """The split Top-K's workgroups meet in a per-row histogram: each adds its bins, then takes a ticket, and the last to arrive
    reads the histogram.  Nothing but a wait for outstanding memory operations orders a wave's adds before the ticket, so
    `s_waitcnt vmcnt(0)` has to stand between the last add without a result and the barrier in front of the ticket."""
    passes = [(name, body) for name, body in kernels("topk.hip") if "mw_pass_kernel" in name]
    assert len(passes) == 7  # three of 11 bits, four of 8
    for name, body in passes:
        ops = re.findall(r"^\s+(global_atomic_add\b.*|s_barrier\b|s_waitcnt\b.*)$", body, re.M)
        adds = [i for i, op in enumerate(ops) if op.startswith("global_atomic_add")]
        bins = [i for i in adds if "sc0" not in ops[i]]  # sc0: the old value is returned
        ticket = next(i for i in adds if i > bins[-1])
        barriers = [i for i in range(bins[-1], ticket) if ops[i].startswith("s_barrier")]
        assert barriers, name
        assert any("vmcnt(0)" in op for op in ops[bins[-1]:barriers[-1]]), name


@pytest.mark.parametrize("source", ["score_lse.hip", "score_colmax.hip"])
def test_no_scoring_tile_waits_for_its_own_prefetch(source):
    """The resident operand is loaded once, in front of the loop.  Where the compiler cannot tell that it has landed, it puts a
    wait for global loads in front of the loop's MFMAs, and every tile then waits for the prefetch it has just issued."""
    seen = 0
    for name, body in kernels(source):
        ops = re.findall(r"^\s+(s_waitcnt\b.*|v_mfma\w*|s_barrier|v_\w+|ds_\w+|global_\w+)", body, re.M)
        if not any(op.startswith("v_mfma") for op in ops):
            continue
        seen += 1
        first = next(i for i, op in enumerate(ops) if op.startswith("s_barrier"))
        waiting = [i for i in range(first, len(ops)) if ops[i].startswith("v_mfma") and "vmcnt" in ops[i - 1]]
        assert not waiting, f"{name}: {len(waiting)} MFMAs behind a wait for global loads"
    assert seen >= 4


@pytest.mark.parametrize("source", ["score_lse_fp32.hip", "score_lse_piped.hip"])
def test_no_other_pass_1_tile_waits_for_its_own_prefetch(source):
    """The same for pass 1's kernel on fp32 inputs and for the piped one, which spills nothing either."""
    (name, body), = [(name, body) for name, body in kernels(source) if "score_lse_kernel" in name]
    ops = re.findall(r"^\s+(s_waitcnt\b.*|v_mfma\w*|s_barrier|v_\w+|ds_\w+|global_\w+)", body, re.M)
    first = next(i for i, op in enumerate(ops) if op.startswith("s_barrier"))
    assert not [i for i in range(first, len(ops)) if ops[i].startswith("v_mfma") and "vmcnt" in ops[i - 1]], name
    assert "scratch_" not in body


def test_scoring_masks_do_not_branch_per_element():
    """A column sees one range of keys, so the mask of a cut tile is a comparison per element.  Written as a choice per element
    it compiles to hundreds of branches, fetched for the few cut tiles of a short input."""
    passes = [(name, body) for name, body in kernels("score_lse.hip") if "score_lse_kernel" in name]
    assert len(passes) == 4
    for name, body in passes:
        assert len(re.findall(r"^\s+s_cbranch", body, re.M)) < 128, name


def test_in_place_compaction_keeps_its_loads_in_flight():
    """A thread asks for all pieces of a chunk back to back, behind indices that it asked for a chunk earlier.  With an index and a
    branch in front of every piece the compiler waits for all loads before each of them."""
    moves = [(name, body) for name, body in kernels("compact.hip") if "compact_inplace_kernel" in name]
    assert len(moves) == 5
    for name, body in moves:
        ops = re.findall(r"^\s+(s_barrier|s_waitcnt\b.*|global_load_dwordx4)", body, re.M)
        loop = ops[next(i for i, op in enumerate(ops) if op.startswith("s_barrier")):]
        loads = [i for i, op in enumerate(loop) if op.startswith("global_load_dwordx4")]
        assert loads and not any("vmcnt(0)" in loop[i - 1] for i in loads), name


def test_in_place_compaction_holds_a_chunk_before_it_stores_one():
    """A token's new place may be another's old one, so a thread's loads of a chunk have to be over before any thread of the workgroup
    stores that chunk.  The barrier between does not wait for loads: a wait that leaves at most the next chunk's loads and
    the indices behind them stands in front of it, and none of the stored registers is waited for behind it."""
    for name, body in kernels("compact.hip"):
        if "compact_inplace_kernel" not in name:
            continue
        per = int(re.search(r"compact_inplace_kernelILi(\d+)E", name)[1])
        ops = re.findall(r"^\s+(s_barrier|s_waitcnt\b.*|global_\w+)", body, re.M)
        for i in [i for i, op in enumerate(ops) if op.startswith("s_barrier")]:
            waits = []
            for op in ops[i - 1::-1]:
                if op.startswith("global_load") or op.startswith("s_barrier"):
                    break
                waits += [int(n) for n in re.findall(r"vmcnt\((\d+)\)", op)]
            assert waits and min(waits) <= 2 * per, (name, ops[max(0, i - 8):i + 1])
            behind = ops[i + 1:i + 2 + 2 * per]
            stores = [j for j, op in enumerate(behind) if op.startswith("global_store")]
            assert not stores or not any("vmcnt" in op for op in behind[:stores[0]]), (name, behind)


def _compaction_in_parts():
    (body,) = [body for name, body in kernels("compact.hip") if "compact_parts_kernel" in name]
    return body


def test_compaction_in_parts_never_gives_up_its_wait():
    """A part that stores before the parts in front of it in its row have been loaded destroys what they still have to move.  Those have started and wait for
    earlier ones only, so the wait ends; one bounded by a clock, which goes on while the queue is off the chip, might end too early."""
    body = _compaction_in_parts()
    assert "s_memrealtime" not in body and "s_memtime" not in body and "s_getreg" not in body
    waits = [loop for loop in loops(body) if "s_sleep" in loop and "global_load_dword " in loop]
    assert waits and all(len(re.findall(r"^\s+s_sleep", loop, re.M)) == 1 for loop in waits)


def test_compaction_in_parts_holds_its_part_before_it_says_so():
    """A part's flag lets the parts behind it store where it loads from, so all loads of its pieces, of every wave, have to be over before the flag is
    stored: a wait for all of them, then a barrier, which by itself waits for no load, then the flag; and no piece is stored in front of the barrier
    behind the wait for the parts in front."""
    ops = re.findall(r"^\s+(s_barrier|s_waitcnt\b.*|s_sleep|global_\w+)", _compaction_in_parts(), re.M)
    loads = [i for i, op in enumerate(ops) if op == "global_load_dwordx4"]
    stores = [i for i, op in enumerate(ops) if op == "global_store_dwordx4"]
    (flag,) = [i for i, op in enumerate(ops) if op == "global_store_dword"]
    wait = [i for i, op in enumerate(ops) if op == "s_sleep"][-1]
    assert len(loads) == len(stores) == 20
    barrier = next(i for i in range(loads[-1], len(ops)) if ops[i] == "s_barrier")
    assert any("vmcnt(0)" in op for op in ops[loads[-1]:barrier]) and barrier < flag
    assert flag < wait and "s_barrier" in ops[wait:stores[0]] and stores[0] > wait


def _registers(text):
    """{("v", 3), ("v", 4), ...} named in an operand list"""
    out = set()
    for kind, one, lo, hi in re.findall(r"\b([av])(?:(\d+)\b|\[(\d+):(\d+)\])", text):
        out |= {(kind, int(one))} if one else {(kind, i) for i in range(int(lo), int(hi) + 1)}
    return out


def test_written_out_matrix_instructions_keep_their_distances():
    """The compiler does not look into inline assembly for hazards: no operand of such a matrix instruction may come from a vector
    instruction less than two wait states before it, and nothing but a matrix instruction may touch its result less than 19 behind."""
    seen = 0
    for name, body in kernels("mapper_block.hip"):
        if "encoder_block_kernel" not in name:
            continue
        lines = [l.strip() for l in body.splitlines()]
        ops, inside = [], False
        for l in lines:
            inside = l.startswith(";;#ASMSTART") or (inside and not l.startswith(";;#ASMEND"))
            if re.match(r"[vsdgb][a-z]*_", l):
                ops.append((l, inside))
        for i, (op, written_out) in enumerate(ops):
            if not (written_out and op.startswith("v_mfma")):
                continue
            seen += 1
            dst, src = op.split(None, 1)[1].split(",", 1)
            dst, src, states = _registers(dst), _registers(src), 0
            for before, _ in reversed(ops[max(0, i - 2):i]):
                states += 1 + (int(before.split()[1]) if before.startswith("s_nop") else 0)
                if before.startswith("v_") and not before.startswith("v_mfma") and states <= 2:
                    assert not _registers(before.split(None, 1)[1].split(",", 1)[0]) & src, (name, before, op)
            states = 0
            for behind, _ in ops[i + 1:i + 20]:
                if states >= 19 or behind.startswith("s_cbranch"):
                    break
                assert behind.startswith("v_mfma") or not _registers(behind) & dst, (name, op, behind)
                # a matrix instruction behind it holds the next one back for four passes
                states += 1 + (int(behind.split()[1]) if behind.startswith("s_nop") else 3 if behind.startswith("v_mfma") else 0)
    assert seen >= 500


def loops(body):
    """The text of every loop: from a label to a branch back to it, conditional or not."""
    labels, out = {}, []
    for m in re.finditer(r"^(\.LBB\w+):|^\s+s_c?branch\w* (\.LBB\w+)", body, re.M):
        if m[1]:
            labels[m[1]] = m.end()
        elif m[2] in labels:
            out.append(body[labels[m[2]]:m.start()])
    return out


def test_encoder_block_keeps_its_registers():
    """256 accumulators and 128 more for the hidden features leave little: nothing may be spilled inside the loops over K and over chunks of
    the hidden features.  (A block of the last launch spills 20 registers once, around its first LayerNorm.)"""
    blocks = [(name, body) for name, body in kernels("mapper_block.hip") if "encoder_block_kernel" in name]
    assert len(blocks) == 6  # whole and half blocks: first, middle and last launch
    for name, body in blocks:
        tiles, first, last = re.search(r"kernelILi(\d)ELb(\d)ELb(\d)E", name).groups()
        found = [(loop.count("v_mfma"), "scratch_" in loop) for loop in loops(body)]
        found = [(mfmas, spills) for mfmas, spills in found if mfmas]
        # one per product with the token tile (out-projection; q, k, v), the first FFN product's and the chunks' around it
        assert len(found) == (1 + 2) * (first == "0") + 3 * (last == "0"), (name, found)
        # a chunk: biases, the first product's last steps in line, all of the second product
        assert max(mfmas for mfmas, _ in found) >= (int(tiles) * 80 if first == "0" else int(tiles) * 16), (name, found)
        assert not any(spills for _, spills in found), (name, found)


def test_small_mapper_loads_a_row_once():
    """The products that normalise their 64 rows first load each once, whatever follows them: with a scale, a shift and the weights a lane
    asks for 40 times 16 bytes.  (A layer with a second window, whose rows would be averaged, has too many rows for these kernels.)"""
    wide = [(name, body) for name, body in kernels("mapper_small.hip") if "small_wide_kernel" in name]
    loads = {name: len(re.findall(r"^\s+global_load_dwordx4", body[:body.index("v_mfma")], re.M)) for name, body in wide}
    assert sorted(loads.values()) == [0, 40, 40, 40], loads  # (the first product's operands go to LDS directly)
