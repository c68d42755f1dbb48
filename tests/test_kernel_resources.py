"""What the compiler made of the GEMM kernel: all 256 accumulator registers of a wavefront in the AGPR half of
its register file, one wavefront per SIMD, and nothing spilled to scratch memory in any instantiation (a spill
inside the K loop costs far more than the few registers it saves; outside it, it still means the loop's
register budget was exceeded somewhere); the order of the loads that the hand-counted waits of this kernel, of the few-rows
GEMM and of the fp32 GEMM rely on; and the registers of the table scorers, whose launches are planned by residency.  Compiles the device code; no
GPU needed."""
import re

import pytest

from paper_2402_14800_amd import build


@pytest.fixture(scope="module")
def gemm_usage():
    return build.kernel_resource_usage("gemm_bf16_packed.hip")


def test_packed_gemm_instantiations_do_not_spill(gemm_usage):
    gemms = {n: u for n, u in gemm_usage.items() if "gemm_packed_kernel" in n}
    assert len(gemms) >= 5                       # dense store / SwiGLU, grouped store / SwiGLU / row-scaled fp32
    for name, u in gemms.items():
        assert u["ScratchSize"] == 0, (name, u)
        assert u["VGPRs Spill"] == 0 and u["SGPRs Spill"] == 0, (name, u)
        assert u["AGPRs"] == 256 and u["VGPRs"] <= 256, (name, u)
        assert u["Occupancy"] == 1, (name, u)


def test_pack_kernel_is_light(gemm_usage):
    pack = [u for n, u in gemm_usage.items() if "pack_kernel" in n]
    assert pack and all(u["ScratchSize"] == 0 for u in pack)


@pytest.fixture(scope="module")
def enumerate_usage():
    return build.kernel_resource_usage("enumerate.hip")


def test_table_scorer_keeps_three_wavefronts_per_simd_without_spilling(enumerate_usage):
    """The look-up scorer of more than 16 experts is planned as one resident round of workgroups, three per CU: every
    instantiation has to fit three wavefronts per SIMD with its per-subset look-up addresses in registers, not in scratch memory."""
    luts = {n: u for n, u in enumerate_usage.items() if re.search(r"\d+score_lut_kernel", n)}
    assert len(luts) == 4                        # 5 to 8 nibbles of the kept mask
    for name, u in luts.items():
        assert u["ScratchSize"] == 0 and u["VGPRs Spill"] == 0, (name, u)
        assert u["Occupancy"] >= 3, (name, u)


def test_fused_table_scorer_keeps_eight_wavefronts_per_simd_without_spilling(enumerate_usage):
    """The scorer with tables in LDS is planned as two workgroups of 1024 threads or four of 512 per CU: eight wavefronts per
    SIMD, hence at most 64 vector registers, and none in scratch memory."""
    fused = {n: u for n, u in enumerate_usage.items() if "fused_score_lut_kernel" in n}
    assert len(fused) == 7                       # records of 4 to 12 ranks, 4 or 14 subsets per lane (4 ranks: 4)
    for name, u in fused.items():
        assert u["ScratchSize"] == 0 and u["VGPRs Spill"] == 0, (name, u)
        assert u["Occupancy"] == 8, (name, u)


def k_loops(kernel):
    """The single-block loops of a kernel's lines that multiply on the matrix units, each as its number of MFMAs and its
    vector-memory operations, waits for them and barriers in order; a load as the register of its lane offset."""
    label = at = None
    for i, line in enumerate(kernel):
        if m := re.match(r"(\.LBB\d+_\d+):", line):
            label, at = m.group(1), i
        elif (m := re.match(r"\s+s_cbranch\S*\s+(\.LBB\d+_\d+)", line)) and m.group(1) == label:
            ops = []
            for word in (w for w in map(str.split, kernel[at:i]) if w):
                if word[0].startswith(("global_", "buffer_", "flat_", "scratch_")):
                    assert "lds" in word[-1] or "_lds_" in word[0], word                 # nothing but loads into the ring
                    ops.append(word[1].rstrip(","))
                elif word[0] == "s_barrier":
                    ops.append(word[0])
                elif word[0] == "s_waitcnt" and (m := re.search(r"vmcnt\((\d+)\)", " ".join(word))):
                    ops.append(int(m.group(1)))
            mfmas = sum("v_mfma_f32_16x16x32_bf16" in x for x in kernel[at:i])
            if mfmas:
                yield mfmas, ops


def test_packed_gemm_waits_for_the_loads_it_means():
    """A wavefront of the 256-row GEMM waits until all but its newest N loads have landed.  Blocked weights: N loads are a step's,
    every second step.  Row-major weights: in front of an odd step the newest step's and the A loads of the one before, which is
    right only if every step issues its weight loads BEFORE its A loads; a load merged, dropped or moved by the compiler would be
    a silent race.  Checked in all six bodies (tile widths and heights) of every instantiation."""
    text = build.device_assembly("gemm_bf16_packed.hip").splitlines()
    starts = [i for i, line in enumerate(text) if re.match(r"_ZN\S*gemm_packed_kernel\S*:", line)]
    assert len(starts) == 10                     # 3 epilogues, dense (2 of them) or grouped, 2 weight layouts
    for start in starts:
        row_major = re.search(r"kernelILi\d+ELb[01]ELb([01])E", text[start]).group(1) == "1"
        bodies = set()
        for mfmas, ops in k_loops(text[start:next(i for i in range(start, len(text)) if ".Lfunc_end" in text[i])]):
            at = [i for i, o in enumerate(ops) if o == "s_barrier"]
            steps = [ops[b:e] for b, e in zip([0] + [i + 1 for i in at], at)]
            assert ops[-1] == "s_barrier" and len(steps) == (2 if row_major else 1), (text[start], ops)
            assert all(isinstance(s[-1], int) and not any(isinstance(o, int) for o in s[:-1]) for s in steps), (text[start], ops)
            loads, waits = [s[:-1] for s in steps], [s[-1] for s in steps]
            if row_major:                        # weights by two lane offsets in turn, then the rows of A by a third
                w = max(i for i, o in enumerate(loads[0]) if o != loads[0][-1]) + 1
                a = len(loads[0]) - w
                for step in loads:
                    assert len(step) == w + a and w % 2 == 0, (text[start], ops)
                    assert len(set(step[0:w:2])) == len(set(step[1:w:2])) == len(set(step[w:])) == 1, (text[start], ops)
                    assert len({step[0], step[1], step[w]}) == 3, (text[start], ops)
                assert waits == [w + 2 * a, 2 * (w + a)], (text[start], ops)
                assert mfmas == 2 * (2 * w) * (2 * a), (text[start], mfmas)
                bodies.add((2 * w, 2 * a))
            else:
                assert len(loads[0]) == 2 * waits[0], (text[start], ops)
                bodies.add((mfmas, waits[0]))
        tiles = [(ng, mg) for ng in (4, 8) for mg in (4, 6, 8)]
        assert bodies == ({*tiles} if row_major else {(2 * ng * mg, (ng + mg) // 2) for ng, mg in tiles}), (text[start], bodies)


def few_rows_body(text, header):
    """The inner loop that starts at line `header` of a kernel's lines, as a list of its vector-memory loads and hand-written
    waits, and the line after it."""
    label = re.match(r"(\.LBB\d+_\d+):", text[header]).group(1)
    end = next(i for i in range(header + 1, len(text)) if re.match(r"\s+s_c?branch\S*\s+" + re.escape(label) + r"\b", text[i]))
    return loads_and_waits(text[header:end]), end + 1


def loads_and_waits(lines):
    ops = []
    for i, line in enumerate(lines):
        op = line.split()[0] if line.split() else ""
        if op.startswith("global_load_lds_dwordx4"):
            ops.append("weights")
        elif op == "global_load_dwordx4":
            ops.append("rows")
        elif op.startswith(("global_load", "flat_", "buffer_", "scratch_", "global_store", "global_atomic")):
            ops.append(op)
        elif op == "s_waitcnt" and "sched_barrier" in lines[i - 1]:
            ops.append(int(re.search(r"vmcnt\((\d+)\)", line).group(1)))
    return ops


def test_few_rows_gemm_waits_for_the_loads_it_means():
    """A wavefront of gemm_few_kernel waits until all but the newest N loads have landed.  That is right only if every pair of
    slices is exactly 2 NF loads of weights and 2 M of rows, all issued before the wait: a load merged, dropped or moved by the
    compiler would be a silent race.  Counted here in every body of every instantiation."""
    text = build.device_assembly("gemm_few.hip").splitlines()
    starts = [i for i, line in enumerate(text) if re.match(r"_ZN\S*gemm_few_kernel\S*:", line)]
    assert len(starts) == 36                     # 3 epilogues, 2 weight layouts, 3 sizes of the row group, 2 rings
    for start in starts:
        epi, mmax, ring = map(int, re.search(r"kernelILi(\d+)ELb[01]ELi(\d+)ELi(\d+)E", text[start]).groups())
        kernel = text[start:next(i for i in range(start, len(text)) if ".Lfunc_end" in text[i])]
        weights, ahead, bodies, at = (8 if epi == 1 else 4), ring > 16384, [], 0
        while True:
            header = next((i for i in range(at, len(kernel)) if "Inner Loop Header" in kernel[i]), None)
            if header is None:
                break
            before = loads_and_waits(kernel[at:header])
            loop, at = few_rows_body(kernel, header)
            waits = [o for o in loop if isinstance(o, int)]
            rows = loop.count("rows") // len(waits)
            per_pair, depth = weights + rows, len(waits)
            flying = (depth - 2 if ahead else depth - 1) * per_pair
            assert depth >= 2 and set(waits) == {flying} and flying < 64, (text[start], waits)
            steps = " ".join(map(str, loop)).split(f" {flying}")
            assert all(sorted(s.split()) == ["rows"] * rows + ["weights"] * weights for s in steps[:depth]) and not steps[depth].strip()
            # in front of the loop: all pairs of the ring but one
            assert before.count("weights") == (depth - 1) * weights and before.count("rows") == (depth - 1) * rows, text[start]
            last_load = max(i for i, o in enumerate(before) if o in ("weights", "rows"))
            assert [o for o in before[last_load + 1:] if isinstance(o, int)] == ([flying] if ahead else []), (text[start], before)
            bodies.append(rows // 2)
        assert sorted(bodies) == sorted(2 * [m for m in (1, 2, 4) if m <= mmax]), (text[start], bodies)


def test_few_rows_gemm_does_not_spill():
    usage = {n: u for n, u in build.kernel_resource_usage("gemm_few.hip").items() if "gemm_few_kernel" in n}
    assert len(usage) == 36
    for name, u in usage.items():
        assert u["ScratchSize"] == 0 and u["VGPRs Spill"] == 0 and u["SGPRs Spill"] == 0, (name, u)
        assert u["Occupancy"] >= (1 if "Li40960E" in name else 2), (name, u)      # as many wavefronts as the rings leave room for


def test_fp32_gemm_waits_for_the_loads_it_means():
    """A wavefront of gemm_f32_kernel waits until all but the loads of the newest AHEAD - 1 slabs have landed.  That is right only if
    a slab is exactly (TM + TB) / 32 loads into the ring, AHEAD slabs of them in front of the loop and one in every step of it, after
    the barrier, and nothing else of that kind: a load merged, dropped or moved by the compiler would be a silent race.  Past the
    loop everything has landed before the ring is used again."""
    text = build.device_assembly("gemm_f32.hip").splitlines()
    starts = [i for i, line in enumerate(text) if re.match(r"_ZN\S*gemm_f32_kernel\S*:", line)]
    assert len(starts) == 15                     # 3 epilogues; 64 x 128 and 32 x 128 with one and two slabs ahead, 32 x 64 with two
    for start in starts:
        tm, tb, ahead = map(int, re.search(r"kernelILi\d+ELi(\d+)ELi(\d+)ELi(\d+)E", text[start]).groups())
        kernel = text[start:next(i for i in range(start, len(text)) if ".Lfunc_end" in text[i])]
        loads = (tm + tb) // 32
        header = next(i for i, line in enumerate(kernel) if "Inner Loop Header" in line)
        label = re.match(r"(\.LBB\d+_\d+):", kernel[header]).group(1)
        end = next(i for i in range(header + 1, len(kernel)) if re.match(r"\s+s_c?branch\S*\s+" + re.escape(label) + r"\b", kernel[i]))

        def ops(lines):
            found = []
            for line in lines:
                op = line.split()[0] if line.split() else ""
                if op.startswith(("global_", "flat_", "buffer_", "scratch_")):
                    found.append("ring" if op == "global_load_lds_dwordx4" else op)
                elif op == "s_barrier":
                    found.append(op)
                elif op == "s_waitcnt" and (m := re.search(r"vmcnt\((\d+)\)", line)):
                    found.append(int(m.group(1)))
            return found

        before, loop, after = ops(kernel[:header]), ops(kernel[header:end]), ops(kernel[end:])
        assert loop == [(ahead - 1) * loads, "s_barrier"] + loads * ["ring"], (text[start], loop)
        assert before[-ahead * loads:] == ahead * loads * ["ring"] and before.count("ring") == ahead * loads, (text[start], before)
        assert after[:2] == [0, "s_barrier"] and "ring" not in after, (text[start], after)
        assert sum("v_mfma_f32_16x16x4_f32" in line for line in kernel[header:end]) == 8 * (tm // 32) * (tb // 32), text[start]


def test_fp32_gemm_does_not_spill():
    usage = {n: u for n, u in build.kernel_resource_usage("gemm_f32.hip").items() if "gemm_f32_kernel" in n}
    assert len(usage) == 15
    for name, u in usage.items():
        tm, tb, ahead = map(int, re.search(r"kernelILi\d+ELi(\d+)ELi(\d+)ELi(\d+)E", name).groups())
        assert u["ScratchSize"] == 0 and u["VGPRs Spill"] == 0 and u["SGPRs Spill"] == 0, (name, u)
        # the workgroups per compute unit that f32_slabs_ahead counts on
        assert u["Occupancy"] >= {(64, 2): 2, (64, 1): 3, (32, 2): 2 if tb == 128 else 4, (32, 1): 4}[tm, ahead], (name, u)
