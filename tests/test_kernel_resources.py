"""What the compiler made of the GEMM kernel: all 256 accumulator registers of a wavefront in the AGPR half of
its register file, one wavefront per SIMD, and nothing spilled to scratch memory in any instantiation (a spill
inside the K loop costs far more than the few registers it saves; outside it, it still means the loop's
register budget was exceeded somewhere); and what it made of the few-rows GEMM, whose waits count loads.  Compiles the device
code; no GPU needed."""
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


def test_table_scorer_keeps_three_wavefronts_per_simd_without_spilling():
    """The look-up scorer is planned as one resident round of workgroups, three per CU: every instantiation has to
    fit three wavefronts per SIMD with its per-subset look-up addresses in registers, not in scratch memory."""
    usage = build.kernel_resource_usage("enumerate.hip")
    luts = {n: u for n, u in usage.items() if "score_lut_kernel" in n}
    assert len(luts) >= 7
    for name, u in luts.items():
        assert u["ScratchSize"] == 0 and u["VGPRs Spill"] == 0, (name, u)
        assert u["Occupancy"] >= 3, (name, u)


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
