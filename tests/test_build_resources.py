"""What the compiler made of the kernels (registers, spills, occupancy), read from the remarks the build keeps
in kernel_resources.json.  A change in front of a kernel's loads can silently cost it a wave per SIMD or push it
into scratch memory (a three-line branch once did: 35 registers, 98 spilled, a 2.4 times slower call), so the
kernels that the five workloads launch are pinned here."""
import glob
import json
import os
import re

import pytest

import paper_2605_14844_amd as xfp

PATH = os.path.join(os.path.dirname(xfp.library_path()), "kernel_resources.json")


def resources():
    if not os.path.exists(PATH):
        pytest.skip("kernel_resources.json is written by paper_2605_14844_amd.build.build()")
    with open(PATH) as f:
        return json.load(f)


def find(res, *parts):
    hits = [v for k, v in res.items() if all(p in k for p in parts)]
    assert len(hits) == 1, (parts, len(hits))
    return hits[0]


def test_no_kernel_spills_more_than_a_few_registers():
    res = resources()
    assert len(res) > 500
    worst = max(res.items(), key=lambda kv: kv[1]["vgpr_spills"])
    assert worst[1]["vgpr_spills"] <= 16, worst
    assert sum(1 for v in res.values() if v["vgpr_spills"] > 0) <= 10


@pytest.mark.parametrize("parts,min_waves", [
    (("decode_stream_kernelILi4ELi2ELi1ELb0ELi0ELi2ELi0E",), 4),      # workload 2: 4-bit, K = 4096, two rows per wave
    (("decode_stream_kernelILi4ELi1ELi2ELb0ELi0ELi1ELi0E",), 4),      # workload 1: K = 1024
    (("decode_stream_kernelILi3ELi2ELi1ELb0ELi1ELi2ELi0E",), 4),      # workload 3: V2a 3-bit
    (("decode_stream_kernelILi3ELi2ELi1ELb0ELi2ELi2ELi0E",), 4),      # the same with a scale and a mid-point per group
    (("decode_stream_kernelILi3ELi2ELi1ELb0ELi0ELi4ELi0E",), 4),      # workload 4 gate_up
    (("decode_stream_kernelILi3ELi1ELi2ELb0ELi0ELi4ELi0E",), 4),      # workload 4 down
    (("decode_batch_kernelILi4ELi0ELi8ELi8ELb0ELb0E",), 1),           # workload 5: 8 waves, 8 groups each
    (("decode_tile_kernelILi4ELi16ELb0E",), 4),                       # 8192 x 28672: sixteen waves, one tile per CU
    (("decode_tile_kernelILi4ELi8ELb0E",), 4),                        # large 4-bit matrices: two workgroups per CU
    (("decode_wide_kernelILi4ELi4ELi0E",), 4),                        # 64 tokens in one pass: two workgroups per CU
    (("decode_wide_kernelILi4ELi2ELi0E",), 4),
    (("decode_wide_kernelILi3ELi4ELi0E",), 4),
    (("decode_wide_kernelILi3ELi4ELi1E",), 4),                        # V2a
    (("decode_wide_kernelILi4ELi4ELi1E",), 4),
    (("decode_wide_kernelILi4ELi1ELi2E",), 4),                        # V2a with a scale and a mid-point per group, 16 tokens
    (("decode_wide_kernelILi3ELi1ELi2E",), 4),
    (("decode_gemm_kernelILi4ELi0ENS0_8GemmTileILi1ELi4E",), 2),      # prompts, many tiles: 8 waves, a workgroup per CU
    (("decode_gemm_kernelILi2ELi1ENS0_8GemmTileILi1ELi2ELi4ELi4E",), 4),   # prompts, few tiles, 2 bits: 16 waves
])
def test_the_workloads_kernels_keep_their_registers(parts, min_waves):
    k = find(resources(), *parts)
    assert k["vgpr_spills"] == 0 and k["scratch_bytes_per_lane"] == 0, k
    assert k["waves_per_simd"] >= min_waves, k


def test_the_prompt_kernels_stay_in_registers():
    prompt = {k: v for k, v in resources().items() if "decode_gemm_kernel" in k}
    assert len(prompt) == 32                                          # 2 to 4 bits, V2 and V2a, three tiles, two of them for short rows too; one of 16 waves at 2 bits
    for k, v in prompt.items():
        assert v["vgpr_spills"] == 0 and v["agprs"] == 0 and v["scratch_bytes_per_lane"] == 0, (k, v)


def test_the_tiles_of_tall_matrices_stay_in_registers():
    """The same loop, with the same counted waits, under another name."""
    tiles = {k: v for k, v in resources().items() if "decode_wide_tiles_kernel" in k}
    assert len(tiles) == 6                                            # 2 to 4 bits, V2 and V2a
    for k, v in tiles.items():
        assert v["vgpr_spills"] == 0 and v["agprs"] == 0 and v["scratch_bytes_per_lane"] == 0 and v["waves_per_simd"] >= 3, (k, v)


def test_the_general_kernel_keeps_its_waves_at_5_and_6_bits():
    """A wave there owns a row or two: eight of them per SIMD are what hides a round trip, in 64 registers."""
    rows = {k: v for k, v in resources().items() if re.search(r"decode_rows_kernelILi[56]ELi0E", k)}
    assert len(rows) == 4
    for k, v in rows.items():
        assert v["waves_per_simd"] == 8 and v["vgpr_spills"] == 0 and v["sgpr_spills"] == 0 and v["scratch_bytes_per_lane"] == 0, (k, v)


def test_the_resident_kernels_stay_in_registers():
    """Scratch memory is read through the counter that the kernel's waits for its index words count on."""
    few = {k: v for k, v in resources().items() if "decode_few_kernel" in k}
    assert len(few) == 33                                             # 16, 32, 64 tokens: three formats at 2 to 4 bits, V2 at 5 and 6
    for k, v in few.items():
        assert v["vgpr_spills"] == 0 and v["agprs"] == 0 and v["scratch_bytes_per_lane"] == 0, (k, v)


def test_no_load_in_inline_asm_has_a_result_register():
    """The compiler takes an asm statement's results as there when it ends: it may move, reuse or overwrite their
    registers while the load is under way.  A load into registers is a builtin's; asm loads go to LDS."""
    found = 0
    for path in glob.glob(os.path.join(os.path.dirname(xfp.library_path()), "csrc", "*")):
        with open(path) as f:
            text = f.read()
        for m in re.finditer(r"\basm\b[^(;]*\((.*?)\);", text, re.S):
            code, _, operands = re.sub(r'"((?:[^"\\]|\\.)*)"\s*(?="|:|$)', r"\1", m.group(1)).partition("::")
            if re.search(r"(global|buffer|flat|scratch)_load|ds_read|s_load", m.group(1)):
                found += 1
                assert operands and re.search(r"\blds\b", code), (path, m.group(0))
    assert found == 1                                                 # load_to_lds (index words, activations)


def test_the_resident_kernel_reads_no_token_behind_the_last():
    """Its activations are the first thing in a workgroup's LDS, a row per token: a row that is not there may lie behind all
    of it (three rows of 28672 columns behind the only one are 172 KB).  Every row that it addresses is one of the call's."""
    with open(os.path.join(os.path.dirname(xfp.library_path()), "csrc", "xfp_decode_few.inc.h")) as f:
        rows = re.findall(r"((?:min\([^()]*\)|\([^()]*\)|[\w\[\]]+)) \* fa\.xpitch", f.read())
    # M: the size of them all; xm[b]: staged only below M
    assert sorted(rows) == ["M", "min(16u * t + i, M - 1)", "min(chunk0 + m4 + m, M - 1)", "xm[b]"]


def test_kernels_that_address_lds_from_zero_have_no_static_lds():
    """The matrix-core kernels, the tile kernel, the V2a streaming kernels and the down projection with the router's sum
    form lookup addresses that assume their tables at LDS offset 0 (one v_perm_b32 writes the whole address).  That holds because they declare
    dynamic LDS only; a static __shared__ array added to one of them would move the tables and the kernel would
    return without writing (its guard).  This pins the guarantee at build time."""
    res = resources()
    names = [k for k in res if any(p in k for p in ("decode_batch_kernel", "decode_tile_kernel", "decode_wide_kernel", "decode_combine_kernel"))]
    assert sum("decode_combine_kernel" in k for k in names) >= 30
    # the streaming kernel's V2a instantiations: template argument 5 (MODE) is 1, or 2 with a scale and a mid-point per group
    names += [k for k in res if "decode_stream_kernelILi" in k and k.split("decode_stream_kernelI")[1].split("E")[4] in ("Li1", "Li2")]
    assert len(names) >= 100
    for k in names:
        assert res[k]["lds_bytes"] == 0, (k, res[k])
