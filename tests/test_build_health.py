"""The hot kernels must not spill registers inside their loops: a scratch (private memory) access there
is a memory operation whose wait also drains the asynchronous global -> LDS copies in flight, which has
cost the Q-smoothing backward 15 % once.  This compiles the device code to assembly (no GPU needed)
and reads each kernel's register and scratch figures from the code object metadata."""
import os
import re
import subprocess
import tempfile

import pytest

from paper_2603_02170_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


_TEXT = []      # the assembly that `kernels` was read from


@pytest.fixture(scope="module")
def kernels():
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "sagebwd.s")
        cmd = [build.hipcc_path(), "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
               "-packed-fp32-ops", "-Wno-unused-command-line-argument", "-I", os.path.join(ROOT, "include"),
               "-I", os.path.join(ROOT, "paper_2603_02170_amd", "csrc"), "--cuda-device-only", "-S",
               os.path.join(ROOT, "paper_2603_02170_amd", "csrc", "sagebwd_api.hip"), "-o", out]
        res = subprocess.run(cmd, capture_output=True, text=True)
        assert res.returncode == 0, res.stderr[-2000:]
        text = open(out).read()
    info = {}
    for block in text.split(".amdhsa_kernel ")[1:]:
        name = block.split("\n")[0].strip()
        get = lambda key: int(re.search(key + r"\s+(\d+)", block).group(1))
        info[name] = dict(vgpr=get(r"\.amdhsa_next_free_vgpr"), scratch=get(r"\.amdhsa_private_segment_fixed_size"),
                          lds=get(r"\.amdhsa_group_segment_fixed_size"))
    assert not re.search(r"\bv_pk_(fma|mul|add)_f32\b", text), "packed FP32 instructions must stay out of the build"
    _TEXT.append(text)
    return info


def _pick(kernels, stem, *template_bits):
    hits = [v for k, v in kernels.items() if stem in k and all(b in k for b in template_bits)]
    assert hits, (stem, template_bits)
    return hits


def test_backward_kernels_keep_their_loops_free_of_scratch(kernels):
    # sage_bwd_kernel<D, CAUSAL, QSMOOTH>: the instantiations the benchmark workloads run
    # (..., MODE, KV128>: ELi0ELb0E is the 64 x 64 kernel; the instantiations for numerics blocks of 128 may park
    # a few registers, they are not the fast path)
    for bits in (("ILi128ELb1ELb0E",), ("ILi128ELb0ELb0E",), ("ILi128ELb1ELb1E",), ("ILi64ELb1ELb0E",), ("ILi64ELb1ELb1E",)):
        for k in _pick(kernels, "sage_bwd_kernel", *bits, "ELi0ELb0EEEv"):
            assert k["scratch"] == 0 and k["vgpr"] <= 256, (bits, k)
            assert k["lds"] <= 160 * 1024
    for k in _pick(kernels, "sage_bwd_kernel"):
        assert k["scratch"] <= 24 and k["vgpr"] <= 256 and k["lds"] <= 160 * 1024, k
    for k in _pick(kernels, "sage_bwd_dq_split_kernel", "ILi128E"):
        # two workgroups of eight waves per CU
        assert k["scratch"] == 0 and k["vgpr"] <= 128 and 2 * k["lds"] <= 160 * 1024, k
    for k in _pick(kernels, "sage_bwd_dq_split_kernel", "ILi64E"):
        assert k["scratch"] == 0 and k["vgpr"] <= 168 and 3 * k["lds"] <= 160 * 1024, k
    for k in _pick(kernels, "sage_bwd_dq_kernel"):
        # three workgroups of four waves per CU: 168 registers, a third of the LDS
        assert k["scratch"] == 0 and k["vgpr"] <= 168 and 3 * k["lds"] <= 160 * 1024, k


def test_forward_kernels_fit_their_occupancy(kernels):
    # four-wave workgroups, two per CU at d = 128 (256 registers) and three at d = 64 (168), nothing in scratch, with numerics
    # blocks of 64 keys or 128
    for k in _pick(kernels, "sage_fwd_kernel", "ILi128E"):
        assert k["vgpr"] <= 256 and k["scratch"] == 0 and 2 * k["lds"] <= 160 * 1024, k
    for k in _pick(kernels, "sage_fwd_kernel", "ILi64E"):
        assert k["vgpr"] <= 168 and k["scratch"] == 0 and 3 * k["lds"] <= 160 * 1024, k


def test_the_forms_for_calls_that_do_not_fill_the_machine(kernels):
    # one wave per SIMD of four-wave workgroups and two: registers only, nothing in scratch
    for k in _pick(kernels, "sage_fwd_pair_kernel"):
        assert k["scratch"] == 0 and k["vgpr"] <= 256 and 2 * k["lds"] <= 160 * 1024, k
    # eight waves and most of the LDS of a CU
    for k in _pick(kernels, "sage_fwd_split_kernel") + _pick(kernels, "sage_fwd_quad_kernel"):
        assert k["scratch"] == 0 and k["vgpr"] <= 256 and k["lds"] <= 160 * 1024, k
    # nothing in scratch
    for k in _pick(kernels, "sage_fwd_decode_kernel"):
        assert k["scratch"] == 0 and k["vgpr"] <= 512 and k["lds"] <= 160 * 1024, k
    # one KV block per workgroup: two workgroups per CU at d = 64 without Q-smoothing
    for k in _pick(kernels, "sage_bwd_single_kernel"):
        assert k["scratch"] == 0 and k["vgpr"] <= 256 and k["lds"] <= 160 * 1024, k
    for bits in ("ILi64ELb1ELb0E", "ILi64ELb0ELb0E"):
        for k in _pick(kernels, "sage_bwd_single_kernel", bits):
            assert k["vgpr"] <= 128 and 2 * k["lds"] <= 160 * 1024, k


def test_workgroups_share_a_cu_as_the_order_of_their_launch_says(kernels):
    # fwd_per_cu, kMaxSweepPerCu, bwd_single_per_cu: waves per SIMD by their registers (512, in eights), workgroups by that and by the LDS
    def per_cu(k, waves):
        return min(512 // (-(-k["vgpr"] // 8) * 8) * 4 // waves, 160 * 1024 // k["lds"])

    for d, at_least in (("ILi64E", 3), ("ILi128E", 2)):
        assert all(per_cu(k, 4) >= at_least for k in _pick(kernels, "sage_fwd_kernel", d))
        assert all(per_cu(k, 4) >= 2 for k in _pick(kernels, "sage_fwd_pair_kernel", d))
        assert all(per_cu(k, 8) == 2 for k in _pick(kernels, "sage_bwd_kernel", d, "ELi1ELb0EEEv"))
    for bits, n in (("ILi64ELb1ELb0E", 2), ("ILi64ELb1ELb1E", 1), ("ILi128ELb1ELb0E", 1), ("ILi128ELb1ELb1E", 1)):
        assert all(per_cu(k, 8) == n for k in _pick(kernels, "sage_bwd_single_kernel", bits))


def test_the_sums_of_plain_keys_do_not_pay_for_the_normalising_ones(kernels):
    # five waves per SIMD of the quantiser at d = 128 with the mean inside, seven of the chunk sums
    for k in _pick(kernels, "prepass_quant_kernel", "ILi128ELi1ELi1E") + _pick(kernels, "prepass_quant_kernel", "ILi64ELi2ELi1E"):
        assert k["scratch"] == 0 and k["vgpr"] <= 96, k
    for k in _pick(kernels, "kmean_partial_kernel", "ELi0E"):
        assert k["scratch"] == 0 and k["vgpr"] <= 72, k


def test_two_workgroups_of_the_decoding_kernel_share_a_cu(kernels):
    for k in _pick(kernels, "sage_fwd_decode_kernel"):
        assert k["vgpr"] <= 256 and 2 * k["lds"] <= 160 * 1024, k


def test_backward_with_four_kv_blocks_keeps_its_operands_in_registers(kernels):
    # two waves per SIMD and 157 KB of LDS
    for k in _pick(kernels, "sage_bwd_wide_kernel"):
        assert k["scratch"] == 0 and k["vgpr"] <= 256 and k["lds"] <= 160 * 1024, k


def _registers(operands):
    """Vector registers that an instruction names, as (first, last) ranges."""
    return [(int(m[1]), int(m[2] or m[1])) for m in re.finditer(r"\bv\[?(\d+)(?::(\d+)\])?", operands)]


def test_products_that_start_from_the_inline_constant_are_read_by_their_chain_only(kernels):
    """mfma_from_bias is assembly that the compiler does not know for a matrix product: its result may not lie on its
    operands' registers, and the first thing that touches it has to be the next product of the chain, with it as C."""
    code = [line.split(";")[0].strip() for line in _TEXT[0].split("\n")]
    code = [line for line in code if line and not (line.startswith(".") and not line.startswith(".LBB"))]
    starts = [n for n, line in enumerate(code) if line.startswith("v_mfma") and "0.15915494" in line]
    assert len(starts) > 100
    overlaps = lambda a, b: a[0] <= b[1] and b[0] <= a[1]
    for n in starts:
        dst, *operands = _registers(code[n])
        assert dst[1] - dst[0] == 15 and len(operands) == 2
        assert not any(overlaps(dst, r) for r in operands), code[n]
        for line in code[n + 1:]:
            assert not line.startswith((".LBB", "s_cbranch", "s_branch", "s_endpgm")), (code[n], line)
            if any(overlaps(dst, r) for r in _registers(line)):
                assert line.startswith("v_mfma_i32_32x32x32_i8") and _registers(line)[3:] == [dst], (code[n], line)
                break


def test_kernels_of_short_heads(kernels):
    # nothing in scratch; with one block at d = 128 two workgroups of eight waves per CU, of the forward with two blocks as well
    for stem in ("sage_fwd_short_kernel", "sage_bwd_short_kernel"):
        for k in _pick(kernels, stem):
            assert k["scratch"] == 0 and k["vgpr"] <= 256 and k["lds"] <= 160 * 1024, k
    for k in _pick(kernels, "sage_bwd_short_kernel", "ILi128E", "ELi1ELb") + _pick(kernels, "sage_fwd_short_kernel", "ILi128E"):
        assert k["vgpr"] <= 128 and 2 * k["lds"] <= 160 * 1024, k
