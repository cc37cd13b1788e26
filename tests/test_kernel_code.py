"""Properties of the fused kernel's gfx950 device code (CPU only: compiles
rip_kernels.hip to AMDGPU assembly with the library's own flags).

* bf16 results are stored through v_cvt_pk_bf16_f32 (the conversion that
  tests/test_gpu_ieee_edges.py checks on all 2^32 inputs against
  round-to-nearest-even), and no software rounding sequence stands in for it;
* fp32 subnormals are kept, not flushed (the kernel descriptors' fp32 denorm
  mode is 3: inputs and outputs preserved), as the exact group mean needs;
* no fused multiply-add or multiply-accumulate is emitted: every product and
  sum rounds on its own, in the order the oracle follows;
* no packed fp32 arithmetic is emitted (the library is built without it);
* the pause between the stores of large momentum groups is in one of two copies
  of their code (small launches run the other);
* the registers of the kernel of groups above eight hold the waves per CU that
  the launch policy counts on.
"""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    import importlib.util
    spec = importlib.util.spec_from_file_location(
        "rip_build", os.path.join(ROOT, "paper_1909_08029_amd", "build.py"))
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    out = str(tmp_path_factory.mktemp("asm") / "rip_kernels.s")
    flags = [f for f in b.COMMON if f not in ("-fPIC", "-shared")]
    csrc = os.path.join(ROOT, "paper_1909_08029_amd", "csrc")
    subprocess.run([b.HIPCC, *flags, "--cuda-device-only", "-S", "-I",
                    os.path.join(ROOT, "include"), "-I", csrc, "-x", "hip",
                    os.path.join(csrc, "rip_kernels.hip"), "-o", out],
                   check=True, capture_output=True, text=True, timeout=600)
    return open(out).read()


def instructions(text):
    return re.findall(r"^\s+(v_[a-z0-9_]+)", text, flags=re.M)


def test_bf16_stores_use_the_hardware_conversion(asm):
    ins = instructions(asm)
    assert "v_cvt_pk_bf16_f32" in ins
    # a software round-to-nearest-even would add 0x7fff plus the lsb with
    # 32-bit integer adds and extract bit 16
    assert not re.search(r"0x7fff\b", asm)


def test_fp32_subnormals_are_preserved(asm):
    modes = re.findall(r"\.amdhsa_float_denorm_mode_32\s+(\d+)", asm)
    assert modes and set(modes) == {"3"}


def test_no_fused_multiply_add(asm):
    ins = set(instructions(asm))
    fused = {i for i in ins if re.match(r"v_(pk_)?(fma|fmac|mac|mad|fmamk|fmaak|madmk|madak)", i)
             and "f32" in i}
    assert not fused, fused


def test_no_packed_fp32_arithmetic(asm):
    ins = set(instructions(asm))
    assert not {i for i in ins if i.startswith("v_pk_") and i.endswith("_f32")}


def test_small_launches_store_without_the_pause(asm):
    """Units of k members store 2k vectors a slot with momentum.  Tiles: four
    slots and one for k = 1, two and one for k = 2, one for k = 3 to 5, and for
    k = 6 to 8 one with a pause after each store and one without."""
    kernels = re.findall(r"^_ZN\S*fused_step_kernelILb\dELb1ELb\dE\S*:\s(.*?)\.end_amdhsa_kernel", asm,
                         flags=re.S | re.M)
    assert len(kernels) == 4
    paced = sum(2 * k for k in (6, 7, 8))
    for k in kernels:
        assert len(re.findall(r"\bs_nop 15\b", k)) == paced
        assert len(re.findall(r"\bbuffer_store_dwordx4\b", k)) == \
            (8 + 2) + (8 + 4) + sum(2 * k for k in (3, 4, 5)) + 2 * paced


def test_waves_of_the_wide_kernel_that_registers_hold(asm):
    with open(os.path.join(ROOT, "paper_1909_08029_amd", "csrc", "rip_launch_policy.h")) as f:
        m = re.search(r"int wide_resident\(bool bf16, bool mom\) \{ return bf16 \? "
                      r"\(mom \? (\d+) : (\d+)\) : \(mom \? (\d+) : (\d+)\); \}", f.read())
    bf16_mom, bf16_sgd, f32_mom, f32_sgd = (int(x) for x in m.groups())
    want = {("1", "1"): bf16_mom, ("1", "0"): bf16_sgd, ("0", "1"): f32_mom, ("0", "0"): f32_sgd}
    vgprs = re.findall(r"wide_step_kernelILb(\d)ELb(\d)ELb\dE\S+\n(?:.*\n)*?\s+\.vgpr_count:\s+(\d+)",
                       asm[asm.index("amdhsa.kernels:"):])
    assert len(vgprs) == 8
    for bf16, mom, v in vgprs:
        # 512 registers per lane and SIMD, in blocks of eight; four SIMDs
        assert 4 * min(8, 512 // (-(-int(v) // 8) * 8)) == want[bf16, mom], (bf16, mom, v)
