"""The gfx950 kernels compile with no scratch memory and no register spills
(a private segment in a layer kernel means operands round-trip through
memory and the MFMA pipes starve).  CPU only: cross-compiles with hipcc."""

import shutil

import pytest

from paper_2107_02737_amd.build import compile_command, hipcc, kernel_resources


@pytest.fixture(scope="module")
def resources():
    try:
        hipcc()
    except RuntimeError:
        pytest.skip("hipcc not available")
    return kernel_resources()


def test_every_kernel_present(resources):
    names = " ".join(resources)
    for k in ["k_gershgorin_rows", "k_bounds_final", "k_input_layer", "k_split", "k_sym_split",
              "k_sym_f32", "k_finish_loop", "k_split_tail", "k_mirror_upper", "k_lz_matvec",
              "k_lz_apply", "k_lz_bounds", "k_mulliken", "k_atom_matvec", "k_xl_step",
              "k_xl_finish", "k_nvt_first", "k_nvt_second"]:
        assert k in names


def test_no_scratch_no_spills(resources):
    for name, r in resources.items():
        if "k_sym_split" in name:
            # register file full by design (256 AGPR accumulators + double-buffered
            # fragments): a few scalars may spill outside the K loop, never inside
            assert r["hot_loop_scratch"] == 0, name
            assert r["private_segment_fixed_size"] <= 64 and r["vgpr_spill_count"] <= 8, name
        else:
            assert r["private_segment_fixed_size"] == 0, name
            assert r["vgpr_spill_count"] == 0, name


def test_mfma_kernels_have_a_clean_hot_loop(resources):
    for name, r in resources.items():
        if "k_sym" in name:
            assert r["hot_loop_scratch"] == 0, name


def test_layer_kernels_fit_their_occupancy(resources):
    for name, r in resources.items():
        if "k_sym" in name:
            assert r["vgpr_count"] <= 512, name
            assert r["group_segment_fixed_size"] <= 160 * 1024, name


def test_kernels_of_smaller_orders(resources):
    """Every tile size of every kind is there, without spills in the loop, within the
    registers and the LDS of its occupancy."""
    names = " ".join(resources)
    for kind in range(3):
        for rows in (1, 2, 3):
            assert f"k_sym_waveILi{kind}ELi{rows}ELi1EE" in names
        assert f"k_sym_midILi{kind}ELi1EE" in names
    for rows in (1, 2, 3):
        assert f"k_sym_waveILi0ELi{rows}ELi2EE" in names
        for segments in (1, 2, 4):
            assert f"k_wave_f32ILi{rows}ELi{segments}EE" in names
    assert "k_sym_midILi0ELi2EE" in names
    for name, r in resources.items():
        if "k_wave_f32" in name:
            assert r["hot_loop_scratch"] == 0, name
            # eight waves, two per SIMD; four of the 96-row tiles
            assert r["vgpr_count"] <= (512 if "ILi3E" in name else 256), name
            assert r["group_segment_fixed_size"] <= 160 * 1024, name


@pytest.mark.parametrize("segments", [1, 2, 3, 4])
def test_segments_of_an_fp32_product(tmp_path, segments):
    """A launch passes as many operands as its kernel reads: a sum of three does
    not compile (the four-segment kernel would read a null operand)."""
    import subprocess
    src = tmp_path / "segments.hip"
    src.write_text(f"""
#include "sp2_capi.hip"
sp2_status call(const WS& w, const float* x, const Epi& e, const Decide& d, hipStream_t st) {{
  const float* A[{segments}] = {{{", ".join(["x"] * segments)}}};
  return launch_f32(w, A, A, e, d, st);
}}
""")
    cmd = [c for c in compile_command(str(tmp_path / "out"), [str(src)]) if c != "-shared"]
    res = subprocess.run(cmd[:-2] + ["--offload-host-only", "-fsyntax-only"], capture_output=True,
                         text=True)
    assert (res.returncode == 0) == (segments != 3), res.stderr
    if segments == 3:
        assert "segments of an FP32 product" in res.stderr


def test_hipcc_on_path_or_rocm():
    assert shutil.which("hipcc") or hipcc()
