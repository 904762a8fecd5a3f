"""Facts about the gfx950 code of single kernels that their speed rests on, read from the instructions that the library's own
sources compile to (hipcc cross-compiles, so no GPU is needed)."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2504_11681_amd", "csrc")


def instructions(tmp_path, header, instance):
    """Instructions of the explicitly instantiated kernel templates of `instance`, in order, by mangled name."""
    src = tmp_path / "kernels.hip"
    src.write_text(f'#include "{header}"\nnamespace tfno {{\n{instance}\n}}\n')
    out = tmp_path / "kernels.s"
    subprocess.run(["hipcc", "--cuda-device-only", "--offload-arch=gfx950", "-O3", "-std=c++17", "-fno-gpu-rdc", "-Xclang",
                    "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", CSRC, "-S", "-o", str(out), str(src)],
                   check=True, capture_output=True, timeout=300)
    kernels = {}
    for m in re.finditer(r"^(_Z\w+I\w+EvP\w+):[^\n]*\n(.*?)s_endpgm", out.read_text(), flags=re.S | re.M):
        kernels[m.group(1)] = re.findall(r"^\s+([a-z]\w+)", m.group(2), flags=re.M)
    assert kernels
    return kernels


def test_the_direct_contraction_of_tiles_addresses_with_32_bits(tmp_path):
    """Spectra in tiles of 128 modes have their channels 128 apart.  With that distance in 64 bits, as spectra in rows need it, every
    channel's address is a shift of two registers in the loop (B 758, 54 -> 131 channels, 43 points, 8 modes: 33.9 -> 37.0 us the layer)."""
    for name, code in instructions(tmp_path, "cgemm_modes_kernel.h",
                                   "template __global__ void k_cgemm_modes_direct<4, 6>(const c64 *, const c64 *, c64 *, int, int, float, ModeRows);\n"
                                   "template __global__ void k_cgemm_modes_direct<2, 8>(const c64 *, const c64 *, c64 *, int, int, float, ModeRows);").items():
        assert "v_mfma_f32_32x32x16_bf16" in code, name
        assert code.count("v_lshlrev_b64") == 0, (name, code.count("v_lshlrev_b64"))


def test_pruned_kernels_of_1024_points_build_their_tables_first_and_divide_in_32_bits(tmp_path):
    """The pencil of a lane is taken apart into batch element and channel with a 32-bit division (a 64-bit one is some 120 instructions
    before the first load; its estimate is a v_rcp_f32), and the twiddle tables are under way before the first load of the field: behind the loads
    both kernels of an 1024-point layer were 0.2 - 0.6 us slower."""
    code = instructions(tmp_path, "pruned1d_kernel.h", "".join(
        f"template __global__ void k_fwd1d<1024, 64, {real}, 0>(const c64 *, c64 *, int, long long, int, int, long long, long long);\n"
        f"template __global__ void k_inv1d<1024, 64, {real}, 0>(const c64 *, c64 *, int, long long, int, int, long long);\n" for real in ("true", "false")))
    assert len(code) == 4
    for name, ins in code.items():
        assert not [i for i in ins if i.startswith("v_rcp_f32")], name
        first = {kind: next(k for k, i in enumerate(ins) if i.startswith(kind)) for kind in ("ds_write", "global_load")}
        assert first["ds_write"] < first["global_load"], (name, first)
