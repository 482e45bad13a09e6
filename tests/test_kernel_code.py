"""Properties of the compiled kernels that no run can show: instantiations are
compiled to gfx950 assembly here (no GPU is needed) and their instructions read.
"""
import os
import re
import subprocess

import pytest

from paper_2509_25840_amd import build as hip_build

ARGS = {"k_hwave": "const Geom, const Tabs, const PCube, const {T} *, const {T} *, {T} *, const double, const int",
        "k_pwave": "const Geom, const Tabs, const PCube, const {T} *, {T} *, const double *",
        "k_pwave2": "const Geom, const Tabs, const PCube, const {T} *, {T} *, const double *"}


def assembly(tmp_path, kernel, T, args):
    """The assembly of one instantiation, a list of instruction lines."""
    if not os.path.exists(hip_build.HIPCC):
        pytest.skip("no hipcc")
    src, out = tmp_path / "one.hip", tmp_path / "one.s"
    src.write_text('#include "wave.h"\nnamespace chfpe {\n'
                   f"template __global__ void {kernel}<{args}>({ARGS[kernel].format(T=T)});\n}}\n")
    subprocess.run([hip_build.HIPCC, *hip_build.FLAGS, "-I", os.path.join(hip_build.ROOT, "include"), "-I",
                    hip_build.CSRC, "--cuda-device-only", "-S", str(src), "-o", str(out)], check=True,
                   stderr=subprocess.DEVNULL)
    return [ln.strip() for ln in out.read_text().splitlines() if re.match(r"\s+[a-z]", ln)]


@pytest.mark.parametrize("args", ["double, 8, 0, 2", "double, 24, 6, 2", "double, 32, 0, 2", "float, 16, 0, 2"])
def test_the_waves_of_two_mode_k_hwave_meet_at_no_barrier(tmp_path, args):
    """The waves of a two-mode workgroup hold tasks of different hierarchy
    elements and branch on them: with a barrier in both paths the waves of a
    workgroup would wait at different ones."""
    code = assembly(tmp_path, "k_hwave", args.split(",")[0], args)
    assert not any(ln.startswith("s_barrier") for ln in code)


@pytest.mark.parametrize("kernel,args", [("k_pwave", "double, double, 8, 1, false, false"),
                                         ("k_pwave", "double, double, 24, 0, false, false"),
                                         ("k_pwave", "double, double, 24, 9, false, false"),
                                         ("k_pwave", "float, float, 16, 0, false, false"),
                                         ("k_pwave2", "double, double, 16, 4, false, false")])
def test_buffer_loads_keep_their_whole_offset_under_the_bounds_check(tmp_path, kernel, args):
    """Loads past a block, and of a neighbour that is not there, rely on the
    buffer's size.  Only the offset per lane is compared with it, so the
    instruction's scalar offset (the operand before "offen") has to be zero."""
    code = [ln for ln in assembly(tmp_path, kernel, args.split(",")[0], args) if ln.startswith("buffer_load")]
    assert code
    for ln in code:
        assert re.search(r", 0 offen( offset:\d+)?$", ln), ln
