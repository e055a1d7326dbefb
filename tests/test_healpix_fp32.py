"""The walk's FP32 pixel against the FP64 form, on the CPU (g++)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_fp32_pixel_is_the_fp64_pixel_or_undecided(tmp_path):
    exe = str(tmp_path / "healpix")
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off",
                    "-I", os.path.join(ROOT, "paper_2310_15235_amd", "csrc"),
                    os.path.join(ROOT, "tests", "healpix_main.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    rows = [list(map(int, ln.split())) for ln in out.splitlines()]
    assert [r[0] for r in rows] == [1, 2, 4, 8, 16]
    for nside, plain, plain_unsure, _, wrong in rows:
        assert wrong == 0
        # three floors, each within 1e-5 N of an integer on either side
        assert plain_unsure <= 1.5 * 3 * 2e-5 * nside * plain + 1e-4 * plain
