"""Shared-memory sizes of the training kernels against the indexes they use, for every hash width (compiled on the CPU)."""
import os
import subprocess

from paper_2506_02572_amd import build


def test_column_sums_have_a_row_per_wave_and_per_slice(tmp_path):
    src = tmp_path / "shapes.hip"
    src.write_text('#include "%s"\n' % os.path.join(build.CSRC, "hata_train.hip") + "".join(
        "static_assert(hata::TrainShape<%d>::COL_ROWS >= hata::TrainShape<%d>::THREADS / %s, \"rows\");\n" % (r, r, per)
        for r in (32, 64, 128, 256) for per in ("64", "hata::TrainShape<%d>::COLS" % r)))
    res = subprocess.run([build.HIPCC, "--offload-arch=gfx950", "-std=c++17", "-fsyntax-only", "--cuda-host-only", str(src)],
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout
