"""The CG product reads a slice of the padded matrix through a buffer descriptor
and runs past the slice's width by design.  Only the lane and immediate offsets
of such a load are bounded by the descriptor, so the scalar offset must be 0 in
every one of them; the values read past the width are discarded, so no result
shows it.  Checked in the assembly that the build's flags give."""
import re
import subprocess

from paper_2005_05899_amd import build


def test_every_load_is_bounded_by_the_descriptor(tmp_path):
    out = tmp_path / "stepper.s"
    subprocess.run(["hipcc", *build.HIPCC_FLAGS, "-I", f"{build.ROOT}/include", "-I", build.CSRC, "-S",
                    "--cuda-device-only", f"{build.CSRC}/stepper.hip", "-o", str(out)],
                   check=True, capture_output=True, text=True)
    kernels = re.findall(r"^(_ZN6lesasm15k_spmv_sell_dot\w+):(.*?)^\.Lfunc_end", out.read_text(), re.M | re.S)
    assert len(kernels) == 2
    for name, body in kernels:
        offsets = re.findall(r"\bbuffer_load_\w+ +v\S*, v\w+, s\[\d+:\d+\], (\S+) offen", body)
        assert len(offsets) == body.count("buffer_load_") >= 18, name
        assert set(offsets) == {"0"}, name
