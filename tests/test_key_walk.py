"""The scalar arithmetic of the fused kernels' walks (KeyWalk, FastDiv of rsa_common.h), on the host: every order of
ranks, both ownerships, splits and groups against the stages written out one by one; the rows in the order of their tokens."""
import os

from test_sanitizers import ROOT, SAN, run


def test_walks_and_divisions(tmp_path):
    exe = str(tmp_path / "walks")
    run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "-O1", "-std=c++17",
         "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2105_13120_amd", "csrc"),
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument",
         "-Xarch_host", "-fsanitize=undefined", "-Xarch_host", "-fno-sanitize-recover=all",
         "-x", "hip", os.path.join(SAN, "walk_driver.cpp"), "-o", exe])
    assert "WALKS_OK" in run([exe])
