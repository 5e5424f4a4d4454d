"""The selection's histogram scan reads sixteen bytes at a time: what it is handed carries that alignment in its type, and a plain
array of words (promised four bytes, wherever the compiler happens to place it) does not compile.  CPU only: syntax checks of the
device code."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TOPK = os.path.join(ROOT, "paper_2604_06746_amd", "csrc", "topk.hip")


@pytest.mark.parametrize("bins,compiles", [("__shared__ LdsBins<kBins> h", True), ("__shared__ uint32_t h[kBins]", False)])
def test_histograms_are_aligned_by_type(tmp_path, bins, compiles):
    src = tmp_path / "scan.hip"
    src.write_text("""#include "%s"
namespace skv { namespace {
__global__ void scan_kernel(uint32_t* out) {
  %s;
  __shared__ uint32_t scan[8], res[3];
  select_bin<512, kBins>(h, 1u, scan, res, out, out + 1);
}
} }
""" % (TOPK, bins))
    r = subprocess.run(["hipcc", "--offload-arch=gfx950", "-std=c++17", "--cuda-device-only", "-fsyntax-only", "-x", "hip", str(src)],
                       capture_output=True, text=True)
    assert (r.returncode == 0) == compiles, r.stderr[-2000:]
    assert compiles or "16-byte aligned" in r.stderr
