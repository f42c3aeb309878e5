"""AdamW's update loop on bf16 parameters requests a whole batch of parameters and moments before it waits
for any of them: the compiled kernel is looked through, since a wait between the loads (for registers
that an earlier, conditional load may still be writing) shows in no result."""
import os
import re
import subprocess

from paper_2502_06728_amd import build

KERNEL = r"""
#include "split_kernels.hip.h"
namespace deto {
template __global__ void decompress_split<32, 4, true>(KParams, int64_t, int64_t, int64_t, const void*, int64_t,
                                                       const void*, int64_t, void*, AdamPtrs, float*);
}
"""


def shape(text):
    """The order of the update's accesses: p (bf16 parameters), m (a moment), s (stores), w (waits)."""
    kinds = (("p", r"\s*global_load_dwordx2 .* nt$"), ("m", r"\s*global_load_dwordx4 .* nt$"),
             ("s", r"\s*global_store_dwordx[24] .* nt$"), ("w", r"\s*s_waitcnt vmcnt"))
    return "".join(k for line in text.splitlines() for k, pat in kinds if re.match(pat, line))


def test_a_batch_is_requested_together(tmp_path):
    (tmp_path / "kernel.hip").write_text(KERNEL)
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *build.HIPCC_FLAGS, "--cuda-device-only",
                    "-S", "-I", build.CSRC, "-o", str(tmp_path / "kernel.s"), str(tmp_path / "kernel.hip")],
                   check=True, capture_output=True)
    # two pieces a batch at this size: parameters and both moments of each, then the first wait
    assert "pmmpmmw" in shape((tmp_path / "kernel.s").read_text())
