"""A carry (VCC or a register pair) that a vector instruction has written is read by another one after two
wait states at the earliest.  The compiler pads its own code; inside an asm statement nobody does, so the
kernels whose selection counts with compares and additions with carry are compiled and looked through."""
import os
import re
import subprocess

from paper_2502_06728_amd import build

KERNELS = r"""
#include "direct_kernels.hip.h"
#include "half_tile_kernels.hip.h"
#include "pair_kernels.hip.h"
namespace deto {
#define ARGS KParams, int64_t, int64_t, int64_t, const void*, float*, void*, void*, float*
template __global__ void compress_direct<16, false>(ARGS);
template __global__ void compress_split<64, 2, false>(ARGS);
template __global__ void compress_halves<false, 16, false>(ARGS);
template __global__ void compress_pair<96, false>(ARGS);
}
"""
WAITS = 2


def early_reads(text):
    """(line number, reading instruction) of every carry that is read too early, and the number looked at."""
    early, seen, written, at = [], 0, {}, 0
    for number, line in enumerate(text.splitlines(), 1):
        line = line.split(";")[0].strip()
        if not line or line.startswith((".", "//")) or line.endswith(":"):
            if line.endswith(":"):
                written = {}
            continue
        op, _, rest = line.partition(" ")
        args = [a.strip() for a in rest.split(",")]
        if op == "s_nop":
            at += int(args[0]) + 1
            continue
        if re.match(r"v_(addc|subb|subbrev)_co|v_cndmask", op):
            carry = args[-1] if args[-1] == "vcc" or args[-1].startswith("s[") else "vcc"
            if carry in written:
                seen += 1
                if at - written[carry] < WAITS:
                    early.append((number, line))
        at += 1
        if re.match(r"v_cmp_", op):
            written[args[0]] = at
        elif re.match(r"v_(addc?|subb?|subrev|subbrev)_co", op):
            written[args[1]] = at
    return early, seen


def test_the_search_finds_what_it_looks_for():
    pair = "v_cmp_ge_u32 vcc, v1, v2\n{}v_addc_co_u32 v0, vcc, v0, v0, vcc\n"
    assert early_reads(pair.format(""))[0] and early_reads(pair.format("s_nop 0\n"))[0]
    assert early_reads(pair.format("s_nop 1\n")) == ([], 1)
    assert early_reads(pair.format("v_mov_b32 v3, v4\nv_mov_b32 v3, v4\n")) == ([], 1)


def test_no_carry_is_read_before_it_is_there(tmp_path):
    (tmp_path / "kernels.hip").write_text(KERNELS)
    flags = ["-O1" if f == "-O3" else f for f in build.HIPCC_FLAGS]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--cuda-device-only", "-S",
                    "-I", build.CSRC, "-o", str(tmp_path / "kernels.s"), str(tmp_path / "kernels.hip")],
                   check=True, capture_output=True)
    early, seen = early_reads((tmp_path / "kernels.s").read_text())
    assert seen > 200 and not early, early[:5]
