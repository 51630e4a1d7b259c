"""The inline assembly of the tile kernels' banded sums and sweeps (csrc/tile.h), compiled for gfx950 with operands that
start equal to the sums: no operand may live in a register that the block writes before it reads the operand.  The
numbers of reads of a block's own results are those of its recurrence."""
import os
import re
import subprocess

import pytest

from paper_2206_09878_amd import build

LOADS = "double T[24], X[12]; for (int i = 0; i < 24; ++i) T[i] = t[i * 64 + threadIdx.x];" \
        " for (int i = 0; i < 12; ++i) X[i] = t[(24 + i) * 64 + threadIdx.x];"
ZEROS = "double T[8], X[6] = {0}, V[4] = {0}, Z[4] = {0}; for (int i = 0; i < 8; ++i) T[i] = t[i * 64 + threadIdx.x];"
# name: (body, each sum starting as the operand that the block reads last or as zero with all of them; reads of own results)
BLOCKS = {
    "fb8": (LOADS + "double a = X[0], b = 0, c = 0; fb8<3>(a, T, X);", 0),
    "fb12": (LOADS + "double a = X[11], b = 0, c = 0; fb12<3>(a, T, X);", 0),
    "fb2x4": (LOADS + "double a = X[3], b = X[3], c = 0; fb2x4<3>(a, b, T, T + 4, X);", 0),
    "fb3x4": (LOADS + "double a = X[3], b = X[3], c = X[3]; fb3x4<3>(a, b, c, T, T + 4, T + 8, X);", 0),
    "fb2x5": (LOADS + "double a = X[4], b = X[4], c = 0; fb2x5<3>(a, b, T, T + 5, X);", 0),
    "fb_l4": (ZEROS + "fb_l4<0>(V, T, X); double a = V[0] + V[1], b = V[2], c = V[3];", 1 + 2 + 3),
    "fb_u4": (ZEROS + "fb_u4<15>(V, Z, T, X); double a = Z[0] + Z[1], b = Z[2], c = Z[3];", 4 + 1 + 2 + 3),
}


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    """Assembly of one kernel for each block."""
    with open(os.path.join(build.CSRC, "tile.h")) as f:
        src = f.read()
    helpers = src[src.index("#define LMVD_FB("):src.index("template <int I, int E, class F>")]
    kernels = ['extern "C" __global__ void k_%s(const double* t, double* o) { %s o[threadIdx.x] = a;'
               " o[64 + threadIdx.x] = b; o[128 + threadIdx.x] = c; }\n" % (name, body) for name, (body, _) in BLOCKS.items()]
    d = tmp_path_factory.mktemp("asm")
    (d / "blocks.hip").write_text("#include <hip/hip_runtime.h>\n" + helpers + "".join(kernels))
    subprocess.run([build.hipcc(), "-O3", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-S", "--offload-device-only", str(d / "blocks.hip"), "-o", str(d / "blocks.s")],
                   check=True, capture_output=True)
    return (d / "blocks.s").read_text()


@pytest.mark.parametrize("name", sorted(BLOCKS))
def test_operands_keep_their_registers(listing, name):
    body = listing[listing.index("\nk_%s:" % name):]
    body = body[:body.index("s_endpgm")]
    block = body[body.index(";#ASMSTART"):body.index(";#ASMEND")]
    ops = re.findall(r"v_fmac_f64_dpp (v\[\S+\]), (v\[\S+\]), (v\[\S+\]) ", block)
    assert len(ops) == block.count("v_fmac_f64_dpp") > 0
    written = {d for d, _, _ in ops}
    assert not written & {s for _, s, _ in ops}                       # tables
    assert all(d != x for d, _, x in ops)                             # no sum is its own operand
    assert sum(x in written for _, _, x in ops) == BLOCKS[name][1]
