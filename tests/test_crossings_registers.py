"""The crossings' inline asm writes some operands before it reads others: no
input may share a register with an operand that the block writes, also where a
caller passes one value as both (a crossing count and its step, a crossing and
their minimum, an increment and what it moves).  Compiles such callers for
gfx950 and reads the registers of the blocks in the compiler's output."""
import os
import re
import subprocess

import pytest

from paper_1512_02110_amd import build

SOURCE = r"""
#include "mcrt_crossings.hpp"
using namespace mcrt;

template <typename R, bool LAYER>
__global__ void cross(R* f, int* i) {
    const int t = threadIdx.x;
    R x = f[t], y = f[t + 64], z = f[t + 128];
    int a = i[t], iz = i[t + 64];
    const R r0 = x, r1 = y, r2 = z;
    R rx = r0, ry = r1, rz = r2, tx = r0, ty = r1, tz = r2;
    int k = a;
    const int layer = iz;
    cross_axes<LAYER>(r2, k, rx, ry, rz, tx, ty, tz, a, a, a, r0, r1, r2, r2, r0, r1, iz, layer);
    f[t] = rx; f[t + 64] = ry; f[t + 128] = rz; f[t + 192] = tx; f[t + 256] = ty; f[t + 320] = tz;
    i[t] = k; i[t + 64] = iz;
}

template <typename R>
__global__ void deposit(R* f, int* i) {
    const int t = threadIdx.x;
    const R x = f[t], y = f[t + 64], z = f[t + 128];
    const int a = i[t];
    R tx = x, ty = y, tz = z;
    int k = a;
    dep_cross<R>(z, k, tx, ty, tz, a, a, a, x, y, z);
    f[t] = tx; f[t + 64] = ty; f[t + 128] = tz;
    i[t] = k;
}

template <typename R>
__global__ void flight(R* f, uint32_t* i, int* c, unsigned long long on, unsigned long long go) {
    const int t = threadIdx.x;
    const R x = f[t], y = f[t + 64], z = f[t + 128];
    uint32_t k = i[t];
    int cx = c[t], cy = c[t + 64], cz = c[t + 128];
    const int kx = cx, ky = cy, kz = (int)k;
    unsigned long long mx, my, mz;
    flight_leave<R>(on, z, x, y, k, cx, cy, cz, kx, ky, kz, mx, my, mz);
    R rx = x, ry = y, rz = z, tx = y, ty = z, tz = x, tau = x, tt = y;
    flight_enter<R>(mx, my, mz, go, rx, ry, rz, tx, ty, tz, x, y, z, y, z, x, tau, y, tt, x);
    f[t] = rx + tau; f[t + 64] = ry + tt; f[t + 128] = rz; f[t + 192] = tx; f[t + 256] = ty; f[t + 320] = tz;
    i[t] = k; c[t] = cx; c[t + 64] = cy; c[t + 128] = cz;
}

template __global__ void cross<float, false>(float*, int*);
template __global__ void cross<float, true>(float*, int*);
template __global__ void cross<double, false>(double*, int*);
template __global__ void cross<double, true>(double*, int*);
template __global__ void deposit<float>(float*, int*);
template __global__ void deposit<double>(double*, int*);
template __global__ void flight<float>(float*, uint32_t*, int*, unsigned long long, unsigned long long);
template __global__ void flight<double>(double*, uint32_t*, int*, unsigned long long, unsigned long long);
"""


def _regs(op):
    """Vector registers of an operand."""
    m = re.fullmatch(r"v(\d+)", op) or re.fullmatch(r"v\[(\d+):\d+\]", op)
    if not m:
        return set()
    n = re.fullmatch(r"v\[(\d+):(\d+)\]", op)
    return set(range(int(n[1]), int(n[2]) + 1)) if n else {int(m[1])}


def shared_inputs(block):
    """Instructions of the block whose pure input is a register that the block writes."""
    code = []
    for line in block:
        m = re.match(r"\s*(v_\w+)\s+(.*)", line)
        if m:
            code.append((m[1], [o.strip() for o in m[2].split(",")], line.strip()))
    written = set()
    for op, args, _ in code:
        if not op.startswith("v_cmpx"):
            written |= _regs(args[0])
    bad = []
    for op, args, line in code:
        # the operand that only goes in: of a compare the minimum, of a sum the step, of a product the factor
        pure = args[1] if op.startswith(("v_cmpx", "v_add", "v_mov")) else args[2]
        if _regs(pure) & written:
            bad.append(line)
    return bad


def test_no_input_shares_a_written_register(tmp_path):
    if not os.path.exists(build.hipcc()):
        pytest.skip("no hipcc")
    src, out = tmp_path / "crossings.hip", tmp_path / "crossings.s"
    src.write_text(SOURCE)
    subprocess.run([build.hipcc(), "-S", "--cuda-device-only", str(src), "-o", str(out), "-I", build.CSRC]
                   + build.HIP_FLAGS, check=True, capture_output=True)
    blocks = re.findall(r";;?#ASMSTART\n(.*?)\s*;;?#ASMEND", out.read_text(), flags=re.S)
    blocks = [b.splitlines() for b in blocks if "v_" in b]
    assert len(blocks) == 10  # four crossings, two deposits, two flights of two blocks
    bad = [line for b in blocks for line in shared_inputs(b)]
    assert not bad, bad
