"""Register assignment of the DPP blocks in csrc/lanes.h.  A block of several
instructions writes its first outputs before it reads its last inputs, so no
output may share a register with an input that is read later: not even where
both hold the same value on entry (a zero accumulator and a zero row)."""
import os
import re
import subprocess

import pytest

from paper_1805_05278_amd import build

PROBE = r"""
#include "lanes.h"
using namespace miqr;
#define FILL(a, n) for (int i = 0; i < n; ++i) a[i] = c
template <typename T, int N>
__device__ void dots(T* o, T c) {
  T x[N], d0 = c, d1 = c;
  FILL(x, N);
  dots_bcast<3>(x, d0, d1);
  o[threadIdx.x] = d0 + d1;
}
template <typename T, int N>
__device__ void update(T* o, T c) {
  T x[N];
  FILL(x, N);
  update_bcast<3>(x, c);
  for (int i = 0; i < N; ++i) o[threadIdx.x + 64 * i] = x[i];
}
__global__ void k_dots(double* o, float* f, double c, float cf) {
  dots<double, 16>(o, 0.0);
  dots<double, 8>(o + 64, c);
  dots<float, 16>(f, cf);
}
__global__ void k_update(double* o, float* f, double c, float cf) {
  update<double, 16>(o, c);
  update<double, 8>(o + 1024, c);
  update<float, 16>(f, cf);
}
__global__ void k_terms(double* o, const double* v) {
  double t[16], s0 = 0.0, s1 = 0.0;
  for (int i = 0; i < 16; ++i) t[i] = 0.0;
  bcast_terms<0>(v[threadIdx.x], t, s0, s1);
  o[threadIdx.x] = s0 + s1;
}
__global__ void k_axpy(double* o, double c) {
  double y[16];
  FILL(y, 16);
  bcast_axpy<0, 15>(c, c, y);
  for (int i = 0; i < 16; ++i) o[threadIdx.x + 64 * i] = y[i];
}
__global__ void k_fmacs(double* o, double c) {
  double x[16], y[16];
  FILL(x, 16);
  FILL(y, 16);
  bcast_fmacs<2, 1, 16>(x, y, c);
  bcast_fmacs_self<2, 3, 16>(x, c);
  for (int i = 0; i < 16; ++i) o[threadIdx.x + 64 * i] = x[i] + y[i];
}
"""


def assembly(src, out):
    cmd = [build.HIPCC] + build.FLAGS + ["-x", "hip", "--offload-device-only", "-S", src, "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    with open(out) as f:
        return f.read()


def registers(operand):
    m = re.match(r"v\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.match(r"v(\d+)$", operand)
    return {int(m.group(1))} if m else set()


def overlaps(text):
    """(blocks with DPP products, instructions that read what an earlier one of
    their block wrote)."""
    blocks, bad = 0, []
    for body in re.findall(r";+\s*#?ASMSTART(.*?);+\s*#?ASMEND", text, re.S):
        lines = [x.strip() for x in body.splitlines() if "v_fmac" in x]
        blocks += bool(lines)
        written = set()
        for line in lines:
            ops = [x.strip().split(" ")[0] for x in line.split(None, 1)[1].split(",")]
            if any(registers(x) & written for x in ops[1:3]):
                bad.append(line)
            written |= registers(ops[0])
    return blocks, bad


def test_outputs_apart_from_later_inputs(tmp_path):
    src = tmp_path / "probe.hip"
    src.write_text(PROBE)
    blocks, bad = overlaps(assembly(str(src), str(tmp_path / "probe.s")))
    assert blocks >= 16
    assert bad == []


@pytest.mark.parametrize("source", ["tsqr.hip", "batched_blk.hip"])
def test_kernels_outputs_apart_from_later_inputs(source, tmp_path):
    blocks, bad = overlaps(assembly(os.path.join(build.CSRC, source), str(tmp_path / "k.s")))
    assert blocks > 100
    assert bad == []
