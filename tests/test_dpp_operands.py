"""The four-column DPP blocks of the mat-vecs write their accumulators before
they have read all operands: no accumulator may share a register with an
operand, also where it starts with that operand's value (the compiler then
gives both one register unless the accumulator is an early clobber).  Compiled
to assembly on the CPU, with one and two DoF slots a lane, accumulators that
start as the vector or as a matrix column."""
import re
import subprocess

import pytest

from paper_2502_11129_amd import build as B

SOURCE = """
#include "rollout_kernel.hpp"
using namespace simk;
template <int S> __device__ void load(float (&m)[S], const float* p) {
  for (int s = 0; s < S; ++s) m[s] = p[64 * s + threadIdx.x];
}
template <int S, bool COLUMN> __global__ void one(const float* p, float* o) {
  float m0[S], m1[S], m2[S], m3[S], y[S];
  load(m0, p); load(m1, p + 128); load(m2, p + 256); load(m3, p + 384);
  const float x = p[512 + threadIdx.x];
  for (int s = 0; s < S; ++s) y[s] = COLUMN ? m3[s] : x;
  fmac1_bcast<4>(m0, m1, m2, m3, x, y);
  for (int s = 0; s < S; ++s) o[64 * s + threadIdx.x] = y[s];
}
template <int S, bool COLUMN> __global__ void three(const float* p, float* o) {
  float m0[S], m1[S], m2[S], m3[S], a[S], b[S], c[S];
  load(m0, p); load(m1, p + 128); load(m2, p + 256); load(m3, p + 384);
  const float x = p[512 + threadIdx.x], y = p[576 + threadIdx.x], z = p[640 + threadIdx.x];
  for (int s = 0; s < S; ++s) { a[s] = COLUMN ? m3[s] : x; b[s] = COLUMN ? m2[s] : y; c[s] = COLUMN ? m1[s] : z; }
  fmac3_bcast<4>(m0, m1, m2, m3, x, y, z, a, b, c);
  for (int s = 0; s < S; ++s) {
    o[64 * s + threadIdx.x] = a[s]; o[128 + 64 * s + threadIdx.x] = b[s]; o[256 + 64 * s + threadIdx.x] = c[s];
  }
}
template __global__ void KERNEL<SLOTS, COLUMN>(const float*, float*);
"""
FMAC = re.compile(r"v_fmac_f32_dpp (v\d+), -(v\d+), (v\d+) row_newbcast")


@pytest.mark.parametrize("kernel,vectors", [("one", 1), ("three", 3)])
@pytest.mark.parametrize("slots", [1, 2])
@pytest.mark.parametrize("column", ["false", "true"])
def test_accumulators_share_no_register_with_an_operand(tmp_path, kernel, vectors, slots, column):
    src = SOURCE.replace("KERNEL", kernel).replace("SLOTS", str(slots)).replace("<" + str(slots) + ", COLUMN>", f"<{slots}, {column}>")
    (tmp_path / "t.hip").write_text(src)
    out = tmp_path / "t.s"
    r = subprocess.run([B.HIPCC, *B.COMMON, *B.DEVICE, "--cuda-device-only", "-S", "-I", B.CSRC, str(tmp_path / "t.hip"),
                        "-o", str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    ops = FMAC.findall(out.read_text())
    assert len(ops) == 4 * vectors * slots
    acc = {d for d, _, _ in ops}
    assert len(acc) == vectors * slots
    assert not acc & {s for _, a, b in ops for s in (a, b)}
