"""fma_row (csrc/resident_impl.h): no sum shares a register with the factors, which
later instructions of the block still read, also where both start with one value."""
import os
import re
import subprocess

from paper_2506_10257_amd.build import CXXFLAGS, HIPCC

SRC = """
#include "resident_impl.h"
template <int B, typename T> __global__ void k_probe(const T* in, T* out) {
  const T a = in[threadIdx.x], p = in[64 + threadIdx.x];
  T l[B];
  for (int k = 0; k < B; ++k) l[k] = k & 1 ? p : a;
  rpca::fma_row<B>(l, p, a);
  for (int k = 0; k < B; ++k) out[k * 64 + threadIdx.x] = l[k];
}
template __global__ void k_probe<8, float>(const float*, float*);
template __global__ void k_probe<10, float>(const float*, float*);
template __global__ void k_probe<8, double>(const double*, double*);
template __global__ void k_probe<10, double>(const double*, double*);
"""


def test_sums_and_factors_in_different_registers(tmp_path):
    src, out = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(SRC)
    subprocess.run([HIPCC, *CXXFLAGS, "--cuda-device-only", "-S", str(src), "-o", str(out)], check=True,
                   capture_output=True, timeout=300)
    seen = re.findall(r"v_fmac_f(?:32|64)_dpp (v\S+), (v\S+), (v\S+) row_newbcast", out.read_text())
    assert len(seen) == 8 + 10 + 8 + 10
    for total, p, a in seen:
        assert total not in (p, a), (total, p, a)
