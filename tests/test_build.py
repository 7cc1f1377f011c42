"""The build reads the compiler's register figures and refuses kernels that
spill vector registers (no GPU needed)."""
import os

import pytest

from paper_2201_01556_amd import build

# a kernel that keeps %(values)d values per thread; 1,024 threads have 128 registers
KERNEL = r"""
#include <hip/hip_runtime.h>
namespace hf {
__global__ void __launch_bounds__(1024) k_sum(const float* x, float* y) {
  float v[%(values)d];
#pragma unroll
  for (int i = 0; i < %(values)d; ++i) v[i] = x[i * 1024 + threadIdx.x];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < %(values)d; ++i)
    y[i * 1024 + threadIdx.x] = v[i] * v[%(values)d - 1 - i];
}
}  // namespace hf
"""


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="hipcc not available")
@pytest.mark.parametrize("values,spills", [(32, False), (300, True)])
def test_spilled_vector_registers_are_refused(tmp_path, values, spills):
    src, obj = tmp_path / "k.hip", tmp_path / "k.o"
    src.write_text(KERNEL % {"values": values})
    if spills:
        with pytest.raises(RuntimeError, match="k_sum"):
            build.compile_source(str(src), str(obj))
    else:
        build.compile_source(str(src), str(obj))
    assert obj.exists() != spills


def test_spills_are_read_from_the_remarks():
    remark = ("k.hip:1:1: remark: Function Name: {0} [-Rpass-analysis=kernel-resource-usage]\n"
              "k.hip:1:1: remark:     SGPRs Spill: 9 [-Rpass-analysis=kernel-resource-usage]\n"
              "k.hip:1:1: remark:     VGPRs Spill: {1} [-Rpass-analysis=kernel-resource-usage]\n")
    text = remark.format("_ZN2hf3k_aEv", 0) + remark.format("_ZN2hf3k_bEv", 13)
    text += remark.format("_ZN7rocprim1kEv", 4)  # a library header's
    assert build.register_spills(text) == {"_ZN2hf3k_aEv": 0, "_ZN2hf3k_bEv": 13}
