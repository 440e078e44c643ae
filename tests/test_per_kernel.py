"""What the library keeps once per kernel (csrc/per_kernel.h), compiled with g++."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2503_22673_amd", "csrc")
SOURCE = r"""
#include "per_kernel.h"
template <int H> void kernel(int) {}
template <int H> std::atomic<uint64_t>* mask() { return &smem_devices<kernel<H>>; }
int main() {
  constexpr auto k = kernel<4>;
  %s
  smem_devices<kernel<4>>.fetch_or(1);
  return mask<4>() == &smem_devices<k> && mask<4>()->load() == 1 && mask<2>()->load() == 0 && mask<1>()->load() == 0 && mask<1>() != mask<2>() ? 0 : 1;
}
"""


@pytest.mark.parametrize("line, compiles", [("", True), ("auto v = kernel<2>; (void)&smem_devices<v>;", False)])
def test_kernels_of_one_signature_have_masks_of_their_own(tmp_path, line, compiles):
    """A kernel that is only known at run time, as inside a generic lambda that several pass through, is refused by the compiler."""
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(SOURCE % line)
    r = subprocess.run(["g++", "-std=c++17", "-I" + CSRC, str(src), "-o", str(exe)], capture_output=True, text=True)
    assert (r.returncode == 0) == compiles, r.stderr
    if compiles:
        assert subprocess.run([str(exe)]).returncode == 0
