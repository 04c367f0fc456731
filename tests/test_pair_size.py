"""A Riccati step at d >= 32 keeps notes of its split products behind the pair it works on in LDS.  A pair without room for them
has to be refused by the compiler: the writes past its end would land in whatever the layout puts there, without an error."""
import os
import subprocess

import pytest

from paper_2603_09221_amd import build

KERNEL = """
#include "ttc_tv.hpp"
namespace ttc {
__global__ void __launch_bounds__(Cfg<%(d)d>::NTHR) step_kernel(const float* A, const float* B, const float* R, float* out) {
  using C = Cfg<%(d)d>;
  __shared__ __attribute__((aligned(16))) float W[%(size)s];
  Cols<%(d)d> wk, pn;
  out[threadIdx.x] = riccati_step<%(d)d, float>(W, A, B, R, wk, pn, threadIdx.x);
}
}  // namespace ttc
"""


def _accepted(tmp_path, d, size):
    src = os.path.join(tmp_path, "step.hip")
    with open(src, "w") as f:
        f.write(KERNEL % dict(d=d, size=size))
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + build.HIPCC_FLAGS
    cmd += ["-fsyntax-only", "-I", build.CSRC, "-I", build.INCLUDE, src]
    return subprocess.run(cmd, capture_output=True, text=True).returncode == 0


@pytest.mark.parametrize("d", [32, 64, 128])
def test_a_pair_without_room_for_the_notes_is_refused(tmp_path, d):
    assert _accepted(tmp_path, d, "C::PAIR")
    assert not _accepted(tmp_path, d, "%d * C::PITCH" % d)
