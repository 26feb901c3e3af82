"""Sizes that two kernels have to agree on, checked by the compiler (no device code is generated)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2106_03452_amd", "csrc")


def _compiles(tmp_path, source, *flags):
    src = tmp_path / "check.hip"
    src.write_text(source)
    got = subprocess.run([shutil.which("hipcc") or "/opt/rocm/bin/hipcc", "--offload-arch=gfx950", "-std=c++17",
                          "-fsyntax-only", "-Wno-unused-command-line-argument", *flags, "-I", os.path.join(ROOT, "include"),
                          "-I", CSRC, str(src)], capture_output=True, text=True, timeout=300)
    assert got.returncode == 0, got.stderr[-3000:]


@pytest.mark.parametrize("split", [32, 64, 128, 256])
def test_backward_sums_are_read_as_they_are_written(tmp_path, split):
    """A single backward at 32 to 128 leaves one FP64 sum of G per plane and chunk
    of its rows, and the next pass adds them: also where the planes are split."""
    _compiles(tmp_path, """#include "psr_kernels.hip"
using namespace psr;
template <int R> constexpr bool agree() {
  using P = Plane<R, plane_threads(1)>;
  return plane_sums(R) == R * P::NCHUNK && P::NCHUNK * P::RC == R && P::KP == plane_parts(R);
}
static_assert(agree<32>() && agree<64>() && agree<128>());
""", f"-DPSR_PLANE_SPLIT_MIN={split}")


def test_small_cloud_sort_takes_what_it_can_hold(tmp_path):
    """The clouds that get the coarse cells are those the two-launch sort takes:
    16-bit keys, counts and positions, and a pair of keys per thread and turn."""
    _compiles(tmp_path, """#include "psr_opt.hip"
using namespace psr::opt;
static_assert(kNnSmall <= 65535 && kNnSmall == 2 * 1024 * kNnSortPairs && kNnFineCells <= 65535);
static_assert(kNnOne % 1024 == 0 && kNnOne <= kNnSmall && nn_one(kNnOne, kNnOne));
static_assert(nn_cell_bits(kNnOne, kNnOne) == kNnSmallBits && !nn_one(kNnOne + 1, 1) && !nn_one(1, kNnOne + 1));
static_assert(nn_cell_bits(kNnSmall, 1) == kNnSmallBits && nn_cell_bits(1, kNnSmall) == kNnSmallBits);
static_assert(nn_cell_bits(kNnSmall + 1, 1) > kNnSmallBits && nn_cell_bits(1, kNnSmall + 1) > kNnSmallBits);
static_assert(nn_small(kNnSmall, 1) && nn_small(1, kNnSmall) && !nn_small(kNnSmall + 1, 1) && !nn_small(1, kNnSmall + 1));
""")
