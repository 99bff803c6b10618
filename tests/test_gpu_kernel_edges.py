"""GPU parity at the sizes where a kernel or a dispatch rule changes its path: edges of tiles, remainders, the smallest
calls.  Reference: the fp64 oracle's unsplit attention; tolerances: tests/parity.py (per data type)."""
import pytest

from tests import parity as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("lens,C,Hq,Hkv,scale", [
    ([1], 8, 1, 1, None),                                  # one row, one key
    ([15, 16, 17, 1, 2], 64, 3, 1, None),                  # around the 16-row block
    ([255, 256, 257, 270], 300, 2, 2, None),               # 16 blocks: one per wavefront; then a second round
    ([530], 100, 4, 2, None),                              # slices whose prefix is no multiple of 16
    ([70, 40], 32, 2, 1, -0.125), ([70, 40], 32, 2, 1, 0.0),   # any scale
])
def test_fp32_blocks(D, lens, C, Hq, Hkv, scale):
    got, _ = P.run_gpu(lens, C, Hq, Hkv, D, "fp32", seed=31, scale=scale)
    ref = P.run_oracle(lens, Hq, Hkv, D, "fp32", seed=31, scale=scale)
    P.check(got, ref, "fp32", f"lens={lens} C={C} D={D} scale={scale}")
