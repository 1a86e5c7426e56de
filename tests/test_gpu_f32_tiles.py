"""The fp32 matrix-core kernels at the edges of their tiles: a workgroup's four waves are the quarters of a 64 x 64 square,
so lengths around 32, 64, 96 and 128 leave waves idle, blocks ragged, or one wave of a pair without anything to add.  With a
large max_len the same batch goes through the scheduler kernel, with a tight one the kernels build their schedule."""
import pytest

from paper_2409_15373_amd.synthetic import make_custom
import test_gpu_causal
import test_gpu_cross
import test_gpu_f32

pytestmark = pytest.mark.gpu
EDGES = [1, 31, 32, 33, 0, 63, 64, 65, 95, 96, 97, 127, 128, 129, 200]


@pytest.mark.parametrize("max_len", [200, 4096])
@pytest.mark.parametrize("D", [32, 64, 128])
def test_self(oracle, D, max_len):
    test_gpu_f32.run_case(oracle, make_custom("edges", EDGES, 1, D, dtype="f32", seed=31 + D, max_len=max_len))


@pytest.mark.parametrize("max_len", [200, 4096])
@pytest.mark.parametrize("D", [32, 64, 128])
def test_causal(D, max_len):
    test_gpu_causal.run(make_custom("edges", EDGES, 1, D, dtype="f32", seed=32 + D), max_len)


@pytest.mark.parametrize("max_len", [200, 4096])
@pytest.mark.parametrize("D", [32, 64, 128])
def test_cross(D, max_len):
    keys = EDGES[4:] + EDGES[:4]
    got, ref, oq, ok = test_gpu_cross.run(EDGES, keys, 1, D, "f32", 33 + D, max_len, max_len)
    test_gpu_cross.compare(got, ref, "f32", oq, ok, EDGES, keys)
