"""GPU TSDF integration over table sizes: 64 to 512 table slots a block."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import tsdf as T  # noqa: E402
from test_gpu_tsdf import DEV, R, _compare, _frames  # noqa: E402, F401


@pytest.mark.parametrize("log2_blocks", [15, 16, 17, 18, 19])
def test_table_sizes(R, log2_blocks):
    # tables of 2^16 slots are walked 64 slots a block, 2^17 128, 2^18 256, larger ones 512
    m = R.TsdfMap(DEV, max_blocks=1 << log2_blocks)
    ref = T.TsdfMap(voxel=0.01)
    try:
        for k, (cam, depth, _) in enumerate(_frames(3, 80, 60, 2)):
            m.integrate(torch.from_numpy(depth).to(DEV), cam)
            met = ref.integrate(depth, cam)
            inf = m.info()
            assert inf["flags"] == 0 and inf["met_last"] == len(met)
            _compare(m, ref, k + 1, f"2^{log2_blocks} frame {k}")
    finally:
        m.free()
