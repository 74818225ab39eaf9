"""The work items a batch chooses: the size whose most loaded block has least to
march; in FP32, which memory bounds, only for a clear gain over 8192 nodes."""
import pytest

import lbm_inputs as li

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage,count,sizes,items", [
    ("f32", 64, (32, 48), 8192),  # 12288 would promise 2%
    ("f32", 20, (32, 48), 4096),  # 42%
    ("f16s", 64, (32, 48), 16384),  # 9%
    ("f32", 1, (64,), 4096),
    ("f16n", 1, (64,), 4096),
])
def test_default_items(storage, count, sizes, items):
    from paper_1805_08643_amd.binding import Batch
    b = Batch([dict(p, storage=storage, rho_ref=0.17, f16_exp=0) for p, _ in li.c5_batch(count, 1805, sizes)])
    assert b.tuning()[:2] == ("split", items)
    b.close()
