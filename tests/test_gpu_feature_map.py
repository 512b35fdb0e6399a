"""Feature map at the edges of its tiles: D on both sides of 256 (workgroups of
32 rows x 256 features, above it 16 rows x 512) and of 512, d at its largest,
rows around a multiple of 16, degrees above 3.  A feature is a product of a
rounded weight and at most P - 1 <= 4 coordinates: relative error at most
(1 + 4) 2^-24 = 3e-7 in float32 against the float64 oracle.
"""
import ctypes
import sys

import numpy as np
import pytest

import oracle
import sata_synth as syn
from gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("rows", [1, 16, 33])
@pytest.mark.parametrize("d,P,dtype", [(255, 2, "bf16"), (21, 3, "f32"), (22, 3, "bf16"), (30, 3, "f32"),
                                       (31, 3, "bf16"), (255, 3, "f32"), (8, 5, "bf16"), (13, 5, "f32")])
def test_feature_map_tile_edges(d, P, rows, dtype):
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2602_00294_amd as sata
    print(f"feature_map d={d} P={P} rows={rows} {dtype}", file=sys.stderr, flush=True)
    D = oracle.feature_count(d, P)
    x = syn.head_stream(103, d, P, 0, (rows, d), dtype)
    xd = to_dev(x, dtype)
    buf = torch.full((rows * D + 2,), -7.0, device="cuda")
    st = sata.load_library().sata_feature_map(
        ctypes.c_void_p(xd.data_ptr()), int(dtype == "bf16"), rows, d, P, ctypes.c_void_p(buf.data_ptr() + 4),
        ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == 0
    got = to_host(buf)
    assert got[0] == -7.0 and got[-1] == -7.0
    np.testing.assert_allclose(got[1:-1].reshape(rows, D), oracle.phi_ref(x, P), rtol=5 * 2.0 ** -24, atol=1e-30)
