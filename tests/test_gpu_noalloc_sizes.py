"""The caller-link measurement on either side of its lines: links lane by lane
up to 256 tiles of 64 sites and through LDS above, sums by 256 threads up to
1024 partial slots (341 tiles) and by 1024 above, tiles filled and ragged.  All
give bit for bit what tgf_measure gives on a context that holds the links."""

import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2107_03747_amd import gen, tgf          # noqa: E402


@pytest.mark.parametrize("dims,tiles", [((2, 2, 2, 2), 1), ((8, 8, 16, 16), 256), ((5, 5, 25, 27), 264),
                                        ((7, 7, 21, 21), 338), ((8, 8, 11, 31), 341),
                                        ((8, 8, 18, 19), 342), ((9, 9, 27, 27), 923)])
def test_caller_links_measured_as_stored_ones(dims, tiles):
    twist = (1, 2, 1, 2, 1, 2)
    assert (int(np.prod(dims)) + 63) // 64 == tiles
    U = gen.haar(dims, seed=tiles, device="cuda")
    f = tgf.Flow([(dims, twist)], "f64")
    f.load(0, U)
    ref = f.measure()[0]
    out = torch.full((6,), float("nan"), dtype=torch.float64, device="cuda")
    s = torch.cuda.current_stream()
    tgf.check(tgf.tgf_measure_noalloc(tgf.make_geoms([(dims, twist)]), ctypes.c_void_p(U.data_ptr()),
                                      0.0, ctypes.c_void_p(out.data_ptr()),
                                      ctypes.c_void_p(s.cuda_stream)))
    torch.cuda.synchronize()
    print(f"  {dims} ({tiles} tiles): {ref}", flush=True)
    assert np.array_equal(out.cpu().numpy(), ref)
