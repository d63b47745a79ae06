"""GPU parity of pass A's shifted row phases (rows off 4-byte boundaries) at the
sizes where it can go wrong: each count of units per workgroup the library picks,
rows that end one to fifteen columns into their last unit (where a further unit
holds what shifted windows have left, or nothing), rows that keep to 4 bytes in an
input that does not, channels inside units, units over block ends, and blocks that
end inside a batch of rows. The sums are integers, compared bit for bit with the
oracle; no byte next to the input decides a result (it lies between bytes of
power)."""
import ctypes

import numpy as np
import pytest

import oracle
from parity import check_result

torch = pytest.importorskip("torch")
sk = pytest.importorskip("paper_1808_10365_amd")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (N, F, M, blocks, units per workgroup, input offset in bytes)
SHAPES = [
    (509, 1, 200, 70, 16, 0),        # 13 columns in the last unit
    (79, 2, 256, 200, 16, 0),        # 14: one more unit for windows that start before it
    (159, 1, 1000, 100, 16, 2),      # 15
    (145, 1, 130, 210, 16, 0),       # 1
    (3, 43, 256, 120, 16, 0),        # 129-byte rows, six channels in a unit
    (131, 1, 639, 150, 16, 0),       # one row short of five whole batches
    (512, 1, 256, 33, 16, 1),        # whole units, an input off its boundary
    (512, 1, 256, 33, 16, 3),
    (2047, 1, 193, 128, 32, 0),
    (509, 5, 129, 101, 64, 0),
    (1001, 3, 128, 128, 128, 0),
    (1021, 1, 64, 2100, 128, 0),     # short blocks
]


@pytest.mark.parametrize("k", range(len(SHAPES)))
def test_shifted_shapes(k):
    N, F, M, B, want, off = SHAPES[k]
    T = M * B
    rng = np.random.default_rng(7300 + k)
    x = rng.integers(0, 256, size=(T, F, N), dtype=np.uint8)
    print(f"case N={N} F={F} M={M} B={B} units={want} offset={off}", flush=True)
    buf = torch.full((T * F * N + off + 16,), 0x0F, dtype=torch.uint8, device=DEV)
    xd = buf[off:off + T * F * N].view(T, F, N)
    xd.copy_(torch.from_numpy(x))
    plan = sk.Plan(N, F, T, M, norm_window=3)
    vec, lanes, wgs = ctypes.c_int32(), ctypes.c_int32(), ctypes.c_int64()
    assert sk.load_library().sk_plan_get_pass_a_tile(plan.handle, ctypes.c_void_p(xd.data_ptr()), ctypes.byref(vec),
                                                     ctypes.byref(lanes), ctypes.byref(wgs)) == 0
    assert (vec.value, lanes.value) == (16, want)
    assert wgs.value == (B * ((F * N + 18) // 16) + want - 2) // (want - 1)
    out = plan.compute(xd, want=sk.ALL_OUTPUTS)
    torch.cuda.synchronize()
    check_result(out, oracle.sk(x, M, 3), M, 3, what=f"shifted shape {k}")
    plan.close()
