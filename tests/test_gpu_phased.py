"""GPU parity of pass A's row-phase kernel at the sizes where it can go wrong:
each count of 16-byte units per workgroup the library picks (so each number of
row phases), rows that 16 does not divide (the last unit is moved back and its
columns summed twice), units that straddle channels and block ends, rows off a
4-byte boundary, blocks that end inside a batch of rows, and blocks with fewer
rows than phases. The sums are integers, compared bit for bit with the oracle."""
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
    (16, 1, 256, 1500, 16, 0),       # one unit a row
    (17, 4, 64, 256, 32, 0),         # 68-byte rows: a moved-back unit, channels inside units
    (3, 24, 130, 260, 16, 0),        # 72-byte rows, five channels in a unit
    (48, 1, 40, 800, 64, 0),         # three units a row: 21 blocks and a third in a workgroup
    (1004, 3, 33, 100, 64, 0),       # 3012-byte rows, an odd row count
    (1000, 1, 16, 40, 128, 0),       # four rows a lane
    (501, 4, 16, 400, 256, 0),       # two phases
    (1000, 1, 128, 1301, 512, 0),    # one phase: stored from registers
    (64, 1, 1030, 300, 16, 0),       # 8 batches of 128 rows and 6 rows
    (64, 1, 639, 300, 16, 0),        # one row short of five whole batches
    (1024, 2, 32, 200, 128, 0),
    (2047, 1, 193, 470, 256, 0),     # rows off a 4-byte boundary
]


@pytest.mark.parametrize("k", range(len(SHAPES)))
def test_phased_shapes(k):
    N, F, M, B, want, off = SHAPES[k]
    T = M * B
    rng = np.random.default_rng(4200 + k)
    x = rng.integers(0, 256, size=(T, F, N), dtype=np.uint8)
    print(f"case N={N} F={F} M={M} B={B} units={want} offset={off}", flush=True)
    buf = torch.empty(T * F * N + off, dtype=torch.uint8, device=DEV)
    xd = buf[off:].view(T, F, N)
    xd.copy_(torch.from_numpy(x))
    plan = sk.Plan(N, F, T, M, norm_window=3)
    vec, lanes, wgs = ctypes.c_int32(), ctypes.c_int32(), ctypes.c_int64()
    assert sk.load_library().sk_plan_get_pass_a_tile(plan.handle, ctypes.c_void_p(xd.data_ptr()), ctypes.byref(vec),
                                                     ctypes.byref(lanes), ctypes.byref(wgs)) == 0
    assert (vec.value, lanes.value) == (16, want)
    assert wgs.value == (B * ((F * N + 15) // 16) + want - 1) // want
    out = plan.compute(xd, want=sk.ALL_OUTPUTS)
    torch.cuda.synchronize()
    check_result(out, oracle.sk(x, M, 3), M, 3, what=f"phased shape {k}")
    plan.close()
