"""GPU parity of pass B with one input per lane (up to 64 inputs, no multiple of 4):
the window kernel, the stepped combine's runs and the plain combine, at one to 63
inputs, windows inside and past the call, segments that end inside a workgroup. Two
calls on one plan against the oracle, and bit for bit against the scanning path, which
sums in the same order."""
import numpy as np
import pytest

import oracle
from parity import check_result

torch = pytest.importorskip("torch")
sk = pytest.importorskip("paper_1808_10365_amd")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (N, F, M, B, L)
SHAPES = [(1, 1, 4, 9, 3), (2, 3, 8, 65, 130), (3, 1, 4, 700, 64), (5, 2, 8, 33, 5), (7, 1, 16, 1, 9), (63, 4, 4, 40, 300),
          (61, 1, 2, 33000, 16), (5, 1, 2, 33003, 2000), (11, 2, 4, 20, 1), (13, 1, 8, 21, 0)]


@pytest.mark.parametrize("k", range(len(SHAPES)))
def test_small_odd_shapes(k):
    N, F, M, B, L = SHAPES[k]
    print(f"case N={N} F={F} M={M} B={B} L={L}", flush=True)
    rng = np.random.default_rng(9300 + k)
    x = rng.integers(0, 256, size=(2 * M * B, F, N), dtype=np.uint8)
    mask = (rng.random((F, N)) > 0.2).astype(np.uint8) if k % 2 else None
    md = None if mask is None else torch.from_numpy(mask).to(DEV)
    xd = torch.from_numpy(x).to(DEV)
    first = None
    for R, vec in ((0, 0), (2, 0), (0, 1), (4, 1)):
        plan = sk.Plan(N, F, M * B, M, norm_window=L)
        if R or vec:
            plan.set_pass_b_tile(R, vec)
        calls = [plan.compute(xd[c * M * B:(c + 1) * M * B], mask=md, want=sk.ALL_OUTPUTS) for c in range(2)]
        torch.cuda.synchronize()
        state = plan.export_state()
        plan.close()
        out = sk.Result(**{n: torch.cat([getattr(c, n) for c in calls], 1) for n in sk.ALL_OUTPUTS})
        if first is None:
            first, first_state = out, state
            check_result(out, oracle.sk(x, M, L, 0, 5.0, 0.0, 0.0, mask), M, L, what=f"small odd shape {k}")
        assert state == first_state, (R, vec)
        for n in sk.ALL_OUTPUTS:
            a, b = getattr(first, n).cpu().numpy(), getattr(out, n).cpu().numpy()
            assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f"), (R, vec, n)
