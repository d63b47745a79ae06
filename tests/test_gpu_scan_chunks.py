"""GPU parity of the plans' prefix scans: both kernels at each chunk length, calls of
one round of the scan, one row more and less, and several rounds; one input per lane,
so that no call is summed directly; windows inside the call, longer than it (older
history moves on) and of whole runs; two calls each. Chunk lengths do not change a
result: bit for bit between them, and against the oracle."""
import numpy as np
import pytest

import oracle
from parity import check_result

torch = pytest.importorskip("torch")
sk = pytest.importorskip("paper_1808_10365_amd")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (N, F, M, B, L); 16384 inputs: more workgroups than CUs
SHAPES = [(2, 1, 8, 1023, 100), (3, 2, 4, 1025, 7), (65, 1, 4, 2049, 2100), (70, 3, 2, 37, 300), (129, 1, 4, 1024, 64),
          (16384, 1, 2, 20, 33)]


@pytest.mark.parametrize("k", range(len(SHAPES)))
def test_scans(k):
    N, F, M, B, L = SHAPES[k]
    print(f"case N={N} F={F} M={M} B={B} L={L}", flush=True)
    x = np.random.default_rng(8100 + k).integers(0, 256, size=(2 * M * B, F, N), dtype=np.uint8)
    ref = oracle.sk(x, M, L)
    xd = torch.from_numpy(x).to(DEV)
    first = None
    for R in (1, 2, 4):
        plan = sk.Plan(N, F, M * B, M, norm_window=L)
        plan.set_pass_b_tile(R, 1)
        calls = [plan.compute(xd[c * M * B:(c + 1) * M * B], want=sk.ALL_OUTPUTS) for c in range(2)]
        torch.cuda.synchronize()
        out = sk.Result(**{n: torch.cat([getattr(c, n) for c in calls], 1) for n in sk.ALL_OUTPUTS})
        plan.close()
        if first is None:
            first = out
            check_result(out, ref, M, L, what=f"scan shape {k} R={R}")
        for n in sk.ALL_OUTPUTS:
            a, b = getattr(first, n).cpu().numpy(), getattr(out, n).cpu().numpy()
            assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f"), (R, n)
