"""GPU parity of the stepped combine (pass B with prefix sums, up to 16 blocks
per wavefront) at the sizes where it can go wrong: one to eight groups of 256
inputs, last groups of one to three inputs, runs cut off by the end of the call
inside a chunk and between chunks, one chunk per run and 16 blocks per run,
windows that end inside a run and windows longer than the call (history values,
older history carried on), 32- and 64-bit wavefront sums, masked and dead inputs.
Each runs two calls on one plan against the oracle, and the integers and the
carried state equal those of the one-input-per-lane path, which takes one chunk
per wavefront."""
from types import SimpleNamespace

import numpy as np
import pytest

import oracle
from parity import check_result

torch = pytest.importorskip("torch")
sk = pytest.importorskip("paper_1808_10365_amd")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (N, F, blocks per call, L, M)
SHAPES = [
    (2048, 2, 520, 300, 2), (2047, 2, 203, 2000, 2), (300, 8, 1025, 997, 2), (1000, 3, 701, 603, 2),   # one chunk a run
    (2048, 4, 1024, 256, 2), (257, 8, 2051, 500, 2), (64, 8, 4099, 700, 2), (1021, 3, 2735, 5000, 2),  # 16 blocks a run
    (4, 1, 3001, 3000, 2048),                                                                         # 64-bit sums
]


@pytest.mark.parametrize("R", [0, 1, 2, 4])
@pytest.mark.parametrize("k", range(len(SHAPES)))
def test_stepped_shapes(k, R):
    N, F, B, L, M = SHAPES[k]
    calls = 2
    T = M * B
    rng = np.random.default_rng(6200 + k)
    x = rng.integers(0, 256, size=(calls * T, F, N), dtype=np.uint8)
    x[T // 2:, :, N // 2] = 0x88
    mask = (rng.random((F, N)) > 0.1).astype(np.uint8) if k % 2 else None
    print(f"case N={N} F={F} B={B} L={L} M={M} R={R}", flush=True)
    md = None if mask is None else torch.from_numpy(mask).to(DEV)
    plan, one = sk.Plan(N, F, T, M, norm_window=L), sk.Plan(N, F, T, M, norm_window=L)
    if R:
        plan.set_pass_b_tile(R, 0)
    one.set_pass_b_tile(0, 1)
    outs = []
    for c in range(calls):
        xd = torch.from_numpy(np.ascontiguousarray(x[c * T:(c + 1) * T])).to(DEV)
        outs.append(plan.compute(xd, mask=md, want=sk.ALL_OUTPUTS))
        ref = one.compute(xd, mask=md, want=sk.ALL_OUTPUTS)
        torch.cuda.synchronize()
        assert plan.export_state() == one.export_state(), c
        for n in ("s1", "s2", "r1", "r2", "n_eff"):
            assert torch.equal(getattr(outs[-1], n), getattr(ref, n)), (n, c)
    got = SimpleNamespace(**{n: torch.cat([getattr(o, n) for o in outs], dim=1) for n in sk.ALL_OUTPUTS})
    check_result(got, oracle.sk(x, M, L, 0, 5.0, 0.0, 0.0, mask), M, L, what=f"stepped shape {k} R={R}")
    plan.close()
    one.close()
