"""GPU parity of the window kernel (pass B without the prefix scan) at the sizes
where it can go wrong: one to eight slices of 256 inputs and more groups than
slices, last groups of one to three inputs, segments that end inside a
workgroup, windows shorter and longer than a segment and than the call (older
history carried on), masked and dead inputs, and calls on either side of the
line to the scan. Each runs three calls on one plan against the oracle, and the
carried state equals that of the one-input-per-lane path, which scans."""
from types import SimpleNamespace

import numpy as np
import pytest

import oracle
from parity import check_result

torch = pytest.importorskip("torch")
sk = pytest.importorskip("paper_1808_10365_amd")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (N, F, blocks per call, L)
SHAPES = [
    (4, 1, 7, 2), (5, 2, 20, 5), (7, 1, 9, 30),
    (255, 2, 33, 9), (256, 4, 192, 256), (257, 3, 33, 33), (258, 1, 8, 3),
    (509, 5, 65, 7), (1000, 3, 70, 16), (2047, 1, 100, 64), (2048, 1, 1, 30),
    (2049, 1, 40, 9), (4100, 1, 17, 40),
    (2048, 2, 128, 128), (2048, 2, 130, 400),      # just below the line, and above it (scan)
    (64, 1, 600, 300),
]


@pytest.mark.parametrize("R", [0, 1, 2, 4])
@pytest.mark.parametrize("k", range(len(SHAPES)))
def test_window_shapes(k, R):
    N, F, B, L = SHAPES[k]
    M, calls = 8, 3
    T = M * B
    rng = np.random.default_rng(5100 + k)
    x = rng.integers(0, 256, size=(calls * T, F, N), dtype=np.uint8)
    x[T // 2:, :, N // 2] = 0x88
    mask = (rng.random((F, N)) > 0.1).astype(np.uint8) if k % 2 else None
    print(f"case N={N} F={F} B={B} L={L} R={R}", flush=True)
    md = None if mask is None else torch.from_numpy(mask).to(DEV)
    plan, scan = sk.Plan(N, F, T, M, norm_window=L), sk.Plan(N, F, T, M, norm_window=L)
    if R:
        plan.set_pass_b_tile(R, 0)
    scan.set_pass_b_tile(0, 1)
    outs = []
    for c in range(calls):
        xd = torch.from_numpy(np.ascontiguousarray(x[c * T:(c + 1) * T])).to(DEV)
        outs.append(plan.compute(xd, mask=md, want=sk.ALL_OUTPUTS))
        scan.compute(xd, mask=md)
        torch.cuda.synchronize()
        assert plan.export_state() == scan.export_state(), c
    got = SimpleNamespace(**{n: torch.cat([getattr(o, n) for o in outs], dim=1) for n in sk.ALL_OUTPUTS})
    check_result(got, oracle.sk(x, M, L, 0, 5.0, 0.0, 0.0, mask), M, L, what=f"window shape {k} R={R}")
    # The entry point without a plan: the first call, bit for bit.
    out = plan.alloc_outputs(DEV, sk.ALL_OUTPUTS)
    sk.compute_noalloc(torch.from_numpy(np.ascontiguousarray(x[:T])).to(DEV), out, M, norm_window=L, mask=md)
    torch.cuda.synchronize()
    for n in sk.ALL_OUTPUTS:
        a, b = getattr(out, n).cpu().numpy(), getattr(outs[0], n).cpu().numpy()
        assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f"), n
    plan.close()
    scan.close()
