"""The batch's prefix scan with walkers of 32 inputs and only the read prefix rows
written: enough blocks that the stepped combine takes 16 at a time, calls of whole
rounds of rows, one row more and one less, windows that are and are not whole runs of
16 blocks, input counts that end inside a slice, and a call shorter than its window.
Every problem's outputs equal its own plan's bit for bit over three calls, in each
form of the batch."""
import json

import numpy as np
import pytest

torch = pytest.importorskip("torch")
sk = pytest.importorskip("paper_1808_10365_amd")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (N, F, M, B, L)
PROBS = [(1024, 8, 2, 1030, 1024), (96, 2, 2, 512, 64), (48, 1, 4, 1500, 48), (16, 3, 2, 2000, 50), (80, 2, 2, 513, 512),
         (2048, 1, 2, 511, 500), (112, 1, 2, 300, 4096), (64, 4, 2, 1024, 1025)]


@pytest.mark.parametrize("form", [0, 1])
def test_batch_scan_equals_plans(form, tmp_path):
    arch = torch.cuda.get_device_properties(0).gcnArchName
    total = sum(N * F * M * B for N, F, M, B, _ in PROBS)
    cache = tmp_path / "tune.json"
    cache.write_text(json.dumps({f"{arch}|batch|set|n={len(PROBS)}|bytes={total}|form": form}))
    print(f"case form={form} bytes={total}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(31 + form)
    frames = [[torch.randint(0, 256, (M * B, F, N), dtype=torch.uint8, device=DEV, generator=gen)
               for N, F, M, B, _ in PROBS] for _ in range(3)]
    kws = [dict(n_inputs=N, n_channels=F, n_samples=M * B, block_len=M, norm_window=L) for N, F, M, B, L in PROBS]
    batch = sk.Batch(kws, frames[0], autotune=True, tune_cache=str(cache), want=sk.ALL_OUTPUTS)
    plans = [sk.Plan(**kw) for kw in kws]
    for c in range(3):
        outs = batch.compute(frames[c])
        torch.cuda.synchronize()
        for j, (plan, x) in enumerate(zip(plans, frames[c])):
            ref = plan.compute(x, want=sk.ALL_OUTPUTS)
            torch.cuda.synchronize()
            for k in sk.ALL_OUTPUTS:
                a, b = getattr(outs[j], k).cpu().numpy(), getattr(ref, k).cpu().numpy()
                assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f"), (c, j, k)
    batch.close()
    for plan in plans:
        plan.close()
