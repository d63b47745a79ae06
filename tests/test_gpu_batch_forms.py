"""The forms a batch's calls take (the classes' picks; pass A in row phases with
one pass B chunk length), each forced through the tuning cache: every problem's
outputs equal its own plan's bit for bit over two calls, at every count of units
per row-phase task (16 to 64 units, and 512 of whole short blocks), at rows that
end inside a task, and odd block lengths."""
import json

import numpy as np
import pytest

torch = pytest.importorskip("torch")
sk = pytest.importorskip("paper_1808_10365_amd")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (N, F, M, B, L)
SMALL = [(16, 1, 256, 5, 4), (64, 8, 1024, 3, 2), (1024, 4, 64, 40, 64), (2048, 1, 16, 9, 0), (48, 5, 300, 17, 7),
         (256, 3, 2, 33, 5), (2064, 1, 33, 12, 1)]
# Enough bytes for 64 units at M = 256 and 512 units at M = 16.
LARGE = [(1024, 4, 256, 260, 16), (512, 3, 16, 1200, 3), (2048, 1, 1024, 9, 8), (176, 1, 130, 77, 300)]


@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("which", ["small", "large"])
@pytest.mark.parametrize("autotune", [True, False])
def test_batch_forms_equal_plans(which, form, autotune, tmp_path):
    if not autotune and form:
        pytest.skip("without the autotuner the library picks the form")
    probs = SMALL if which == "small" else LARGE
    arch = torch.cuda.get_device_properties(0).gcnArchName
    total = sum(N * F * M * B for N, F, M, B, _ in probs)
    cache = tmp_path / "tune.json"
    cache.write_text(json.dumps({f"{arch}|batch|set|n={len(probs)}|bytes={total}|form": form}))
    print(f"case {which} form={form} autotune={autotune} bytes={total}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(17 + form)
    frames = [[torch.randint(0, 256, (M * B, F, N), dtype=torch.uint8, device=DEV, generator=gen)
               for N, F, M, B, _ in probs] for _ in range(2)]
    kws = [dict(n_inputs=N, n_channels=F, n_samples=M * B, block_len=M, norm_window=L, k_sigma=4.0)
           for N, F, M, B, L in probs]
    batch = sk.Batch(kws, frames[0], autotune=autotune, tune_cache=str(cache), want=sk.ALL_OUTPUTS)
    plans = [sk.Plan(**kw) for kw in kws]
    for c in range(2):
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


@pytest.mark.parametrize("M", [1023, 1024, 2047, 2048])
def test_largest_sums_of_a_wavefront(M):
    # Every sample at power 128: S2 of 256 inputs reaches 2^22 M, past 32 bits
    # from M = 1024 on; below M = 2048 the wavefront sum widens at its last step.
    for N, L in ((256, 2), (2048, 2), (2048, 0)):
        x = torch.zeros((2 * M, 1, N), dtype=torch.uint8, device=DEV)
        plan = sk.Plan(N, 1, 2 * M, M, norm_window=L)
        out = plan.compute(x)
        torch.cuda.synchronize()
        assert out.r1.flatten().tolist() == [128 * M * N] * 2
        assert out.r2.flatten().tolist() == [128 * 128 * M * N] * 2
        plan.close()
