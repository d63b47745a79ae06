"""The form of a batch's calls is cached by the batch's shapes: batches of as many
problems and bytes but other shapes are timed by themselves, the same shapes in another
order are not timed again, and a pick cached for any such batch is still obeyed."""
import json

import pytest

torch = pytest.importorskip("torch")
sk = pytest.importorskip("paper_1808_10365_amd")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

WIDE = [(1024, 2, 64, 8, 4), (512, 2, 64, 16, 4)]
NARROW = [(16, 4, 1024, 16, 4), (64, 1, 512, 32, 4)]


def _create(probs, cache):
    xs = [torch.zeros((M * B, F, N), dtype=torch.uint8, device=DEV) for N, F, M, B, _ in probs]
    kws = [dict(n_inputs=N, n_channels=F, n_samples=M * B, block_len=M, norm_window=L) for N, F, M, B, L in probs]
    sk.Batch(kws, xs, autotune=True, tune_cache=str(cache)).close()
    return {k: v for k, v in json.loads(cache.read_text()).items() if k.endswith("|form")}


def test_form_is_cached_by_shapes(tmp_path):
    assert sum(n * f * m * b for n, f, m, b, _ in WIDE) == sum(n * f * m * b for n, f, m, b, _ in NARROW)
    cache = tmp_path / "tune.json"
    first = _create(WIDE, cache)
    assert len(first) == 1
    assert _create(WIDE[::-1], cache) == first
    both = _create(NARROW, cache)
    assert len(both) == 2 and first.items() <= both.items()


def test_form_of_any_batch_is_obeyed(tmp_path):
    cache = tmp_path / "tune.json"
    arch = torch.cuda.get_device_properties(0).gcnArchName
    total = sum(n * f * m * b for n, f, m, b, _ in WIDE)
    cache.write_text(json.dumps({f"{arch}|batch|set|n={len(WIDE)}|bytes={total}|form": 0}))
    assert len(_create(WIDE, cache)) == 1
