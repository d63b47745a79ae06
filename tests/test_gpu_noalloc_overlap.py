"""Calls of sk_compute_noalloc that overlap on two streams share their scratch and
may spoil each other's results, but never a later call's: after many such overlaps,
of calls whose slices meet in different numbers, each call alone equals a plan's
first call bit for bit. The same for calls of one plan (after a reset)."""
import pytest

torch = pytest.importorskip("torch")
sk = pytest.importorskip("paper_1808_10365_amd")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (N, F, M, B, L): two to eight slices of 256 inputs meet.
CALLS = [(2048, 4, 64, 96, 64), (512, 4, 64, 96, 64), (1280, 3, 64, 70, 9)]


def _frames():
    gen = torch.Generator(device=DEV).manual_seed(5)
    return [torch.randint(0, 256, (M * B, F, N), dtype=torch.uint8, device=DEV, generator=gen) for N, F, M, B, L in CALLS]


def _same(a, b):
    return all(torch.equal(torch.nan_to_num(getattr(a, k)), torch.nan_to_num(getattr(b, k))) for k in sk.ALL_OUTPUTS)


def test_overlapping_noalloc_calls_leave_later_ones_right():
    xs = _frames()
    refs, outs = [], []
    for (N, F, M, B, L), x in zip(CALLS, xs):
        plan = sk.Plan(N, F, M * B, M, norm_window=L)
        refs.append(plan.compute(x, want=sk.ALL_OUTPUTS))
        outs.append([plan.alloc_outputs(DEV, sk.ALL_OUTPUTS) for _ in range(3)])
        torch.cuda.synchronize()
        plan.close()
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    for r in range(300):
        for k, s in enumerate(streams):
            c = (r + k) % len(CALLS)
            sk.compute_noalloc(xs[c], outs[c][k], CALLS[c][2], norm_window=CALLS[c][4], stream=s)
    torch.cuda.synchronize()
    for c in (0, 1, 2, 2, 1, 0):
        out = outs[c][2]
        for k in ("v", "significance"):
            getattr(out, k).fill_(-7.0)
        for k in ("flags", "n_eff", "r1", "r2"):
            getattr(out, k).fill_(77)
        sk.compute_noalloc(xs[c], out, CALLS[c][2], norm_window=CALLS[c][4])
        torch.cuda.synchronize()
        assert _same(out, refs[c]), CALLS[c]


def test_overlapping_noalloc_calls_with_windows_of_one_chunk():
    # These use no scratch: every call is right, overlapped or not.
    calls = [(2048, 4, 64, 1024, 4), (501, 4, 64, 520, 3)]
    gen = torch.Generator(device=DEV).manual_seed(6)
    streams = [torch.cuda.Stream() for _ in calls]
    work = []
    for N, F, M, B, L in calls:
        x = torch.randint(0, 256, (M * B, F, N), dtype=torch.uint8, device=DEV, generator=gen)
        plan = sk.Plan(N, F, M * B, M, norm_window=L)
        ref = plan.compute(x, want=sk.ALL_OUTPUTS)
        work.append((x, ref, [plan.alloc_outputs(DEV, sk.ALL_OUTPUTS) for _ in range(8)], M, L))
        torch.cuda.synchronize()
        plan.close()
    for r in range(200):
        for (x, ref, outs, M, L), s in zip(work, streams):
            sk.compute_noalloc(x, outs[r % 8], M, norm_window=L, stream=s)
    torch.cuda.synchronize()
    for x, ref, outs, M, L in work:
        assert all(_same(out, ref) for out in outs), (x.shape, M, L)


def test_overlapping_calls_of_a_plan_leave_it_right():
    xs = _frames()
    streams = [torch.cuda.Stream() for _ in range(2)]
    for (N, F, M, B, L), x in zip(CALLS, xs):
        plan = sk.Plan(N, F, M * B, M, norm_window=L)
        ref = plan.compute(x, want=sk.ALL_OUTPUTS)
        outs = [plan.alloc_outputs(DEV, sk.ALL_OUTPUTS) for _ in range(2)]
        torch.cuda.synchronize()
        for _ in range(300):
            for s, out in zip(streams, outs):
                plan.compute_into(x, out, stream=s)
        torch.cuda.synchronize()
        plan.reset()
        assert _same(plan.compute(x, want=sk.ALL_OUTPUTS), ref), (N, F, M, B, L)
        plan.close()
