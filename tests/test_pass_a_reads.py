"""The bytes pass A's row-phase kernels read, followed on the CPU through the
kernels' own address functions (tests/host/pass_a_reads.cpp): row phases never
leave the frame, and shifted row phases read only aligned dwords that hold a byte
of it, at every count of units per workgroup, whatever the row length, the input's
place within a dword and the rows of a block's last batches."""
import os
import subprocess

import pytest

from paper_1808_10365_amd import _build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def reads(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "pass_a_reads")
    subprocess.run([_build.hipcc(), "-x", "hip", "--offload-host-only", "-O2", "-std=c++17",
                    "-I", os.path.join(_build.ROOT, "include"), "-I", _build.CSRC,
                    os.path.join(HERE, "host", "pass_a_reads.cpp"), "-x", "none", _build.LIB, "-o", exe,
                    "-Wl,-rpath," + os.path.dirname(_build.LIB)], check=True)

    def run(calls):
        text = "\n".join(" ".join(str(v) for v in c) for c in calls)
        res = subprocess.run([exe], input=text, capture_output=True, text=True, check=True)
        return [tuple(int(v) for v in line.split()) for line in res.stdout.splitlines()]
    return run


def _check(calls, got):
    assert len(got) == len(calls)
    bad = []
    for (kind, want, N, F, M, B, at), (lo, hi, lanes) in zip(calls, got):
        size = N * F * M * B
        below = at % 4 if kind == 6 else 0
        above = -(at + size) % 4 if kind == 6 else 0
        if not (-below <= lo and hi < size + above):
            bad.append((kind, lanes, N, F, M, B, at, lo, hi - size + 1))
    assert not bad, bad


# (N, F, M, blocks): rows of odd and even length off 4-byte boundaries; frames that
# fill their pages (3003 x 65536); blocks of one row more and less than whole batches.
SHAPES = [(3003, 1, 256, 256), (3003, 1, 256, 128), (2545, 1, 256, 16), (2545, 1, 100, 512), (602, 1, 128, 64),
          (4095, 1, 64, 16), (2047, 1, 256, 16), (131, 1, 256, 40), (129, 1, 256, 40), (1001, 3, 128, 33),
          (509, 5, 129, 11), (131, 1, 639, 15), (145, 1, 130, 21), (3, 43, 257, 12), (79, 2, 255, 20)]


def test_shifted_reads_stay_in_the_frames_dwords(reads):
    calls = [(6, lanes, N, F, M, B, at) for N, F, M, B in SHAPES for lanes in (16, 32, 64, 128) for at in range(4)]
    # Blocks around whole batches of every count of units (4 rows times 512 / units).
    calls += [(6, lanes, 1021, 1, m + d, 5, 1) for lanes in (16, 32, 64, 128) for m in (2048 // lanes * k for k in range(1, 7))
              for d in (-1, 0, 1)]
    _check(calls, reads(calls))


def test_shifted_reads_of_the_librarys_choice(reads):
    calls = [(6, 0, N, F, M, B, at) for N, F, M, B in
             [(3003, 1, 256, 128), (3003, 1, 256, 256), (2545, 1, 256, 100), (602, 1, 128, 60), (509, 1, 200, 70),
              (2047, 1, 193, 128), (1001, 3, 128, 128), (1021, 1, 64, 2100)] for at in range(4)]
    got = reads(calls)
    assert any(lanes for _, _, lanes in got)
    _check([c for c, g in zip(calls, got) if g[2]], [g for g in got if g[2]])


def test_phased_reads_stay_in_the_frame(reads):
    calls = [(5, lanes, N, F, M, B, at) for N, F, M, B in SHAPES + [(16, 1, 256, 70), (1000, 3, 33, 17), (17, 1, 64, 90)]
             for lanes in (16, 32, 64, 128, 256, 512) for at in (0, 1)]
    _check(calls, reads(calls))
