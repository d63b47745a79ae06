"""What the library allocates and launches, on the CPU (the fake HIP runtime of
tests/host): properties of the host code that need no kernel to run."""
from host_dispatch import dispatch  # noqa: F401


def test_plan_creation_clears_nothing_and_waits_for_nothing(dispatch):
    # Creating a plan (a server adds arrays while frames run) touches no stream.
    out = dispatch("""
        for N, F, M, B, L in [(16, 1, 256, 16, 4), (2048, 4, 256, 192, 256), (512, 1, 64, 9, 2), (1000, 3, 256, 128, 16)]:
            rc, h = plan(N, F, M, B, L)
            assert rc == 0, sk.sk_last_error()
            print([line for line in log() if not line.startswith("malloc")])
        """)
    assert out.split() == ["[]"] * 4
