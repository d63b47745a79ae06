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


def test_noalloc_windows_of_one_chunk_use_no_scratch(dispatch):
    # The combine alone: no prefix sums, no sums of slices, so such calls may overlap.
    out = dispatch("""
        o = outs()
        for N, F, M, B, L in [(2048, 4, 64, 1024, 2), (2048, 4, 64, 1024, 4), (512, 8, 64, 1024, 4), (1000, 4, 64, 512, 2),
                              (501, 4, 64, 512, 4), (257, 4, 64, 1024, 3), (8192, 1, 64, 1100, 2)]:
            d = desc(N, F, M, B, L)
            assert sk.sk_compute_noalloc(ctypes.byref(d), X, None, ctypes.byref(o), None) == 0, sk.sk_last_error()
            names = launches()
            assert "pass_a" in names[0]
            print(" ".join(names[1:]))
        """)
    assert len(out.splitlines()) == 7
    for line in out.splitlines():
        assert len(line.split()) == 1 and "combine_kernel" in line, line


def test_routes_of_plans_with_a_window(dispatch):
    # Each call takes the kernels that serve its sizes best (measured, in the rules'
    # comments): N, F, M, B, L and what must, and must not, be among pass B's kernels.
    calls = [(2048, 4, 16, 4096, 256, "step_kernel", "window"), (2048, 4, 16, 4096, 100, "scan_chunks", "step"),
             (2048, 4, 16, 4096, 8, "scan_chunks", "window"), (2048, 4, 16, 4096, 2, "combine", "scan"),
             (1024, 8, 32, 2048, 100, "scan_chunks", "step"), (2048, 4, 64, 1000, 100, "scan_chunks", "window"),
             (3000, 4, 32, 1100, 100, "scan_chunks", "window"), (4096, 4, 32, 1024, 100, "scan_chunks", "window"),
             (64, 8, 64, 4096, 2, "combine", "window"), (256, 8, 64, 2048, 3, "combine", "window"),
             (2048, 1, 64, 2048, 20, "window", "scan"), (1024, 4, 64, 512, 64, "window", "scan"),
             (256, 4, 256, 192, 256, "window", "scan"), (2048, 4, 256, 1024, 256, "step_kernel", "chunks"),
             # Rows off 16-byte boundaries.
             (301, 8, 4, 20000, 100, "step_kernel", "chunks"), (2047, 4, 16, 2100, 7, "window", "scan"),
             (190, 1, 4, 8000, 3, "window", "combine"), (301, 1, 4, 8000, 3, "combine", "window")]
    out = dispatch(f"""
        o = outs()
        for N, F, M, B, L, has, no in {calls!r}:
            rc, h = plan(N, F, M, B, L)
            assert rc == 0, sk.sk_last_error()
            log()
            assert sk.sk_compute(h, X, None, ctypes.byref(o), None) == 0, sk.sk_last_error()
            names = " ".join(launches()[1:])
            if has not in names or no in names:
                print(N, F, M, B, L, names)
        """)
    assert out == ""


def test_routes_of_pass_a(dispatch):
    # Row phases only where they are the faster (measured, in the rule's comment): N, F,
    # M, B, the input's place in 16 bytes, and units per workgroup (0: another variant).
    calls = [(2, 8, 1695, 1800, 0, 0), (16, 1, 1700, 1102, 0, 0), (16, 1, 640, 29296, 8, 0), (16, 1, 80, 23437, 8, 0),
             (50, 4, 24, 6250, 0, 0), (104, 1, 200, 14423, 0, 0), (8, 8, 256, 7934, 4, 0), (300, 2, 33, 3535, 0, 0),
             (39, 3, 128, 20905, 0, 0), (123, 1, 392, 3209, 0, 0), (104, 1, 24, 801, 0, 0), (48, 1, 40, 52083, 0, 0), (400, 4, 34, 4183, 0, 256), (16, 1, 1024, 6739, 0, 16),
             (4, 8, 40, 101562, 0, 32), (104, 1, 40, 37500, 0, 512), (88, 4, 128, 6658, 4, 64), (104, 1, 128, 2253, 0, 32),
             (256, 4, 256, 192, 0, 16), (1000, 3, 256, 128, 0, 128), (16, 1, 128, 60000, 0, 16),
             # Rows of dwords off 16-byte boundaries.
             (50, 4, 40, 37500, 0, 0), (8, 4, 1024, 12206, 8, 0), (8, 4, 128, 48828, 8, 16), (16, 4, 140, 3348, 8, 0), (20, 4, 140, 17857, 4, 0),
             (28, 4, 64, 4185, 4, 0), (60, 4, 64, 5208, 4, 0), (60, 4, 64, 1953, 4, 32), (64, 4, 256, 3051, 8, 0), (64, 4, 512, 1525, 8, 128),
             (512, 1, 50, 3125, 8, 0), (512, 1, 56, 2790, 8, 128), (12, 3, 1757, 3815, 8, 16), (16, 3, 1800, 4000, 4, 0),
             # Many units of rows off 4-byte boundaries.
             (500, 2, 192, 2187, 1, -128), (640, 2, 256, 1067, 1, -128), (350, 1, 256, 5357, 0, 512), (350, 1, 512, 2678, 0, -128)]
    out = dispatch(f"""
        o = outs()
        for N, F, M, B, off, units in {calls!r}:
            rc, h = plan(N, F, M, B, 1)
            assert rc == 0, sk.sk_last_error()
            log()
            assert sk.sk_compute(h, ctypes.c_void_p(X.value + off), None, ctypes.byref(o), None) == 0, sk.sk_last_error()
            name = launches()[0]
            kind = "shifted" if units < 0 else "phased"   # (below 0: shifted row phases)
            if (f"{{kind}}_kernelILi{{abs(units)}}E" not in name) if units else ("phased" in name or "shifted" in name):
                print(N, F, M, B, off, name)
            sk.sk_plan_destroy(h)
        """)
    assert out == ""


def test_lanes_of_small_input_counts(dispatch):
    # One input per lane up to 64 inputs that 4 does not divide, four for the others.
    calls = [(5, 8, 4, 20000, 1, "combine_kernelILi1E"), (63, 8, 4, 20000, 0, "combine_kernelILi1E"),
             (65, 8, 4, 20000, 1, "combine_kernelILi4E"), (64, 8, 4, 20000, 1, "combine_kernelILi4E"),
             (13, 1, 64, 300, 33, "window_kernel"), (2, 1, 64, 300, 33, "window_kernel"),
             (51, 8, 4, 20000, 1024, "step_kernel")]
    out = dispatch(f"""
        o = outs()
        for N, F, M, B, L, has in {calls!r}:
            rc, h = plan(N, F, M, B, L)
            log()
            assert sk.sk_compute(h, X, None, ctypes.byref(o), None) == 0, sk.sk_last_error()
            names = " ".join(launches()[1:])
            if has not in names:
                print(N, F, M, B, L, names)
        """)
    assert out == ""


def test_long_histories_fit_a_launch(dispatch):
    # 128 channels of 4 inputs with a window of 8 million blocks, in calls of 64: the
    # history rows that each call moves grow past what one launch can hold.
    out = dispatch("""
        o = outs()
        rc, h = plan(4, 128, 2, 64, 8388607)
        assert rc == 0, sk.sk_last_error()
        r = ctypes.byref(o)
        for c in range(140000):
            assert sk.sk_compute(h, X, None, r, None) == 0, (c, sk.sk_last_error())
            if c % 1000 == 0:
                names = launches()[-2:]
        print(names)
        """)
    assert "scan" in out and "combine" in out


def test_plan_memory(dispatch):
    # N, F, M, B, L and the bytes that plans of these sizes have always fitted in: they
    # still do, with a chunk length that needs fewer prefix rows if it must be, and plans
    # whose calls never take the window kernel hold nothing for it.
    out = dispatch("""
        b = ctypes.c_size_t()
        o = outs()
        for N, F, M, B, L, fits in [(2048, 4, 256, 1024, 256, 109019136), (2048, 4, 16, 4096, 256, 385843200),
                                    (1000, 3, 256, 128, 16, 5748000), (300, 8, 40, 5000, 16, 132297600),
                                    (16, 1, 256, 16, 4, 4032)]:
            fake.fake_limit(ctypes.c_size_t(fits))
            rc, h = plan(N, F, M, B, L)
            assert rc == 0, (N, F, M, B, L, sk.sk_last_error())
            assert sk.sk_compute(h, X, None, ctypes.byref(o), None) == 0, sk.sk_last_error()
            sk.sk_plan_destroy(h)
            assert fake.fake_used() == 0
            fake.fake_limit(ctypes.c_size_t(fits // 2))
            rc, h = plan(N, F, M, B, L)
            assert rc == -3 and not h.value and fake.fake_used() == 0, rc
            fake.fake_limit(ctypes.c_size_t(1 << 40))
        log()
        rc, h = plan(2048, 4, 256, 1024, 256)
        sk.sk_plan_device_bytes(h, ctypes.byref(b))
        print(b.value, len([line for line in log() if line.startswith("malloc")]))
        # Chunk sums come with the chunk length that uses them.
        assert sk.sk_plan_set_pass_b_tile(h, 4, 0) == 0
        print([line for line in log() if line.startswith("malloc")])
        """)
    lines = out.splitlines()
    assert lines[0] == f"{4 * (2 * 1024 + 1025 + 2 * 255) * 2048 * 4} 5"
    assert lines[1] == f"['malloc {4 * 512 * 2048 * 4}']"


def test_pass_a_workgroups_follow_the_devices_cus(dispatch):
    # About one workgroup per CU: a quarter of the CUs, four times the units each.
    out = dispatch("""
        o = outs()
        for cus in (256, 64):
            fake.fake_cus(cus)
            for N, F, M, B, off in [(1000, 3, 256, 128, 0), (1001, 3, 256, 40, 0)]:
                rc, h = plan(N, F, M, B, 1)
                log()
                assert sk.sk_compute(h, X, None, ctypes.byref(o), None) == 0, sk.sk_last_error()
                name = launches()[0]
                print(int(name.split("ILi")[1].split("E")[0]), "shifted" in name)
        """)
    assert out.split("\n")[:4] == ["128 False", "32 True", "512 False", "128 True"], out


def test_a_waiting_drain_is_not_woken_by_every_look(dispatch):
    # A frame that takes its time: the dispatcher looks at it every 10 us, but a thread
    # in sk_server_drain sleeps until it is done.
    out = dispatch("""
        import resource, threading, time

        class Server(ctypes.Structure):
            _fields_ = [("budget", ctypes.c_size_t), ("inflight", ctypes.c_int32), ("streams", ctypes.c_int32),
                        ("queue", ctypes.c_int32)]

        srv, ident, ticket, o = ctypes.c_void_p(), ctypes.c_int32(), ctypes.c_uint64(), outs()
        assert sk.sk_server_create(ctypes.byref(Server(1 << 30, 4, 2, 16)), ctypes.byref(srv)) == 0
        assert sk.sk_server_add_array(srv, ctypes.byref(desc(16, 1, 256, 16, 4)), ctypes.byref(ident)) == 0
        fake.fake_events(0)
        woken = []

        def drain():
            before = resource.getrusage(resource.RUSAGE_THREAD).ru_nvcsw
            assert sk.sk_server_drain(srv) == 0
            woken.append(resource.getrusage(resource.RUSAGE_THREAD).ru_nvcsw - before)

        assert sk.sk_stream_submit(srv, 0, X, 0, ctypes.byref(o), ctypes.c_uint64(0), None, ctypes.byref(ticket)) == 0
        t = threading.Thread(target=drain)
        t.start()
        time.sleep(0.3)
        assert t.is_alive()
        fake.fake_events(1)
        t.join(10)
        assert not t.is_alive()
        print(woken[0])
        sk.sk_server_destroy(srv)
        """)
    assert int(out) < 100, out
