"""What a host dispatch test's program starts from: libsk.so over the fake HIP
runtime (paths: arguments 1 and 2), its structures, and the fake's log. The program
itself is argument 3."""
import ctypes
import sys

fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sk = ctypes.CDLL(sys.argv[2])
fake.fake_log.restype = ctypes.c_char_p
fake.fake_used.restype = ctypes.c_size_t
sk.sk_last_error.restype = ctypes.c_char_p


class Desc(ctypes.Structure):
    _fields_ = [("n_inputs", ctypes.c_int32), ("n_channels", ctypes.c_int32), ("n_samples", ctypes.c_int64),
                ("block_len", ctypes.c_int32), ("norm_window_blocks", ctypes.c_int32), ("estimator", ctypes.c_int32),
                ("k_sigma", ctypes.c_double), ("expect_offset", ctypes.c_double), ("sigma_override", ctypes.c_double)]


class Outs(ctypes.Structure):
    _fields_ = [(k, ctypes.c_void_p) for k in ("s1", "s2", "r1", "r2", "v", "flags", "n_eff", "sk_i", "significance")]


def desc(N, F, M, B, L):
    return Desc(N, F, M * B, M, L, 0, 5.0, 0.0, 0.0)


def outs():
    return Outs(*[0x600000000000 + (k << 36) for k in range(7)], None, None)


def plan(N, F, M, B, L):
    h = ctypes.c_void_p()
    rc = sk.sk_plan_create(ctypes.byref(desc(N, F, M, B, L)), ctypes.byref(h))
    return rc, h


def log():
    return fake.fake_log().decode().splitlines()


def launches():
    return [line.split()[1] for line in log() if line.startswith("launch")]


X = ctypes.c_void_p(0x500000000000)
exec(compile(open(sys.argv[3]).read(), sys.argv[3], "exec"))
