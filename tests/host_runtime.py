"""The library on a host-only HIP runtime (hip_host.cpp): `python tests/host_runtime.py <stub.so>
<name>` runs one check below and prints its result as JSON.  A process of its own, without torch,
because the stand-in has to be loaded before any HIP runtime."""
from __future__ import annotations

import ctypes as C
import json
import os
import subprocess
import sys
import time

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1305_0036_amd", "libtsspin.so")
C128, C64 = 0, 1


def run(tmp_path, check, *args, env=None):
    """Run `check(*args)` in a process with the stand-in preloaded and return its result."""
    so = os.path.join(str(tmp_path), "hip_host.so")
    if not os.path.exists(so):
        subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-I/opt/rocm/include", "-o", so,
                        os.path.join(ROOT, "tests", "hip_host.cpp")], check=True)
    e = dict(os.environ, LD_PRELOAD=so, TSSPIN_NO_TUNE_CACHE="1", **(env or {}))
    p = subprocess.run([sys.executable, os.path.abspath(__file__), check, json.dumps(args)], env=e,
                       capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stderr[-2000:]
    return json.loads(p.stdout.splitlines()[-1])


class Bond(C.Structure):
    _fields_ = [("i", C.c_int32), ("j", C.c_int32), ("jx", C.c_double), ("jy", C.c_double), ("jz", C.c_double)]


class Host:
    def __init__(self):
        self.lib = C.CDLL(LIB)
        self.rt = C.CDLL(os.environ["LD_PRELOAD"])
        for f in ("host_held", "host_peak"):
            getattr(self.rt, f).restype = C.c_size_t
        self.lib.ts_last_error.restype = C.c_char_p

    def ok(self, rc):
        assert rc == 0, (rc, self.lib.ts_last_error())

    @staticmethod
    def bonds(n, ring=False):
        b = [(i, i + 1, 0.7 + 0.01 * i, 0.8, 0.9) for i in range(n - 1)] + ([(0, n - 1, 0.5, 0.6, 0.7)] if ring else [])
        return (Bond * max(1, len(b)))(*b), len(b)

    def system(self, n, ring=False):
        b, nb = self.bonds(n, ring)
        f = (C.c_double * (3 * n))(*[0.1 + 0.01 * i for i in range(3 * n)])
        ctx = C.c_void_p()
        self.ok(self.lib.ts_create(n, b, nb, f, C.byref(ctx)))
        return ctx

    def evolve(self, ctx, dtype, steps, order=4, dt=0.05):
        psi = (C.c_void_p * 1)(4096)   # never dereferenced: the kernels do nothing
        self.ok(self.lib.ts_evolve(ctx, psi, 1, dtype, C.c_double(dt), C.c_int64(steps), order, None, 0, 1, None, None))

    def batch(self, ns):
        b, off, f = [], [0], []
        for n in ns:
            x, nb = self.bonds(n)
            b += list(x)[:nb]
            off.append(len(b))
            f += [0.1 + 0.01 * i for i in range(3 * n)]
        ctx = C.c_void_p()
        self.ok(self.lib.ts_create_batch(len(ns), (C.c_int32 * len(ns))(*ns), (Bond * max(1, len(b)))(*b),
                                         (C.c_int32 * len(off))(*off), (C.c_double * len(f))(*f), C.byref(ctx)))
        return ctx

    def evolve_batch(self, ctx, ns, dtype, steps, order=4, dt=0.05, at=4096):
        off, t = [], 0
        for n in ns:
            off.append(t)
            t += 1 << n
        return self.lib.ts_evolve_batch(ctx, C.c_void_p(at), (C.c_int64 * len(off))(*off), dtype, C.c_double(dt),
                                        C.c_int64(steps), order, None, 0, 1, None, None)

    def autotune(self, ctx, dtype, use_cache, order=4):
        ms = C.c_double()
        self.ok(self.lib.ts_autotune(ctx, dtype, order, C.c_void_p(4096), use_cache, C.byref(ms), None))

    def launches(self, part):
        return self.rt.host_launches(part.encode())


# ---------------------------------------------------------------- checks

def tuned_after_evolving(h, dtype):
    ctx = h.system(20)
    h.evolve(ctx, dtype, 2)
    before = h.launches("cone_kernel")
    h.autotune(ctx, dtype, 1)
    h.rt.host_reset()
    h.evolve(ctx, dtype, 2)
    return {"before": before, "after_cone": h.launches("cone_kernel"), "after_reg": h.launches("sweep_reg_kernel")}


def tuner_launches(h, dtype):
    ctx = h.system(20)
    h.autotune(ctx, dtype, 0)
    return {"cone": h.launches("cone_kernel")}


def first_call(h, n, dtype, steps):
    h.rt.host_reset()
    h.evolve(h.system(n), dtype, steps)
    return {"allocs": h.rt.host_allocs(), "uploads": h.rt.host_uploads(), "sweeps": h.launches("cone_kernel")}


def narrow_first_call(h, n):
    """Least processor time of the first call of a ring at its own width over that at width 12."""
    best = {0: 1e9, 12: 1e9}
    for _ in range(25):
        for width in best:
            ctx = h.system(n, ring=True)
            h.ok(h.lib.ts_set_tile_bits(ctx, C128, width))
            t = time.thread_time()
            h.evolve(ctx, C128, 8)
            best[width] = min(best[width], time.thread_time() - t)
            h.ok(h.lib.ts_destroy(ctx))
    return {"ratio": best[0] / best[12]}


def batch_tables(h, n, chains, dtype, dts, pointers):
    """Device bytes held after each call of a batch: every time step at every state pointer."""
    ctx, ns, held = h.batch([n] * chains), [n] * chains, []
    for dt in dts:
        for at in pointers:
            h.ok(h.evolve_batch(ctx, ns, dtype, 1, dt=dt, at=at))
            held.append(h.rt.host_held())
    return held


def batch_groups(h, n, chains, dtype):
    """Launches of one call's program (they are captured once) and their fills."""
    ctx, ns = h.batch([n] * chains), [n] * chains
    h.rt.host_reset()
    h.ok(h.evolve_batch(ctx, ns, dtype, 1))
    fills = h.launches("resident_phase_kernel") + h.launches("resident_diag_kernel")
    return {"fills": fills, "runs": h.launches("15resident_kernel")}


def batch_short_of_memory(h, n, chains, dtype, spare):
    """A first call with `spare` bytes less than it would like."""
    ctx, ns = h.batch([n] * chains), [n] * chains
    h.ok(h.evolve_batch(ctx, ns, dtype, 1, dt=0.05))
    h.ok(h.lib.ts_destroy(ctx))
    need = h.rt.host_peak()
    ctx = h.batch(ns)
    h.rt.host_limit(C.c_size_t(need - spare))
    rc = h.evolve_batch(ctx, ns, dtype, 1, dt=0.05)
    return {"rc": rc, "failed": h.rt.host_failed()}


def resident_factors(h, n, dtype):
    """Launches that store the factors of a resident state's phase steps, and of its kernel."""
    h.evolve(h.system(n), dtype, 3)
    return {"stored": h.launches("resident_factor_kernel"), "runs": h.launches("15resident_kernel")}


def tuner_widths(h, n, dtype):
    """Launches of the narrow untuned width in a tuning, and the kernel configuration before it."""
    ctx, cfg = h.system(n, ring=True), [C.c_int32() for _ in range(3)]
    h.ok(h.lib.ts_get_kernel_config(ctx, dtype, 4, *[C.byref(c) for c in cfg]))
    h.rt.host_reset()
    h.autotune(ctx, dtype, 0)
    return {"untuned": [c.value for c in cfg[:2]], "timed": h.launches(f"sweep_reg_kernelIdLi{cfg[0].value}ELi{cfg[1].value}E")}


def call_after_a_refused_allocation(h, n, dtype):
    """The result of a call without memory for its tables, and of the same call with it."""
    ctx, psi = h.system(n, ring=True), (C.c_void_p * 1)(4096)
    args = (ctx, psi, 1, dtype, C.c_double(0.05), C.c_int64(2), 4, None, 0, 1, None, None)
    h.rt.host_limit(C.c_size_t(0))
    first = h.lib.ts_evolve(*args)
    h.rt.host_limit(C.c_size_t(1 << 40))
    return [first, h.lib.ts_evolve(*args)]


if __name__ == "__main__":
    print(json.dumps(globals()[sys.argv[1]](Host(), *json.loads(sys.argv[2]))))
