"""What the library's host code asks of HIP, and in which order, without a
GPU: a child process runs a scenario on a preloaded stand-in for the HIP host
calls (tests/hip_standin.c), which runs no kernel and writes the calls down."""
import ctypes as C
import os
import shutil
import subprocess
import sys

import pytest

from paper_2609_27193_amd.build_lib import GRID_CAPPED_LIB, LIB

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DEVICE, HOST = 2, 1  # hipMemoryTypeDevice, hipMemoryTypeHost


@pytest.fixture(scope="module")
def standin(tmp_path_factory):
    gcc, rocm = shutil.which("gcc"), os.environ.get("ROCM_PATH", "/opt/rocm")
    if not gcc or not os.path.exists(LIB) or not os.path.exists(GRID_CAPPED_LIB):
        pytest.skip("needs gcc and the libraries of __graft_entry__.build()")
    so = str(tmp_path_factory.mktemp("standin") / "libhip_standin.so")
    subprocess.run([gcc, "-std=c11", "-O1", "-Wall", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(rocm, "include"), os.path.join(ROOT, "tests", "hip_standin.c"),
                    "-o", so], check=True)
    return so


def in_child(standin, lib, scenario, *args):
    env = dict(os.environ, LD_PRELOAD=standin, HIP_STANDIN=standin, LAYERCHECK_LIB=lib)
    r = subprocess.run([sys.executable, "-c", f"import tests.test_host_calls as t; t.{scenario}(*{args!r})"],
                       cwd=ROOT, env=env, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.stdout + r.stderr)[-3000:]


# ---- in the child: no torch, nothing touches a GPU --------------------------------------------------------------------


def hip():
    h = C.CDLL(os.environ["HIP_STANDIN"])
    h.standin_log.restype = C.c_char_p
    h.standin_alloc.restype = C.c_void_p
    h.standin_alloc.argtypes = [C.c_size_t, C.c_int]
    h.words = lambda: [w.split(":")[0] for w in h.standin_log().decode().split()]
    return h


def context(h, sizes):
    """One fp32 segment a layer, weights, shadow and moments."""
    from paper_2609_27193_amd import layercheck as LC
    segs = [LC.Segment(l, n, *(h.standin_alloc(4 * n, DEVICE) for _ in "ws"), None,
                       *(h.standin_alloc(4 * n, DEVICE) for _ in "mv")) for l, n in enumerate(sizes)]
    ctx = LC.lc_init_layout(LC.LayoutDesc(segs, len(sizes), LC.LC_DT_F32, False, LC.LC_MODE_ACCUM, [1.0] * len(sizes), 9))
    h.standin_clear()
    return LC, ctx


def failed_restore(n_layers, where):
    import numpy as np
    h = hip()
    sizes = [40 * 2048] * 3 + [1] * (n_layers - 3)
    LC, ctx = context(h, sizes)
    total = sum(LC.lc_record_bytes(ctx, l) for l in range(n_layers))
    v = [{"step": 0, "mask": np.ones(n_layers, np.uint8), "payload": h.standin_alloc(total, where), "payload_bytes": total}]
    launches = 0
    for fail in range(1, 1000):  # every launch of the call fails once
        h.standin_clear()
        h.standin_fail_launch(fail)
        try:
            LC.lc_restore_composite(ctx, v, 0, n_layers)
        except LC.LCError as e:
            assert e.code == LC.LC_ERR_HIP
            w = h.words()
            # an earlier launch may still read the payload and write the arrays
            assert w[-1] == "sync", (fail, w)
            launches = fail
            _, ctx = context(h, sizes)  # the failed one is out of use
            continue
        break
    assert launches >= 3, launches


def state_read():
    h = hip()
    LC, ctx = context(h, [5, 3000, 1])
    LC.lc_score_layers(ctx, 1)
    assert h.words()[-1] != "sync"
    LC.lc_read_state(ctx, 3)
    assert h.words()[-1] == "sync", h.words()


def stale_error(where, n_layers):
    import numpy as np
    h = hip()
    LC, ctx = context(h, [3000] * n_layers)
    total = sum(LC.lc_record_bytes(ctx, l) for l in range(n_layers))
    pageable = (C.c_uint8 * total)()
    at = h.standin_alloc(total, where) if where else C.addressof(pageable)
    v = [{"step": 0, "mask": np.ones(n_layers, np.uint8), "payload": at, "payload_bytes": total}]
    h.standin_stale_error()
    LC.lc_read_state(ctx, n_layers)
    h.standin_stale_error()
    LC.lc_restore_composite(ctx, v, 0, n_layers)


def selection_wait():
    import time
    h = hip()
    LC, ctx = context(h, [3000])
    LC.lc_score_layers(ctx, 1)
    h.standin_clear()
    t = time.perf_counter()
    try:
        LC.lc_select(ctx, 1, 1.0, 1)  # no kernel runs: the number never comes
        raise AssertionError("no error")
    except LC.LCError as e:
        assert e.code == LC.LC_ERR_HIP
    took = time.perf_counter() - t
    w = [x for x in h.words() if x in ("query", "sync")]
    assert w == ["query"] and took > 0.5e-3, (w, took)


def gradient_tables(n, fetches):
    h = hip()
    LC, ctx = context(h, [1] * n)
    g = [h.standin_alloc(4, DEVICE)] * n
    LC.lc_sgd_step_score(ctx, 1, g, LC.LC_DT_F32, 1e-3, 0.0)
    first = [w for w in h.words() if "fetch_kernel" in w or w == "query"]
    assert len(first) == fetches and "query" not in first, first  # nothing to wait for yet
    h.standin_clear()
    h.standin_busy(3)  # the fetch has not run: the number it writes is not there, and the stream is busy
    LC.lc_sgd_step_score(ctx, 2, g, LC.LC_DT_F32, 1e-3, 0.0)
    w = [x for x in h.words() if "fetch_kernel" in x or x == "query"]
    assert w == ["query"] * (4 if fetches else 0) + first, w


# ---- the tests ---------------------------------------------------------------------------------------------------------


@pytest.mark.parametrize("where", [DEVICE, HOST], ids=["device", "page-locked"])
@pytest.mark.parametrize("n_layers", [3, 108, 109])
def test_a_failed_restore_waits_for_what_it_launched(standin, n_layers, where):
    """The caller may free or reuse the payload as soon as the call has returned, also with an error; the ranks ride in
    the kernel's arguments up to 108 layers, beyond that in a table."""
    in_child(standin, GRID_CAPPED_LIB, "failed_restore", n_layers, where)


def test_reading_the_state_synchronises_the_stream(standin):
    """As the header promises: the stream is idle when the call returns."""
    in_child(standin, LIB, "state_read")


def test_a_selection_is_polled_for_long_before_the_stream_is_queried(standin):
    """A query just before the selection arrives holds up the pack; a stream that drains without it still ends the wait."""
    in_child(standin, LIB, "selection_wait")


@pytest.mark.parametrize("where", [HOST, 0], ids=["page-locked", "pageable"])
@pytest.mark.parametrize("n_layers", [3, 109])
def test_an_error_of_the_program_fails_no_state_read_or_restore(standin, n_layers, where):
    """A call of the program that failed before leaves its error with the runtime.  The state read and the restore from
    host memory ask for their own launches' errors only, as copies do."""
    in_child(standin, LIB, "stale_error", where, n_layers)


@pytest.mark.parametrize("n,fetches", [(224, 0), (225, 1), (4096, 1), (4097, 2)])
def test_a_gradient_table_waits_for_the_fetch_of_the_one_before(standin, n, fetches):
    """Up to 224 segments the table rides in the kernel's arguments; beyond that the page-locked table may not be written
    while the fetch of the previous call is under way (beyond 4096 a second launch behind the fetch says that it is done)."""
    in_child(standin, LIB, "gradient_tables", n, fetches)
