"""Order of the library's work across streams, without a GPU: the library runs on
a stand-in for the HIP runtime (tests/hip_recorder.cpp) that records launches,
event records and waits, in a process of its own."""
import json
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ROCM = "/opt/rocm/include"
LIB = os.path.join(ROOT, "paper_2604_12083_amd", "libmrs.so")

pytestmark = pytest.mark.skipif(not (os.path.exists(LIB) and shutil.which("g++") and os.path.isdir(ROCM)),
                                reason="needs the built library, g++ and the HIP headers")

# out: what the child reports; A, B: stream handles of the caller; buf(n): an
# array of n doubles; log(): the recorded lines since the last call
_CHILD = """
import ctypes, json, sys
sys.modules["torch"] = None
import numpy as np
import paper_2604_12083_amd as mrs
rec = ctypes.CDLL(None)
rec.rec_take.restype = ctypes.c_char_p
log = lambda: rec.rec_take().decode().splitlines()
ready, capturing = rec.rec_events_ready, lambda s: rec.rec_capturing(ctypes.c_void_p(s))
A, B = 0x1000, 0x2000
keep = []
def buf(n):
    keep.append(np.zeros(n))
    return keep[-1]
def names(lines, kind):
    return [x.split()[1] for x in lines if x.split()[0] == kind]
def status(call, *a, **k):
    try:
        call(*a, **k)
    except mrs.MrsError as e:
        return e.status
    return 0
ctx = mrs.mrs_context_create(0)
def evaluate(n, stream=None, prec=mrs.MRS_FP64, call=mrs.mrs_eval_device):
    log()
    call(ctx, n, buf(3 * n), buf(3 * n), buf(3 * n), 0.1, 1.0, prec, buf(3 * n), buf(3 * n), stream)
    return log()
out = {}
"""


@pytest.fixture(scope="module")
def child(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("rec") / "rec.so")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-w", "-shared", "-fPIC", "-I", ROCM,
                           os.path.join(HERE, "hip_recorder.cpp"), "-o", lib])

    def run(body):
        env = dict(os.environ, LD_PRELOAD=lib, PYTHONPATH=ROOT)
        r = subprocess.run([sys.executable, "-c", _CHILD + body + "\nprint(json.dumps(out))"], cwd=ROOT, env=env,
                           stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=300)
        assert r.returncode == 0, r.stderr
        return json.loads(r.stdout.splitlines()[-1])

    return run


@pytest.mark.parametrize("n", [64, 20000])  # one launch, general path
def test_equal_handle_is_no_proof_of_order(child, n):
    """A stream may be destroyed with work in flight and its handle be given to
    another one: an evaluation waits for an unfinished one before it also on an
    equal handle, but not for a finished one, and a captured one not for what
    its own stream holds."""
    out = child(f"""
n = {n}
waits = lambda lines: names(lines, "wait")
out["first"] = waits(evaluate(n, A))
out["same handle"] = waits(evaluate(n, A))
out["other stream"] = waits(evaluate(n, B))
ready(1)
out["finished"] = waits(evaluate(n, A)); ready(0)
out["context stream"] = len(waits(evaluate(n)))
out["context stream again"] = len(waits(evaluate(n)))
evaluate(n, B); capturing(B)
out["captured"] = waits(evaluate(n, B))
""")
    assert out == {"first": [], "same handle": ["1000"], "other stream": ["2000"], "finished": [], "context stream": 1,
                   "context stream again": 1, "captured": []}


def test_setting_a_stream_waits_for_queued_state(child):
    """State, loads and time may still be on their way in on the stream that
    mrs_context_set_stream replaces, also when the new one has its handle."""
    out = child("""
ens = mrs.mrs_ensemble_create(ctx, [0, 8], buf(24), buf(72), None, None, 0.1, 1.0, mrs.rod_params())
mrs.mrs_context_set_stream(ctx, A)
log()
for name, call in (("state", lambda: mrs.mrs_ensemble_set_state(ctx, ens, buf(24), buf(72))),
                   ("loads", lambda: mrs.mrs_ensemble_set_external(ctx, ens, buf(24), buf(24))),
                   ("time", lambda: mrs.mrs_ensemble_set_time(ctx, ens, 1.0))):
    for stream in (B, B):
        call(); queued = log()
        mrs.mrs_context_set_stream(ctx, stream)
        out[name + " " + str(len(out))] = [x.split()[2] for x in queued if x.startswith("record")][-1:] == names(log(), "eventsync")
""")
    assert len(out) == 6 and all(out.values()), out


def test_state_and_loads_stay_out_of_graphs(child):
    """Rows go in and out through pinned memory that later calls use again, so a
    captured copy would replay other values: calls on a captured context stream
    are refused, without a launch, and leave everything as it was."""
    out = child("""
mrs.mrs_context_set_stream(ctx, A)
make = lambda: mrs.mrs_ensemble_create(ctx, [0, 8], buf(24), buf(72), buf(24), buf(24), 0.1, 1.0, mrs.rod_params())
ens = make()
calls = {"state": lambda: mrs.mrs_ensemble_set_state(ctx, ens, buf(24), buf(72)),
         "loads": lambda: mrs.mrs_ensemble_set_external(ctx, ens, buf(24), buf(24)),
         "time": lambda: mrs.mrs_ensemble_set_time(ctx, ens, 1.0),
         "get": lambda: mrs.mrs_ensemble_get(ctx, ens), "create": make}
for on in (True, False):
    capturing(A if on else None)
    for name, call in calls.items():
        log()
        out[f"{name} {on}"] = [status(call), len(names(log(), "launch")) > 0]
""")
    for name in ("state", "loads", "time", "get", "create"):
        assert out[name + " True"] == [-3, False] and out[name + " False"] == [0, True], (name, out)


def test_long_offset_lists_stay_out_of_graphs(child):
    """Filament offsets that fit the kernel's arguments may be captured; a longer
    list goes through a buffer that later calls use again and is refused."""
    out = child("""
call = lambda off: mrs.mrs_rod_forces_device(ctx, off, buf(3 * off[-1]), buf(9 * off[-1]), mrs.rod_params(), None, None,
                                             buf(3 * off[-1]), buf(3 * off[-1]), A)
uneven = lambda n: np.concatenate([[0], np.cumsum(2 + np.arange(n) % 2)])
capturing(A)
for name, off in (("equal", np.arange(2001) * 3), ("799", uneven(799)), ("800", uneven(800))):
    log()
    out[name] = [status(call, off), log()]
log(); X = buf(30)  # an output over an input goes through copies of the call's own
out["overlap"] = [status(mrs.mrs_rod_forces_device, ctx, [0, 10], X, buf(90), mrs.rod_params(), None, None, X, buf(30), A),
                  log()]
capturing(None)
out["not captured"] = [status(call, uneven(800)), len(names(log(), "launch"))]
""")
    launch = "launch k_rod_forces_aos 1000"
    assert out == {"equal": [0, [launch]], "799": [0, [launch]], "800": [-3, []], "overlap": [-3, []],
                   "not captured": [0, 1]}


@pytest.mark.parametrize("prec,n,entry,untuned,followed", [
    (0, 1000, (0, 1, 4), "k_eval_direct<", "k_pairs_tile_f64<1, false, true>"),
    (0, 2048, (0, 1, 16), "k_eval_direct<", "k_pairs_tile_f64<1, false, true>"),
    (0, 6144, (0, 2, 9), "k_eval_direct<", "k_pairs_tile_f64<2, false, false>"),
    (0, 6145, (0, 2, 9), None, "k_pairs_tile_f64<2, false, false>"),
    (1, 3072, (0, 2, 4), "k_eval_direct<", "k_pairs_tile_f32<2, false, false>"),
    (1, 5120, (0, 2, 4), "k_pairs_tile_f32<1, false, true>", "k_pairs_tile_f32<2, false, false>"),
    (1, 5121, (0, 2, 4), None, "k_pairs_tile_f32<2, false, false>")])
@pytest.mark.parametrize("call", ["mrs_eval_device", "mrs_eval_device_noalloc"])
def test_evaluations_keep_their_own_kernels_in_a_tuned_class(child, tmp_path, prec, n, entry, untuned, followed, call):
    """An entry that the tuner stored (it has times) was timed against the kernels
    of an ensemble: one-shot evaluations follow it only beyond the sizes for which
    they have faster kernels of their own, an entry set by hand always."""
    line = f"{prec} {n.bit_length() - 1} {entry[0]} {entry[1]} {entry[2]} 0"
    files = {}
    for name, times in (("tuned", "0.02 0.03"), ("hand", "-1 -1")):
        files[name] = str(tmp_path / name)
        with open(files[name], "w") as f:
            f.write(f"mrs-pair-tuning 1 gfx950 256 0\n{line} {times}\n")
    out = child(f"""
run = lambda: [x[7:x.rindex(" ")] for x in evaluate({n}, A, {prec}, mrs.{call}) if x.startswith("launch")]
out["none"] = run()
for name, path in {files!r}.items():
    mrs.mrs_tune_load(ctx, path)
    out[name] = run()
    out[name + " chunks"] = mrs.mrs_tune_get(ctx, {n}, {prec})["chunks"]
""")
    tiled = ["k_pack_aos", followed, "k_reduce<0>"]
    assert out["hand"] == tiled and out["hand chunks"] == out["tuned chunks"] == entry[2]
    if untuned is None:
        assert out["tuned"] == tiled
    else:
        assert out["tuned"] == out["none"] and out["tuned"] != tiled and out["tuned"][len(out["tuned"]) // 2].startswith(untuned)


@pytest.mark.parametrize("call", ["mrs_eval_device", "mrs_eval_device_noalloc"])
@pytest.mark.parametrize("prec,n", [(0, 6145), (0, 20000), (1, 5003), (1, 12800)])
def test_captured_work_lists_are_kernel_arguments(child, call, prec, n):
    """A replay reads a captured copy's host memory again, when the call's list is
    gone (or its staging buffer holds another call's): under capture the list
    travels in kernel arguments, ahead of the kernels that read it."""
    out = child(f"""
rec.rec_symbol.restype = ctypes.c_void_p
arrays = [buf(3 * {n}) for _ in range(5)]
def run():
    log()
    mrs.{call}(ctx, {n}, *arrays[:3], 0.1, 1.0, {prec}, *arrays[3:], A)
    return [x.rsplit(" ", 1)[0] if x[0] == "l" else x.split()[0] for x in log()]
out["eager"] = run()
eager = ctypes.string_at(rec.rec_symbol(), 1 << 20)
ctypes.memset(rec.rec_symbol(), 0, 1 << 20)
ctx = mrs.mrs_context_create(0)
capturing(A); out["captured"] = run(); capturing(None)
out["same list"] = [eager == ctypes.string_at(rec.rec_symbol(), 1 << 20), any(eager)]
""")
    assert out["same list"] == [True, call == "mrs_eval_device_noalloc"]
    names = out["captured"]
    lists = names.count("launch k_store_list")
    assert lists and names[:lists] == ["launch k_store_list"] * lists and names[lists] == "launch k_pack_aos"
    assert "copy" not in names and "eventsync" not in names
    kernels = lambda names: [x for x in names if x.startswith("launch") and x != "launch k_store_list"]
    assert kernels(names) == kernels(out["eager"]) and "launch k_store_list" not in out["eager"]
