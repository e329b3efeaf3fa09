"""What a batch launches, computed on the CPU: the library's host code built
against a recorded device (tests/host_plan.cpp), so that limits of workgroups
and LDS are checked for batches of every shape without a GPU."""
import ctypes as C
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

from paper_2006_09616_amd import dtr as D
from paper_2006_09616_amd import workloads as W

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2006_09616_amd", "csrc")
LDS = 160 * 1024
FIELDS = ["group", "sims", "slots", "slot_bytes", "waves", "sweep_chunks", "small_n", "lds_static", "lds_dynamic",
          "stream", "small_at"]


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    if not shutil.which("g++") or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("no g++ or HIP headers")
    so = tmp_path_factory.mktemp("plan") / "libplan.so"
    res = subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__",
                          "-include", "dtr_sim.h", "-I", "/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
                          "-I", CSRC, "-o", str(so), os.path.join(HERE, "host_plan.cpp"),
                          os.path.join(CSRC, "dtr_sim.cpp"), os.path.join(CSRC, "dtr_log.cpp")],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    lib = C.CDLL(str(so))
    lib.dtr_sim_last_error.restype = C.c_char_p
    vp, i32, sz = C.c_void_p, C.c_int32, C.c_size_t
    for kind in ("dtr_sim", "dtr_log"):
        getattr(lib, kind + "_workspace_bytes").argtypes = [vp, i32, vp, i32, vp, C.POINTER(sz)]
        getattr(lib, kind + "_create").argtypes = [vp, i32, vp, i32, vp, vp, sz, vp, C.POINTER(vp)]
    for f in (lib.dtr_sim_run, lib.dtr_sim_run_static):
        f.argtypes = [vp, vp]
    lib.dtr_sim_destroy.argtypes = [vp]
    lib.dtr_sim_launch_info.argtypes = [vp, vp]
    lib.plan_launches.argtypes = [vp, i32]
    lib.plan_streams.argtypes = [vp]
    lib.plan_capture.argtypes = [i32]

    def launches(programs, specs, logs=False, flags=0, slots=0, stream=None):
        opts = {"flags": flags, "slots": slots} if flags or slots else None
        p = (D._PackedLogs if logs else D._Packed)(programs, specs, opts)
        size, h = sz(0), vp()
        kind = "dtr_log" if logs else "dtr_sim"
        check = lambda rc: pytest.fail(lib.dtr_sim_last_error().decode()) if rc else None
        check(getattr(lib, kind + "_workspace_bytes")(*p.args(), C.byref(size)))
        ws = np.empty(size.value + 256, np.uint8)               # only the tables at its head are touched
        at = (ws.ctypes.data + 255) // 256 * 256
        check(getattr(lib, kind + "_create")(*p.args(), at, size, None, C.byref(h)))
        check((lib.dtr_sim_run_static if flags & D.OPT_STATIC_SCRATCH else lib.dtr_sim_run)(h, stream))
        out = (C.c_int64 * (len(FIELDS) * 16))()
        n = lib.plan_launches(out, 16)
        info = D._LaunchInfo()
        check(lib.dtr_sim_launch_info(h, C.byref(info)))
        lib.dtr_sim_destroy(h)
        rows = [dict(zip(FIELDS, out[len(FIELDS) * i:])) for i in range(n)]
        assert n > 0 and sum(r["sims"] for r in rows) == len(specs)
        for r in rows:
            assert r["lds_static"] + r["lds_dynamic"] <= LDS, r
        assert info.lds_bytes == max(r["lds_dynamic"] for r in rows)
        return rows

    keep = []

    def create(programs, specs):
        """A handle that has not run, for its caller to destroy."""
        p, size, h = D._Packed(programs, specs, None), sz(0), vp()
        assert lib.dtr_sim_workspace_bytes(*p.args(), C.byref(size)) == 0
        keep.append(np.empty(size.value + 256, np.uint8))
        assert lib.dtr_sim_create(*p.args(), (keep[-1].ctypes.data + 255) // 256 * 256, size, None, C.byref(h)) == 0
        return h

    launches.lib, launches.create = lib, create
    return launches


def _batch(*parts):
    """Specs of (trace, heuristic, simulations[, search]) parts."""
    return W.make_specs([(t, h, 50 + k, k, W.POLICY_EAGER, s[0] if s else 0)
                         for t, h, n, *s in parts for k in range(n)])


LONG = W.chain_trace(4096)                   # 8192 tensors


@pytest.mark.parametrize("n", [945, 959, 960, 999, 1000, 1023])
def test_workgroups_fit_at_every_wavefront_count(plan, n):
    """Chains of 1892 to 2048 operations, swept with their state in LDS at few
    wavefronts, stay within a workgroup's LDS at every number of wavefronts,
    alone, with the search approximations, and beside a trace of 8192 tensors
    under a heuristic of any class."""
    tr = W.chain_trace(n)
    assert tr.n_tensors <= 2048 and tr.n_ops <= 2048
    for search in (0, 3):
        for waves in (0, 1, 2, 4, 5, 6, 7, 8):
            plan([tr], _batch((0, W.H_DTR, 3, search)), flags=D.opt_walk_waves(waves))
        for h in (W.H_EQ, W.H_LRU, W.H_DTR):
            plan([tr, LONG], _batch((0, W.H_DTR, 3, search), (1, h, 2)))
            plan([tr, LONG, W.chain_trace(700)], _batch((0, W.H_MSPS, 3), (1, h, 2), (2, W.H_DTR, 2, 3)))


@pytest.mark.parametrize("n", [8, 31, 32, 64, 96, 600, 992, 1000])
@pytest.mark.parametrize("waves", [0, 1, 3, 4])
def test_stacks_in_lds_start_at_a_quad(plan, n, waves):
    """The state words and stacks (16-byte quads) follow the sweeps' arrays at
    a multiple of 16 bytes, for odd and even numbers of 64-operation chunks."""
    for search in (0, 3):
        (row,) = plan([W.chain_trace(n)], _batch((0, W.H_DTR, 2, search)), flags=D.opt_walk_waves(waves))
        assert row["small_n"] > 0 and row["sweep_chunks"] == (2 * n + 63) // 64
        assert row["small_at"] % 16 == 0, row


def test_swept_and_lane_walked_traces_are_separate_groups(plan):
    """One batch's traces do not set each other's workgroups: lane walks hold
    no sweep arrays, and a long trace of any group leaves the wavefronts, the
    chunks and the LDS state of the swept ones as they are alone."""
    short, long_ = W.chain_trace(150), W.chain_trace(1100)
    key = lambda r: {f: r[f] for f in ("waves", "sweep_chunks", "small_n", "lds_dynamic")}
    (alone,) = plan([short], _batch((0, W.H_DTR, 4)))
    (lanes,) = plan([long_], _batch((0, W.H_DTR, 4)))
    assert alone["sweep_chunks"] == 5 and alone["waves"] == 4 and alone["small_n"] > 0
    assert lanes["sweep_chunks"] == 0 and lanes["lds_dynamic"] == 0 and lanes["group"] != alone["group"]
    for other in (W.H_DTR, W.H_MSPS, W.H_LRU, W.H_EQ):
        for search in (0, 3):
            rows = plan([short, long_, LONG], _batch((0, W.H_DTR, 4), (1, W.H_DTR, 4), (2, other, 1, search)))
            mine = [r for r in rows if r["group"] == alone["group"]]
            assert len(mine) == 1 and key(mine[0]) == key(alone)
            mixed = [r for r in rows if r["group"] == lanes["group"]]
            assert len(mixed) == 1 and mixed[0]["lds_dynamic"] == 0
            assert mixed[0]["waves"] == (8 if other in (W.H_DTR, W.H_MSPS) and not search else lanes["waves"])
    both = plan([short, W.chain_trace(1000)], _batch((0, W.H_DTR, 2, 1), (1, W.H_DTR, 2)))
    assert sorted(r["sweep_chunks"] for r in both) == [5, 32]


def test_slots_hold_lane_walk_arrays_only_for_lane_walks(plan):
    """Sweeps keep their sets in LDS: a batch whose walks are all swept has the
    slots of a batch without walks, however many wavefronts sweep; a batch
    with a lane-walked trace pays for that group's wavefronts."""
    rn = W.resnet_trace(seed=1, blocks=50)
    slot = lambda specs, tr=(rn,), flags=0: plan(list(tr), specs, flags=flags)[0]["slot_bytes"]
    none = slot(_batch((0, W.H_LRU, 8)))
    for h in (W.H_DTR, W.H_MSPS, W.H_ESTAR):
        for search in (0, 3):
            for waves in (0, 1, 2, 8):
                assert slot(_batch((0, h, 8, search)), flags=D.opt_walk_waves(waves)) == none
    lanes = {w: slot(_batch((0, W.H_DTR, 8)), flags=D.opt_walk_waves(w) | D.OPT_WALK_QUEUE_SMALL) for w in (1, 2)}
    assert none < lanes[1] < lanes[2]
    # a batch in the static working memory is resident as a whole
    specs = _batch((0, W.H_DTR, 256), (0, W.H_EQ, 256), (0, W.H_LRU, 256))
    assert sum(r["slots"] for r in plan([rn], specs, flags=D.OPT_STATIC_SCRATCH)) == 768


@pytest.mark.parametrize("search", [0, 3])
def test_sweeping_wavefronts_by_simulations_in_flight(plan, search):
    """Few simulations sweep with many wavefronts each, many with few: as many
    as leave at most half as many again waiting as are resident (a compute
    unit holds two workgroups of four wavefronts, four of two, eight of one,
    or fewer where their LDS says so); slots and the static working memory
    count as what is in flight."""
    rn, small = W.resnet_trace(seed=1, blocks=50), W.chain_trace(32)
    waves = lambda n, tr=rn, **kw: plan([tr], _batch((0, W.H_DTR, n, search)), **kw)[0]["waves"]
    assert [waves(n) for n in (1, 256, 768, 769, 1536, 1537, 8192)] == [4, 4, 4, 2, 2, 1, 1]
    assert [waves(n, small) for n in (1, 1536, 1537)] == [2, 2, 1]
    assert waves(8192, flags=D.opt_walk_waves(4)) == 4
    assert waves(8192, slots=256) == 4 and waves(8192, slots=1024) == 2
    # 170 KB a simulation: 1586 fit the static working memory, shared with the other group
    both = _batch((0, W.H_DTR, 4096, search), (0, W.H_LRU, 4096, search))
    assert plan([rn], both, flags=D.OPT_STATIC_SCRATCH)[0]["waves"] == 2
    assert plan([rn], both)[0]["waves"] == 1


def _resident(row, small):
    """Simulations that 256 compute units hold of a launch's kernel, by LDS
    and by the wavefronts its registers allow."""
    per_wg = 4 if row["group"] == 0 else 1
    waves = row["waves"] if row["sweep_chunks"] else per_wg
    regs = 12 if row["group"] == 3 else 8
    return 256 * min(LDS // (row["lds_static"] + (row["lds_dynamic"] if small else row["small_at"])), regs // waves) * per_wg


@pytest.mark.parametrize("h,search", [(W.H_LRU, 0), (W.H_LRU, 3), (W.H_EQ, 0), (W.H_EQ, 3), (W.H_DTR, 0), (W.H_DTR, 3)])
@pytest.mark.parametrize("tensors", [30, 96, 130, 604, 1200, 2000, 2048])
def test_lds_state_leaves_no_simulation_waiting(plan, h, search, tensors):
    """State words and stack tops are in LDS while the batch is resident that
    way, and beyond it only where they cost no residency."""
    tr = W.chain_trace(tensors // 2)
    for n in (1, 64, 1000, 1024, 1025, 1280, 1281, 2048, 3000, 4096, 9000):
        (row,) = plan([tr], _batch((0, h, n, search)))
        if row["small_n"] == 0:
            (few,) = plan([tr], _batch((0, h, 1, search)))
            assert few["small_n"] == tr.n_tensors
            if few["waves"] == row["waves"]:
                assert n > _resident(few, True) and _resident(few, True) < _resident(few, False)
        else:
            assert n <= _resident(row, True) or _resident(row, True) == _resident(row, False), (n, row)


@pytest.mark.parametrize("blocks,walks,simple,mixed", [
    (4, (4, 1), 1, (4, 1)), (50, (4, 1), 1, (2, 1)), (58, (2, 1), 1, (2, 1)), (66, (1, 1), 1, (1, 1)),
    (70, (1, 1), 1, (2, 0)), (72, (2, 0), 1, (2, 0)), (80, (1, 0), 1, (1, 0)), (84, (1, 0), 1, (1, 0)),
    (86, None, 1, None), (90, None, 0, None)])
def test_logs_stay_in_lds(plan, blocks, walks, simple, mixed):
    """A residual network's log keeps its state in LDS up to 84 blocks, swept
    up to 70, with the wavefronts that fit: (waves, swept) of a batch with
    walk heuristics and of one with a cyclic log beside it, and whether a
    batch without walks is in LDS."""
    lg, cyclic = W.resnet_log(seed=1, blocks=blocks), W.random_log(5, n_steps=100, n_const=2)
    shape = lambda r: (r["waves"], r["sweep_chunks"]) if r["lds_dynamic"] else None
    for hs in ((W.H_DTR,), (W.H_MSPS, W.H_LRU), (W.H_DTR, W.H_EQ, W.H_LOCAL, W.H_LRU, W.H_SIZE, W.H_RAND)):
        (row,) = plan([lg], _batch(*[(0, h, 2) for h in hs]), logs=True)
        assert shape(row) == walks, row
        assert row["lds_dynamic"] <= LDS
    (row,) = plan([lg], _batch((0, W.H_EQ, 2), (0, W.H_LRU, 2)), logs=True)
    assert (row["lds_dynamic"] > 0) == simple and row["waves"] == 1
    (row,) = plan([lg, cyclic], _batch((0, W.H_DTR, 2), (1, W.H_DTR, 2)), logs=True)
    assert shape(row) == mixed, row
    # a large log without walks holds no rows for a small swept one
    (row,) = plan([lg, W.resnet_log(seed=2, blocks=2)], _batch((0, W.H_LRU, 2), (1, W.H_DTR, 2)), logs=True)
    assert row["sweep_chunks"] == 1 or walks is None


def test_every_uploaded_log_table_is_read():
    """An operator log's device tables are those its kernel reads."""
    body = open(os.path.join(CSRC, "layout_log.h")).read()
    body = body[body.index("struct LogProgDev {"):]
    body = re.sub(r"//.*", "", body[:body.index("\n};")])
    code = re.sub(r"//.*|\w+\.\w+ = \([^;]*\)d\.\w+;", "", open(os.path.join(CSRC, "replay_log.hip")).read())
    tables = [t for line in body.splitlines() if "*" in line for t in re.findall(r"\*\s*(\w+)", line)]
    assert len(tables) > 10
    unread = [t for t in tables if not re.search(rf"\bP\.{t}\b", code)]
    assert not unread, unread


def test_groups_run_at_once_on_streams(plan):
    """Up to three groups each on a stream of its own, the first on the
    caller's if that is the default one; with more, a class's lane walks and
    sweeps share one."""
    short, long_ = W.chain_trace(100), W.chain_trace(1100)
    parts = [(0, W.H_DTR, 2), (1, W.H_DTR, 2), (0, W.H_EQ, 2), (0, W.H_LRU, 2), (0, W.H_DTR, 2, 3), (0, W.H_LRU, 2, 3),
             (0, W.H_EQ, 2, 3), (1, W.H_DTR, 2, 3)]
    for n in range(1, 9):
        rows = plan([short, long_], _batch(*parts[:n]))
        at = {r["group"]: r["stream"] for r in rows}
        assert len(rows) == n and rows[0]["stream"] == 0 and (0 not in [at[g] for g in at if g > 2])
        if n <= 3:
            assert len(set(at.values())) == n
        else:
            assert all(at[g] == at[g - 1] for g in (2, 6) if g in at and g - 1 in at)
            assert len(set(at.values())) >= 3
        mine = {r["group"]: r["stream"] for r in plan([short, long_], _batch(*parts[:n]), stream=1 << 20)}
        assert (1 << 20 in mine.values()) == (n == 1) and len(set(mine.values())) == min(n, 3)


def test_stream_sets_are_kept_for_the_next_handle(plan):
    """A handle with several groups holds four streams of its own; a few sets
    are kept for later handles, from any thread, and none that is capturing."""
    import threading
    lib, tr = plan.lib, W.chain_trace(20)
    count = lambda: (lambda v: (lib.plan_streams(v), v[0], v[1])[1:])((C.c_int64 * 2)())
    two = _batch((0, W.H_DTR, 2), (0, W.H_LRU, 2))
    plan([tr], _batch((0, W.H_DTR, 2)))
    none = count()
    handles = [plan.create([tr], two) for _ in range(10)]
    held = count()
    assert 4 * 10 - 4 * 8 <= held[0] - none[0] <= 4 * 10
    for h in handles:
        lib.dtr_sim_destroy(h)
    kept = count()
    assert kept[1] - held[1] == 4 * 2                      # eight sets are kept
    handles = [plan.create([tr], two) for _ in range(8)]
    assert count()[0] == kept[0]
    lib.plan_capture(1)
    lib.dtr_sim_destroy(handles.pop())
    lib.plan_capture(0)
    assert count()[1] == kept[1] + 4
    for h in handles:
        lib.dtr_sim_destroy(h)

    def work():
        for _ in range(50):
            mine = [plan.create([tr], two) for _ in range(2)]
            for h in mine:
                lib.dtr_sim_destroy(h)
    threads = [threading.Thread(target=work) for _ in range(4)]
    before = count()
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    after = count()
    assert after[0] - before[0] <= 4 * 400 and (after[0] - after[1]) % 4 == 0 and after[0] - after[1] <= 4 * 8
