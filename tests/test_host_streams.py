"""The host side of the two-stream backward pass, without a GPU: libspb.so runs on a stand-in for the HIP runtime
(fake_hip.cpp) that writes down every call and keeps streams on queues.  Each test is a short program of its own process."""
import os
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

PRELUDE = """
import ctypes as C, re, sys
sys.path.insert(0, {root!r})
hip = C.CDLL("libamdhip64.so.7", mode=C.RTLD_GLOBAL)
hip.fake_stream.restype, hip.fake_log.restype = C.c_void_p, C.c_char_p
hip.fake_id.argtypes, hip.fake_capture.argtypes = [C.c_void_p], [C.c_void_p, C.c_int]
hip.fake_move.argtypes = [C.c_void_p, C.c_int]
hip.fake_busy.argtypes, hip.fake_pass.argtypes = [C.c_int, C.c_double], [C.c_double]
import paper_2111_10672_amd as spb

MLP = dict(family="mlp", dtype="bf16", batch=64, dims=[64, 128, 64, 10])
ENCODER = dict(family="encoder", dtype="bf16", batch=2, seq=128, layers=2, hidden=128, heads=2, ffn=256, vocab=97, loss_rows=31)

class Model:
    def __init__(self, cfg):
        self.h = spb.spb_model_create(spb.desc_from_config(cfg))
        self.k = spb.spb_num_units(self.h)
        n = spb.spb_param_count(self.h)
        spb.spb_bind_params(self.h, [4096] * n)       # (addresses that nothing reads)
        spb.spb_bind_grads(self.h, [4096] * n)
    def forward(self, stream=None):
        spb.spb_forward(self.h, 4096, 4096, 4096, self.k, 4096, 1 << 40, 4096, stream)
    def step(self, stream=None):
        '''The step's log, and the streams (by number) that kernels of its backward pass ran on.'''
        hip.fake_clear()
        self.forward(stream)
        at = len(log())
        spb.spb_backward_truncated(self.h, self.k, stream)
        return log(), {{int(l.split()[-1]) for l in log()[at:] if l.startswith("launch")}}
    def close(self):
        spb.spb_model_destroy(self.h)

def log():
    return hip.fake_log().decode().splitlines()
def stream(queue):
    return hip.fake_stream(queue)
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    out = tmp_path_factory.mktemp("fake_hip")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-Wl,-soname,libamdhip64.so.7", os.path.join(HERE, "fake_hip.cpp"),
                    "-o", str(out / "libamdhip64.so.7")], check=True)
    return str(out)


@pytest.fixture
def run(runtime, repo_root):
    def go(program):
        env = dict(os.environ, LD_LIBRARY_PATH=runtime)
        res = subprocess.run([sys.executable, "-c", PRELUDE.format(root=repo_root) + textwrap.dedent(program)], env=env, capture_output=True, text=True, timeout=120)
        assert res.returncode == 0, res.stderr[-3000:]
    return go


def test_a_perceptron_asks_for_no_stream(run):
    """It has nothing to put on one: its forward pass makes no call but its launches, whatever stream it is given."""
    run("""
    m = Model(MLP)
    for s in (None, stream(1), stream(2)):
        hip.fake_clear()
        m.forward(s)
        assert log() and all(l.startswith("launch") for l in log()), log()
        assert m.step(s)[1] == {hip.fake_id(s)}
    """)


@pytest.mark.parametrize("spoil,mend", [("hip.fake_error(101)", "pass"), ("hip.fake_refuse_launches(1)", "hip.fake_refuse_launches(0)")])
def test_an_earlier_error_costs_no_overlap(run, spoil, mend):
    """An error that a call outside the library left behind is reported by the first step, which launches kernels, and no later
    step suffers from it; the same after launches that failed while the streams were set up."""
    run(f"""
    m, s = Model(ENCODER), stream(1)
    {spoil}
    try:
        m.forward(s)
        raise SystemExit("not reported")
    except spb.SpbError as e:
        assert e.code == -5, e
    {mend}
    for _ in range(3):
        used = m.step(s)[1]
        assert hip.fake_id(s) in used and len(used) == 2, used
        hip.fake_wait()
    """)


def test_a_pass_that_ends_in_column_sums_only_has_a_kernel_for_them(run):
    """An encoder's layer norm gradients are one launch at the pass's end, on the caller's stream, of workgroups as small as column
    sums need (those of the CNNs' mixed reductions took 3 to 5 us longer)."""
    run("""
    m, s = Model(ENCODER), stream(1)
    lines, _ = m.step(s)
    sums = [l for l in lines if "column_sums_kernel" in l]
    assert sums and all(l.endswith(f" {hip.fake_id(s)}") for l in sums) and not any("unit_reduce_kernel" in l for l in lines), lines
    """)


def test_callers_streams_share_no_side_stream(run):
    """Workers on streams of their own: neither's weight gradients wait for the other's.  Models on one stream, whose steps
    follow one another anyway, use the same side stream, and nothing stays behind."""
    run("""
    callers = [stream(0), stream(0), stream(2)]
    streams, events = hip.fake_live_streams(), hip.fake_live_events()
    models = [Model(ENCODER) for _ in range(9)]
    for _ in range(4):
        used = [m.step(callers[i % 3])[1] - {hip.fake_id(callers[i % 3])} for i, m in enumerate(models)]
        assert all(len(u) == 1 for u in used) and len(set().union(*used[6:])) == 3, used
        hip.fake_wait()
    assert used[:3] == used[3:6] == used[6:], used
    while models:
        models.pop(1 if len(models) > 1 else 0).close()
    assert (hip.fake_live_streams(), hip.fake_live_events()) == (streams, events)
    """)


def test_models_that_change_streams_leave_nothing_behind(run):
    """Two models over seven caller's streams in different orders: a model holds on to the side streams of four at most, takes
    them along where no other uses them, and a step uses one, never another caller's at that moment."""
    run("""
    streams, events = hip.fake_live_streams(), hip.fake_live_events()
    callers = [stream(q % 4) for q in range(7)] + [None]
    a, b = Model(ENCODER), Model(ENCODER)
    for step in range(400):
        for m, s in ((a, callers[step % 8]), (b, callers[step * 3 % 8])):
            side, = m.step(s)[1] - {hip.fake_id(s)}
            if s == callers[3 * step % 8] == callers[step % 8]:
                assert m is a or side == other, step
            elif m is b:
                assert side != other, step
            other = side
        hip.fake_wait()
    assert hip.fake_live_streams() - streams - 7 <= 2 * 4 * 3
    a.close(), b.close()
    assert (hip.fake_live_streams(), hip.fake_live_events()) == (streams + 7, events)
    """)


@pytest.mark.parametrize("caller", range(4))
@pytest.mark.parametrize("first", range(4))
def test_the_stream_on_another_queue_is_found(run, caller, first):
    """Wherever the caller's stream and the model's lie, from the step after the question was answered the weight gradients
    run on another queue than the caller's."""
    run(f"""
    s = stream({caller})
    hip.fake_next_queue({first})
    m, made = Model(ENCODER), []
    for step in range(4):
        lines, used = m.step(s)
        made += [int(l.split()[-1]) for l in lines if "hipStreamCreate" in l]
        side, = used - {{hip.fake_id(s)}}
        assert step == 0 or ({first} + made.index(side)) % 4 != {caller}, (step, side, made)
        hip.fake_wait()
    """)


@pytest.mark.parametrize("caller", range(4))
def test_a_first_step_makes_one_stream_and_the_caller_runs_nothing_long(run, caller):
    """A first step on a caller's stream pays for what it sets up: one stream, and further ones only if that is on the caller's
    queue.  The first step of another model there pays nothing."""
    run(f"""
    s = stream({caller})
    hip.fake_next_queue(1)
    m, made = Model(ENCODER), []
    for step in range(20):
        lines, _ = m.step(s)
        made.append(sum("hipStreamCreate" in l for l in lines))
        spun = [int(l.split()[-1]) for l in lines if "spin" in l]
        assert len(spun) <= sum(made) and hip.fake_id(s) not in spun, spun
        hip.fake_wait()
    assert made == [1, {int(caller == 1)}] + [0] * 18, made
    other = Model(ENCODER)
    lines, used = other.step(s)
    assert len(used) == 2 and not any("hipStreamCreate" in l or "spin" in l for l in lines), lines
    """)


def test_questions_are_few_however_often_the_caller_changes(run):
    run("""
    m, callers = Model(ENCODER), [stream(q % 4) for q in range(70)]
    asked = 0
    for step in range(1000):
        asked += sum("spin" in l for l in m.step(callers[step % 70])[0])
        hip.fake_wait()
    assert 0 < asked <= 4 * 3 * 9, asked    # four callers' side streams, up to three each, asked after 1, 2, 4, ... 256 calls
    """)


def test_nothing_is_set_up_while_the_caller_captures(run):
    run("""
    m, s = Model(ENCODER), stream(1)
    hip.fake_capture(s, 1)
    lines, used = m.step(s)
    assert used == {hip.fake_id(s)} and all("Create" not in l and "spin" not in l for l in lines)
    hip.fake_capture(s, 0)
    assert len(m.step(s)[1]) == 2
    hip.fake_wait()
    hip.fake_capture(s, 1)
    lines, used = m.step(s)
    assert used == {hip.fake_id(s)} and all("spin" not in l and not l.startswith(("wait", "record")) for l in lines)
    """)


@pytest.mark.parametrize("caller", range(4))
def test_a_question_met_by_busy_queues_is_asked_again(run, caller):
    """While every other queue is busy with other work (another model's, say) no stream is seen beside the caller's, which
    says nothing about the time after."""
    run(f"""
    s = stream({caller})
    hip.fake_next_queue({caller})
    m, made = Model(ENCODER), []
    for step in range(8):
        if step < 2:
            for q in range(4):
                if q != {caller}:
                    hip.fake_busy(q, 50.0)
        lines, used = m.step(s)
        made += [int(l.split()[-1]) for l in lines if "hipStreamCreate" in l]
        side, = used - {{hip.fake_id(s)}}
        hip.fake_wait()
    assert ({caller} + made.index(side)) % 4 != {caller}, (side, made)
    """)


def test_another_stream_behind_the_same_handle_is_noticed(run):
    """A destroyed stream's handle may come back for a new stream on another queue: what was known of the old one does not
    hold for good."""
    run("""
    s = stream(1)
    hip.fake_next_queue(1)
    m = Model(ENCODER)
    where = {}
    for step in range(5200):
        if step == 20:
            hip.fake_move(s, side)
        lines, used = m.step(s)
        for l in lines:
            if "hipStreamCreate" in l:
                where[int(l.split()[-1])] = (1 + len(where)) % 4
        queue, = {where[u] for u in used - {hip.fake_id(s)}}
        if step == 19:
            side = queue
        hip.fake_wait()
    assert queue != side, (queue, side)
    """)
