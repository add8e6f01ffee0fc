"""The library's side streams: callers on different streams, captures and calls
that may create nothing neither wait for each other nor disturb each other."""

import ctypes
import threading

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_1302_2669_amd as mc  # noqa: E402
from paper_1302_2669_amd import _lib  # noqa: E402

DEV = "cuda"
SIDES = 4            # per device, at most
# a batch of both mappings: 2.4 waves of 64 chains on each SIMD of 256 CUs
BOTH = dict(L=9, n=10000, p=0.10, sweeps=40, chains=4)


def setup_module(module):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")


def side_of(stream, may_create=True, in_capture=True):
    """Handle of the side stream that a caller on `stream` gets, None if none."""
    side = ctypes.c_void_p()
    st = _lib._lib().mcmc_side_stream_of(ctypes.c_void_p(stream.cuda_stream), int(may_create),
                                         int(in_capture), ctypes.byref(side))
    assert st == 0, _lib.STATUS.get(st, st)
    return side.value


def keep_busy(stream):
    """Some hundred milliseconds of work on `stream`."""
    with torch.cuda.stream(stream):
        x = torch.ones((8192, 8192), device=DEV)
        for _ in range(40):
            x = x @ x * 1e-4
        done = torch.cuda.Event()
        done.record()
    return done


def batch(L, n, p, sweeps, chains, seed=5):
    syn, _, _ = mc.sample_errors(L, p, seed, n, device=DEV)
    return lambda: mc.decode_batch(syn, L, p, sweeps, seed, chains=chains, want_sums=True,
                                   want_correction=True)


def assert_equal(got, want):
    for k in ("chosen", "correction", "sum_n", "accepts", "class_prob"):
        assert torch.equal(got[k], want[k]), k


def test_a_stream_does_not_take_what_another_still_uses():
    a, b, c = (torch.cuda.Stream() for _ in range(3))
    torch.cuda.synchronize()
    done = keep_busy(a)
    side_a = side_of(a)
    side_b = side_of(b)
    side_c = side_of(c, may_create=False)
    again = side_of(a)
    assert not done.query()          # all of it while a's work was pending
    assert side_a and side_b and side_b != side_a
    assert side_c != side_a          # none at all, or a free one
    assert again == side_a
    torch.cuda.synchronize()
    assert side_of(c, may_create=False) is not None


def test_side_streams_are_bounded():
    streams = [torch.cuda.Stream() for _ in range(SIDES + 2)]
    torch.cuda.synchronize()
    done = keep_busy(streams[0])
    for s in streams[1:]:
        s.wait_event(done)
    sides = [side_of(s) for s in streams]
    assert not done.query()
    held = [s for s in sides if s is not None]
    assert len(held) == len(set(held)) == SIDES
    assert sides[SIDES:] == [None, None]
    torch.cuda.synchronize()


def test_concurrent_batches_of_both_mappings():
    runs = [batch(**BOTH, seed=5), batch(**BOTH, seed=6)]
    alone = [{k: v.clone() for k, v in r().items() if torch.is_tensor(v)} for r in runs]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    got, errors = [None, None], []

    def worker(k):
        try:
            with torch.cuda.stream(streams[k]):
                for _ in range(4):
                    o = runs[k]()
                streams[k].synchronize()
                got[k] = o
        except Exception as e:  # noqa: BLE001 - reported below
            errors.append(e)

    threads = [threading.Thread(target=worker, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for k in range(2):
        assert_equal(got[k], alone[k])


def test_batch_of_both_mappings_without_a_free_side_stream():
    # every side stream busy with another stream's work: one mapping, same outputs
    run = batch(**BOTH)
    want = {k: v.clone() for k, v in run().items() if torch.is_tensor(v)}
    streams = [torch.cuda.Stream() for _ in range(SIDES)]
    mine = torch.cuda.Stream()
    torch.cuda.synchronize()
    done = keep_busy(streams[0])
    for s in streams[1:]:
        s.wait_event(done)
    for s in streams:
        side_of(s)
    with torch.cuda.stream(mine):
        got = run()
    pending = not done.query()
    torch.cuda.synchronize()
    assert pending
    assert_equal(got, want)


def test_batch_of_both_mappings_in_a_capture():
    run = batch(**BOTH)
    want = {k: v.clone() for k, v in run().items() if torch.is_tensor(v)}
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode="thread_local"):
        got = run()
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert_equal(got, want)
        assert_equal(run(), want)    # eager work between the replays
        torch.cuda.synchronize()


@pytest.mark.parametrize("L,n", [(13, 700), (18, 3100)])
def test_two_captures_at_once(L, n):
    # the matching starts fork a side stream (two in large batches) into a capture: a
    # second capture, and eager calls beside both, take others or none
    sets = [mc.sample_errors(L, 0.18, 40 + k, n, device=DEV)[0] for k in range(3)]
    nq = mc.geometry(L)[0]
    want = [mc.init_representatives(s, L, mc.MCMC_INIT_MWPM).clone() for s in sets]
    out = [torch.zeros((n, 4, nq), dtype=torch.uint8, device=DEV) for _ in range(3)]
    streams = [torch.cuda.Stream() for _ in range(3)]
    for s in streams[:2]:
        side_of(s)
    torch.cuda.synchronize()

    def starts(k):
        return _lib._lib().mcmc_init_representatives(
            L, mc.MCMC_INIT_MWPM, ctypes.c_void_p(sets[k].data_ptr()), n,
            ctypes.c_void_p(out[k].data_ptr()), ctypes.c_void_p(streams[k].cuda_stream))

    graphs = [torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()]
    status = []
    for k in range(2):
        with torch.cuda.stream(streams[k]):
            graphs[k].capture_begin(capture_error_mode="thread_local")
            status.append(starts(k))
            status.append(starts(k))                 # the same capture again
    status.append(starts(2))                         # eager, beside both
    for k in range(2):
        with torch.cuda.stream(streams[k]):
            graphs[k].capture_end()
    assert status == [0] * 5
    torch.cuda.synchronize()
    assert torch.equal(out[2], want[2])
    for _ in range(3):
        for k in range(2):
            out[k].zero_()
            graphs[k].replay()
            torch.cuda.synchronize()
            assert torch.equal(out[k], want[k]), k
            assert torch.equal(mc.init_representatives(sets[k], L, mc.MCMC_INIT_MWPM), want[k])
    torch.cuda.synchronize()
