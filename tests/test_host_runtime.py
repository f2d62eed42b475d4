"""The host runtime's bookkeeping and order of calls, on a CPU: the library's host
code against a stand-in for the HIP runtime that reports every call and can make
one fail (hip_stub).  What cannot be seen in an image, or would need a failing
allocation or a second GPU to be seen in one, is tested here."""
import ctypes
import gc
import threading
import time

import numpy as np
import pytest

import hip_stub
from hip_stub import Watch

KV_PAIRS = 128  # (the kernel variant that reads pairs of plane elements)
DEV = 0x20      # DART_DEVICE_PTRS


@pytest.fixture(scope="module")
def dart():
    return hip_stub.load()


@pytest.fixture(autouse=True)
def _no_leftovers():
    """(stacks of the last test are freed before this one counts calls and bytes)"""
    gc.collect()


def _stack(dart, store, dims=(8, 8, 8), M=2, load=True):
    times = np.linspace(-50.0, 50.0, M)
    st = dart.dart_stack_create(dims, (1, 1, 1), times, store)
    if load:
        _fill(dart, st, 0, M)
    return st


def _fill(dart, st, m0, count):
    """A load from device memory (addresses that the stand-in never reads)."""
    dart._check(dart._load().dart_stack_set_epochs(st.handle, m0, count, dart.DART_F32, 4096, 8192,
                                                   DEV, None))


def _view(dart, P=32, flags=0, theta=30.0, out=None):
    return dart.View(theta, 40.0, P, P, 8.0 / P, 0.0, 0.6, flags,
                     dart.DART_F32 if out is None else out)


def _variants(w):
    return [c[2] or 0 for c in w.of("launch_batch")]


def test_failed_refill_leaves_no_pairs(dart):
    """A refill that ends in DART_E_RANGE has written records: batches read neither
    the pairs nor plans made of the old ones."""
    st = _stack(dart, dart.DART_F16)
    big = [_view(dart, 8192, DEV)] * 2  # 1.6e9 cells each by the pairs' rule

    def batch():
        with Watch(dart) as w:
            dart.dart_render_batch([st] * 2, big, [4096, 8192], stats=False)
        return w

    while not any(v & KV_PAIRS for v in _variants(batch())):
        pass
    dart.stub.stub_bad_element(5)
    with pytest.raises(dart.DartError) as ei:
        _fill(dart, st, 0, 1)
    assert ei.value.status == dart.DART_E_RANGE
    w = batch()
    assert w.of("launch_pack_jplane") and not any(v & KV_PAIRS for v in _variants(w))


class _Held:
    """A server whose waves stay in flight until `finish`."""

    def __init__(self, dart, streams=3):
        self.dart = dart
        dart.stub.stub_hold_host_funcs(1)
        self.srv = dart.dart_server_create(64 << 20, 16, streams)
        self.tickets = []

    def submit(self, st, view, image):
        """Sends a request and waits until its wave is on its way."""
        waves = self.dart.dart_server_get_stats(self.srv).waves
        t = ctypes.c_uint64(0)
        v = view.c()
        self.dart._check(self.dart._load().dart_submit(self.srv.handle, st.handle, ctypes.byref(v),
                                                       image, ctypes.byref(t)))
        self.tickets.append(t.value)
        deadline = time.time() + 20
        while self.dart.dart_server_get_timeline(self.srv).enqueue_ms == self._enqueued or \
                self.dart.dart_server_get_stats(self.srv).waves == waves:
            assert time.time() < deadline
            time.sleep(1e-3)
        self._enqueued = self.dart.dart_server_get_timeline(self.srv).enqueue_ms

    _enqueued = 0.0

    def finish(self):
        self.dart.stub.stub_hold_host_funcs(0)
        self.dart.stub.stub_run_host_funcs()
        for t in self.tickets:
            self.dart.dart_wait(self.srv, t)
        self.dart.dart_server_destroy(self.srv)


def test_requests_with_one_destination_write_it_in_order(dart):
    """Of the waves in flight with one device destination, the first renders into it
    and each later one copies behind the one before."""
    st = _stack(dart, dart.DART_F16)
    dest, other = 1 << 20, 2 << 20
    held = _Held(dart)
    with Watch(dart) as w:
        for im in (dest, dest, dest):
            held.submit(st, _view(dart, 32, DEV), im)
    held.finish()
    copies = [k for k, c in enumerate(w.calls) if c[0] == "hipMemcpyAsync" and c[1] == dest]
    assert len(copies) == 2  # (the second and the third)
    streams = [c[1] for c in w.of("launch_totals")]
    assert len(set(streams)) == 3
    ends = {}  # the last event of each wave's stream, behind its copies and totals
    for k, c in enumerate(w.calls):
        if c[0] == "launch_totals":
            ends[c[1]] = next(e[1] for e in w.calls[k:] if e[0] == "hipEventRecord")
    order = [c[1] for c in w.of("launch_totals")]
    for n, k in enumerate(copies):
        mine, before = w.calls[k][2], order[n]
        assert ("hipStreamWaitEvent", mine, ends[before]) in w.calls[:k]
    # once they are done the destination is rendered into again
    held = _Held(dart)
    with Watch(dart) as w:
        for im in (dest, other):
            held.submit(st, _view(dart, 32, DEV), im)
    held.finish()
    assert not w.of("hipMemcpyAsync") and not w.of("hipStreamWaitEvent")


def test_failed_call_leaves_no_plan(dart):
    """A batch that fails between its plan and its descriptors' upload is planned and
    uploaded again by the next equal call."""
    st = _stack(dart, dart.DART_F32)
    n = 24
    views = [_view(dart, 32, DEV)] * n
    images = [(k + 1) << 20 for k in range(n)]
    failed = []

    def answer(name, a, b):
        if name == "hipHostMalloc" and a == 16 * n and not failed:  # (the totals)
            failed.append(name)
            return 2
        return 0

    with Watch(dart, answer) as w:
        with pytest.raises(dart.DartError):
            dart.dart_render_batch([st] * n, views, images)
    assert failed and not w.of("launch_batch")
    with Watch(dart) as w:
        dart.dart_render_batch([st] * n, views, images)
    begins = [k for k, c in enumerate(w.calls) if c[0] == "launch_begin" and c[1]]
    assert begins and begins[0] < w.names().index("launch_batch")


def test_batch_is_refused_under_capture(dart):
    """A new plan's descriptors are staged by the library: a call on a stream that its
    caller captures is refused and enqueues nothing, with and without totals."""
    st = _stack(dart, dart.DART_F32)
    im = [1 << 20]
    dart.dart_render_batch([st], [_view(dart, 32, DEV)], im, stream=4096, stats=False)
    for stats in (False, True):
        for stream in (4097, 4099):  # (odd: under capture)
            with Watch(dart) as w:
                with pytest.raises(dart.DartError) as ei:
                    dart.dart_render_batch([st], [_view(dart, 32, DEV)], im, stream=stream,
                                           stats=stats)
            assert ei.value.status == dart.DART_E_DEVICE
            assert not [c for c in w.calls if c[0].startswith("launch_") or c[0] in
                        ("hipMemcpyAsync", "hipEventRecord", "hipStreamBeginCapture")]


@pytest.mark.parametrize("kind", ["vector", "labelled"])
def test_holder_freed_beside_a_load(dart, kind):
    """A load into a part waits for its holders' renders: a holder lets go of its parts
    before its events end."""
    parts = [_stack(dart, dart.DART_F32) for _ in range(2)]
    for k, p in enumerate(parts):
        dart.dart_stack_set_placement(p, (0, 0, 8 * k if kind == "labelled" else 0), (4, 4, 8))
    holder = (dart.dart_vector_create if kind == "vector" else dart.dart_labelled_create)(parts)
    for _ in range(2):  # (the second packs the planes, which loads then keep in step)
        dart.dart_render_batch([holder], [_view(dart, 32, DEV)], [1 << 20], stats=False)
    dead = []

    def answer(name, a, b):
        if name == "hipEventDestroy" and not dead:
            dead.append(a)
            _fill(dart, parts[0], 0, 1)  # (another thread's load, just now)
        if name == "hipEventSynchronize":
            assert dart.stub.stub_event_alive(a)
        return 0

    with Watch(dart, answer) as w:
        dart.dart_free_epochs(holder)
    assert dead and w.of("launch_convert")
    assert dead[0] not in [c[1] for c in w.of("hipEventSynchronize")]
    for p in parts:
        dart.dart_free_epochs(p)


def test_destination_on_another_gpu_is_copied_to(dart):
    """Only memory of the server's own GPU is rendered into."""
    st = _stack(dart, dart.DART_F16)
    far = 1 << 60  # (the stand-in's second GPU)
    held = _Held(dart)
    with Watch(dart) as w:
        held.submit(st, _view(dart, 32, DEV), far)
        held.submit(st, _view(dart, 32, DEV), 1 << 20)
    held.finish()
    assert [c[1] for c in w.of("hipMemcpyAsync")] == [far]


def test_a_streamers_ring_has_no_plane(dart):
    """A streamed window reads whole records: its FP64 ring is allocated without the
    emissivity plane that an FP64 stack of its size has."""
    dims, M = (128, 128, 160), 5
    times = np.linspace(-50.0, 50.0, M)
    held = dart.stub.stub_held()
    sm = dart.dart_streamer_create(dims, (1, 1, 1), times, dart.DART_F64, ring_epochs=4)
    ring = 4 * int(np.prod(dims)) * 32  # 335 MB
    assert ring <= dart.stub.stub_held() - held < ring + (1 << 20)
    dart.dart_streamer_destroy(sm)
    assert dart.stub.stub_held() == held
    st = dart.dart_stack_create(dims, (1, 1, 1), times[:4], dart.DART_F64)
    assert dart.stub.stub_held() - held > ring * 5 // 4
    dart.dart_free_epochs(st)


def test_labelled_parts_without_planes_are_not_packed(dart):
    """Sub-domains one of which has no plane (FP64, at most 256 MiB) are read as whole
    records: the planes of the others are not packed, call after call, for nothing."""
    M = 4
    dart.stub.stub_room(dart.stub.stub_held() + (900 << 20))  # (none at creation either)
    try:
        big, small = (_stack(dart, dart.DART_F64, d, M) for d in ((128, 128, 160), (8, 8, 8)))
    finally:
        dart.stub.stub_room(256 << 30)
    for k, p in enumerate((big, small)):
        dart.dart_stack_set_placement(p, (0, 0, 160 * k), (64, 64, 84))
    for parts in ((big, small), (small, big)):
        st = dart.dart_labelled_create(parts)
        with Watch(dart) as w:
            for k in range(4):
                dart.dart_render_batch([st], [_view(dart, 32, DEV, 30.0 + k)], [1 << 20], stats=False)
        assert len(w.of("launch_batch")) == 4 and not w.of("launch_pack_jplane")
        dart.dart_free_epochs(st)


def test_labelled_planes_packed_before_an_error_are_used(dart):
    """Planes whose packing was enqueued before a later part's failed are packed once."""
    parts = [_stack(dart, dart.DART_F32) for _ in range(3)]
    for k, p in enumerate(parts):
        dart.dart_stack_set_placement(p, (0, 0, 8 * k), (4, 4, 12))
    st = dart.dart_labelled_create(parts)
    packs = []

    def answer(name, a, b):
        if name == "launch_pack_jplane":
            packs.append(a)
            return 1 if len(packs) == 3 else 0
        return 0

    call = lambda k: dart.dart_render_batch([st], [_view(dart, 32, DEV, 30.0 + k)], [1 << 20],
                                            stats=False)
    with Watch(dart, answer):
        call(0)
        with pytest.raises(dart.DartError):
            call(1)
        call(2)
        call(3)
    assert len(packs) == 4 and packs[3] == packs[2] and len(set(packs)) == 3


def test_tuning_times_no_capture(dart):
    """The replays that the tuner times are graph launches: the graph is captured by the
    warm-up call, as many calls as there were replays and one."""
    st = _stack(dart, dart.DART_F32)
    with Watch(dart) as w:
        dart.dart_autotune([st], [_view(dart, 32)], stream=4096)
    # between the two timing events of a replay
    n = w.names()
    timed = [k for k, c in enumerate(w.calls) if c[0] == "hipGraphLaunch"]
    assert len(timed) > 100
    begin = None
    for k, c in enumerate(w.calls):
        if c[0] == "hipEventElapsedTime":
            end = max(q for q in range(k) if n[q] == "hipEventSynchronize")
            start = max(q for q in range(end) if n[q] == "hipGraphLaunch")
            first = max(q for q in range(start) if n[q] == "hipEventRecord")
            assert "hipGraphInstantiate" not in n[first:end]
            begin = first
    assert begin is not None
    # a tuned stack's next new plan is launched kernel by kernel
    with Watch(dart) as w:
        dart.dart_render_batch([st], [_view(dart, 32, DEV, 77.0)], [1 << 20], stream=4096, stats=False)
    assert "hipGraphInstantiate" not in w.names() and w.of("launch_batch")
    dart.dart_free_epochs(st)


def test_pairs_of_a_served_stack_are_packed_beside_the_caller(dart):
    """dart_submit packs due pairs on a stream of the server's, not behind what the
    caller's blocking streams hold; a request that is refused counts for nothing."""
    st = _stack(dart, dart.DART_F16, (512, 512, 512))
    srv = dart.dart_server_create(64 << 20, 4, 1)
    with Watch(dart) as w:
        for flags, n in ((DEV | dart.DART_ACCUMULATE, 40), (DEV, 12)):  # 8.05e8 cells each, 8.3e9
            for k in range(n):                                        # make them due
                v, t = _view(dart, 1024, flags).c(), ctypes.c_uint64(0)
                rc = dart._load().dart_submit(srv.handle, st.handle, ctypes.byref(v), 1 << 20,
                                              ctypes.byref(t))
                assert (rc == dart.DART_OK) == (flags == DEV)
                if rc == dart.DART_OK:
                    dart.dart_wait(srv, t.value)
            if flags != DEV:
                assert not w.of("launch_pack_pairs")
    packs = w.of("launch_pack_pairs")
    assert len(packs) == 1 and packs[0][2]
    assert ("hipStreamSynchronize", packs[0][2], None) in w.calls
    plane = w.names().index("launch_pack_jplane")  # (the plane's own pack is the only other wait)
    assert [c[1] for c in w.calls[plane:] if c[0] == "hipStreamSynchronize"].count(None) == 1
    streams = {c[1] for c in w.of("launch_totals")}
    assert packs[0][2] not in streams
    dart.dart_server_destroy(srv)
    dart.dart_free_epochs(st)


def test_planning_a_wave_waits_for_no_refresh(dart):
    """While a caller uploads a labelled stack's planes (and may wait for renders with the
    stack locked), the server plans a wave of that stack and answers."""
    parts = [_stack(dart, dart.DART_F32) for _ in range(2)]
    for k, p in enumerate(parts):
        dart.dart_stack_set_placement(p, (0, 0, 8 * k), (4, 4, 8))
    st = dart.dart_labelled_create(parts)
    plain = _stack(dart, dart.DART_F32)
    dart.stub.stub_hold_host_funcs(1)
    srv = dart.dart_server_create(64 << 20, 1, 2)
    tickets, seen = [], []

    def submit(s):
        v, t = _view(dart, 32, DEV).c(), ctypes.c_uint64(0)
        dart._check(dart._load().dart_submit(srv.handle, s.handle, ctypes.byref(v),
                                             (len(tickets) + 1) << 20, ctypes.byref(t)))
        tickets.append(t.value)

    def second_wave():
        while dart.dart_server_get_stats(srv).waves < 2:
            time.sleep(1e-3)
        seen.append("planned")

    def answer(name, a, b):
        if name == "hipMemcpyAsync" and not seen:  # (the blocks, with their planes)
            seen.append("refreshing")
            dart.stub.stub_run_host_funcs()  # (the first wave ends: the queued request is next)
            t = threading.Thread(target=second_wave, daemon=True)
            t.start()
            t.join(5.0)
        return 0

    submit(plain)
    while dart.dart_server_get_stats(srv).waves < 1:
        time.sleep(1e-3)
    submit(st)
    with Watch(dart, answer):
        dart.dart_render_batch([st], [_view(dart, 32, DEV)], [5 << 20], stats=False)
    during = list(seen)
    dart.stub.stub_hold_host_funcs(0)
    for _ in range(200):
        dart.stub.stub_run_host_funcs()
        time.sleep(1e-3)
    for t in tickets:
        dart.dart_wait(srv, t)
    dart.dart_server_destroy(srv)
    assert during == ["refreshing", "planned"]


def test_noalloc_queues_segments_where_they_fit(dart):
    """The allocation-free batch marches the depth segments of small views at once, in the
    scratch that their descriptors leave, and a batch too large for that in sequence."""
    st = _stack(dart, dart.DART_F32, (64, 64, 64))
    one = dart.View(30.0, 40.0, 128, 128, 1.0, 0.0, 0.6, DEV)
    for n, by_segment in ((1, True), (4, True), (20000, False)):
        images = [(k + 1) << 20 for k in range(n)]
        view = one if n < 100 else dart.View(30.0, 40.0, 16, 16, 8.0, 0.0, 0.6, DEV)
        with Watch(dart) as w:
            dart.dart_render_batch_noalloc([st] * n, [view] * n, images, stats=False)
        (_, parts, tiles), = w.of("launch_batch parts")
        assert (parts is not None) == by_segment
        assert not w.of("hipMalloc")
