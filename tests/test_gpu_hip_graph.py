"""nomad_epoch only enqueues kernels on the caller's stream, so a caller can record a run of epochs into a HIP graph
and replay it: the launch-bound small configurations then pay one graph launch instead of two kernel launches per
epoch.  Replays are checked against the eager run, several times, with eager work in between."""
import numpy as np
import pytest
import torch

from paper_2505_15511_amd import Nomad, SCATTER_ATOMIC, SCATTER_DETERMINISTIC, workloads

pytestmark = pytest.mark.gpu


def _case(name):
    if name == "config1":
        return workloads.make_config(1)
    if name == "config3@0.02-groups":
        return workloads.make_config(3, scale=0.02, n_groups=4)
    w = workloads.make_config(3, scale=0.02)
    w.pool_size, w.pool_block = 512, 2048
    return w


@pytest.mark.parametrize("case", ["config1", "config3@0.02-groups", "config3@0.02-pooled"])
def test_recorded_epochs_replay_like_the_eager_run(case):
    w = _case(case)
    T = 12
    theta0 = w.theta0.cuda()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        nm = Nomad.from_workload(w, SCATTER_DETERMINISTIC, stream=side.cuda_stream)
        for t in range(T):                       # eager run
            nm.epoch(t)
        side.synchronize()
        th_eager, g_eager = nm.get_embedding(), nm.get_gradient()
        nm.set_embedding(theta0)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            for t in range(T):
                nm.epoch(t)
        for replay in range(3):
            nm.set_embedding(theta0)             # eager work between the replays
            if replay == 1:
                nm.epoch(0)
                nm.loss(3)
                nm.set_embedding(theta0)
            graph.replay()
            side.synchronize()
            assert np.array_equal(nm.get_embedding(), th_eager), replay
            assert np.array_equal(nm.get_gradient(), g_eager), replay
        nm.close()


def test_recorded_epochs_in_atomic_mode_stay_within_the_bar():
    w = workloads.make_config(1)
    T = 8
    theta0 = w.theta0.cuda()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        ref = Nomad.from_workload(w, SCATTER_DETERMINISTIC, stream=side.cuda_stream)
        nm = Nomad.from_workload(w, SCATTER_ATOMIC, stream=side.cuda_stream)
        # The bar: every epoch's gradient within 1e-5 of its largest component (the atomic path's bar), so positions within the
        # sum of eta_t times that: 2.8e-4 here.  Forty eager runs ended 1.9e-5 to 7.4e-5 apart, a later one 1.04e-4.
        bar = 0.0
        for t in range(T):
            ref.epoch(t)
            bar += 1e-5 * w.lr0 * (1.0 - t / w.n_epochs) * float(np.abs(ref.get_gradient()).max())
        nm.epoch(0)
        nm.set_embedding(theta0)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            for t in range(T):
                nm.epoch(t)
        for _ in range(2):
            nm.set_embedding(theta0)
            graph.replay()
            side.synchronize()
            assert np.abs(nm.get_embedding() - ref.get_embedding()).max() < bar
        nm.close()
        ref.close()


def test_results_wait_for_the_work_their_memory_still_has():
    """A context on a side stream, called outside of it: the result's block was freed with work on the default stream pending."""
    w = workloads.make_config(3, scale=0.2)
    side = torch.cuda.Stream()
    nm = Nomad.from_workload(w, SCATTER_DETERMINISTIC, stream=side.cuda_stream)
    nm.epoch(0)
    theta, g = nm.get_embedding(), nm.get_gradient()
    nodes = torch.empty(1 << 26, device="cuda")
    for get, want in ((nm.get_embedding, theta), (nm.get_gradient, g)):
        block = torch.empty(w.n, 2, device="cuda")
        for _ in range(40):
            nodes.normal_()                      # some milliseconds ahead of the write below
        block.fill_(7.0)
        del block
        out = get(device=True)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), want)
    # inputs made on the current stream: a conversion that has not run yet
    for _ in range(40):
        nodes.normal_()
    nm.set_embedding(torch.from_numpy(theta).cuda().double() + 1.0)
    assert np.array_equal(nm.get_embedding(), theta + np.float32(1.0))
    nm.close()


@pytest.mark.parametrize("ending", ["close", "set_graph"])
def test_memory_is_given_back_when_replays_on_other_streams_have_ended(ending):
    w = workloads.make_config(3, scale=0.02)
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(side):
        nm = Nomad.from_workload(w, SCATTER_DETERMINISTIC, stream=side.cuda_stream)
        nm.epoch(0)
        want = nm.get_embedding()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            nm.epoch(1)
        side.synchronize()
    with torch.cuda.stream(other):
        for _ in range(300):
            graph.replay()
        if ending == "close":
            nm.close()
        else:
            nm.set_graph(w.row_ptr, w.col_idx, w.weights, w.cluster_of, w.cluster_group)
        assert other.query()
    fresh = Nomad.from_workload(w, SCATTER_DETERMINISTIC)
    fresh.epoch(0)
    assert np.array_equal(fresh.get_embedding(), want)
    fresh.close()
    nm.close()


@pytest.mark.parametrize("grouped", [False, True])
def test_device_buffers_of_a_context_on_a_side_stream(grouped):
    """Graph, embedding, means and mean-field sums as device buffers: copies complete before they are used or returned."""
    import ctypes as C
    w = workloads.make_config(3, scale=0.02, n_groups=4 if grouped else None)
    side = torch.cuda.Stream()
    dev = {k: None if getattr(w, k) is None else torch.as_tensor(getattr(w, k)).cuda() for k in ("row_ptr", "col_idx", "weights", "cluster_of", "cluster_group")}
    theta = torch.as_tensor(w.theta0).cuda()
    ref = Nomad.from_workload(w)
    nm = Nomad.from_workload(w, stream=side.cuda_stream)
    nm.set_graph(*dev.values())
    nm.set_embedding(theta)
    mu, A, B = (torch.full(shape, 7.0, device="cuda") for shape in ((nm.R, 2), (nm.n,), (nm.n, 2)))
    counts = torch.zeros(nm.R, dtype=torch.int64, device="cuda")
    nm._check(nm.lib.nomad_get_means(nm.ctx, C.c_void_p(mu.data_ptr()), C.c_void_p(counts.data_ptr()), 1))
    nm._check(nm.lib.nomad_get_mean_field(nm.ctx, C.c_void_p(A.data_ptr()), C.c_void_p(B.data_ptr()), 1))
    with torch.cuda.stream(torch.cuda.Stream()):         # a reader that no stream of the calls is ordered with
        got = [t.cpu().numpy() for t in (mu, counts, A, B)]
    for a, b in zip(got, (*ref.get_means(), *ref.get_mean_field())):
        assert np.array_equal(a, b)
    nm.epoch(0)
    ref.epoch(0)
    assert np.array_equal(nm.get_embedding(), ref.get_embedding())
    assert np.array_equal(nm.get_negatives(3, 10, 5_000, device=True).cpu().numpy(), ref.get_negatives(3, 10, 5_000))
    nm.close()
    ref.close()
