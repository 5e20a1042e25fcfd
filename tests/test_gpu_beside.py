"""Which parts of a call run at the same time must not show in its results.

The full-loss call whose two passes run at the same time (small batches) against the two
calls one after the other: the same bits, also with empty sequences in the batch, from another
stream than the default one and replayed from a HIP graph."""
import numpy as np
import pytest

from paper_2005_09824_amd import binding, workloads

pytestmark = pytest.mark.gpu


def _den_graph(pdf_by_state, seed):
    rng = np.random.default_rng(seed)
    if pdf_by_state:
        return workloads.hmm_den_graph(rng, 14, 6, 0.5)
    return workloads.random_den_graph(rng, 700, 5, 28, 0.5)


def _setup(B, pdf_by_state, seed, empty=False):
    import torch
    rng = np.random.default_rng(seed)
    den = _den_graph(pdf_by_state, seed)
    P = den["num_pdfs"]
    num = [workloads.phone_string_num_graph(rng.integers(1, P // 2, size=int(n)), P)
           for n in rng.integers(4, 14, size=B)]
    lens = rng.integers(30, 90, size=B).astype(np.int32)
    if B < 8:
        lens[0] = 256  # fewer sequences run at the same time from 256 frames on
    if empty:
        lens[B // 2] = 0
    x = torch.from_numpy(rng.normal(0, 2, size=(B, lens.max() + 5, P)).astype(np.float32)).cuda()
    return binding.lfmmi_graph_create_batch(num), binding.lfmmi_graph_create(den), x, lens


def _in_turn(num, den, x, lens):
    objf, grad, st = binding.lfmmi_forward_backward(num, x, lens, 1e-5, 1.0, False)
    binding.lfmmi_forward_backward(den, x, lens, 1e-5, -1.0, True, objf, grad, st)
    return objf, grad, st


# A denominator whose numerators run at the same time takes 8 bytes a sequence more for what its
# recursion leaves aside: whether they did shows in the workspace of a fresh handle.
def _den_workspace(num, den_graph, x, lens, out, monkeypatch, beside):
    import torch
    monkeypatch.setenv("LFMMI_BESIDE", beside)
    den = binding.lfmmi_graph_create(den_graph)
    binding.lfmmi_loss(num, den, x, lens, 1e-5, *out)
    torch.cuda.synchronize()
    n = binding.lfmmi_graph_info(den)["workspace_bytes"]
    den.close()
    monkeypatch.delenv("LFMMI_BESIDE")
    return n


# 64 sequences: the largest batch whose 4 B workgroups fit 256 compute units; 65: one more
@pytest.mark.parametrize("B,pdf_by_state,empty", [(1, False, False), (1, True, False), (9, True, True),
                                                  (7, False, False), (8, True, False), (64, True, False),
                                                  (64, False, False), (65, True, False)])
def test_same_bits_as_the_two_passes_in_turn(B, pdf_by_state, empty, monkeypatch):
    import torch
    num, den, x, lens = _setup(B, pdf_by_state, 100 + B, empty)
    want = _in_turn(num, den, x, lens)
    torch.cuda.synchronize()
    out = (torch.full_like(want[0], 7.0), torch.full_like(want[1], -3.0), torch.full_like(want[2], 5))
    for stream in (torch.cuda.current_stream(), torch.cuda.Stream()):
        for t in out:
            t.fill_(9)
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            for _ in range(3):
                binding.lfmmi_loss(num, den, x, lens, 1e-5, *out)
            got = [t.clone() for t in out]
        torch.cuda.synchronize()
        for a, b in zip(got, want):
            assert torch.equal(a, b)
    g = _den_graph(pdf_by_state, 100 + B)
    more = [_den_workspace(num, g, x, lens, out, monkeypatch, v) for v in "01"]
    assert (more[1] > more[0]) == (B <= 64 and not empty)
    num.close()
    den.close()


# A NaN logit, an utterance too short for its numerator, both and neither, with the status asked
# for and not: what the denominator's pass leaves aside meets what the numerators' pass wrote,
# in every kernel that adds it: by state, by arc with planes, one frame at a time, fp64
@pytest.mark.parametrize("kind", ["by_state", "by_arc", "frame_at_a_time", "fp64"])
def test_flagged_sequences_side_by_side(kind, monkeypatch):
    import torch
    if kind == "frame_at_a_time":
        monkeypatch.setenv("LFMMI_OCC_MULTI", "0")
    num, den, x, lens = _setup(10, kind == "by_state", 77)
    if kind == "fp64":
        g = _den_graph(False, 77)
        g["final_prob"][::3] = 0
        den.close()
        den = binding.lfmmi_graph_create(g)
        assert binding.lfmmi_graph_info(den)["fp64"] == 1
    lens[[2, 6]] = 2  # two frames: no path through four phones or more
    x[3, 5, 4] = float("nan")
    x[6, 1, 0] = float("nan")
    want = _in_turn(num, den, x, lens)
    torch.cuda.synchronize()
    st = want[2].cpu().numpy()
    assert st[2] & 1 and st[3] & 2 and st[6] & 2 and np.all(np.delete(st, [2, 3, 6]) == 0)
    for status in (torch.full_like(want[2], 5), None):
        out = [torch.full_like(want[0], 9.0), torch.full_like(want[1], 9.0), status]
        if status is None:  # (the wrapper would make one)
            import ctypes
            assert binding.load_library().lfmmi_loss(
                num.handle, den.handle, ctypes.c_void_p(x.data_ptr()), ctypes.c_void_p(lens.ctypes.data),
                *x.shape, 1e-5, ctypes.c_void_p(out[0].data_ptr()), ctypes.c_void_p(out[1].data_ptr()),
                None, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
        else:
            binding.lfmmi_loss(num, den, x, lens, 1e-5, *out)
        torch.cuda.synchronize()
        for a, b in zip(out, want):
            if a is not None:
                assert np.array_equal(a.cpu().numpy(), b.cpu().numpy(), equal_nan=a.dtype.is_floating_point)
    num.close()
    den.close()


def test_replays_from_a_hip_graph():
    import torch
    num, den, x, lens = _setup(6, True, 5)
    want = _in_turn(num, den, x, lens)
    out = tuple(torch.empty_like(t) for t in want)
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        binding.lfmmi_loss(num, den, x, lens, 1e-5, *out)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=side, capture_error_mode="relaxed"):
            binding.lfmmi_loss(num, den, x, lens, 1e-5, *out)
    for _ in range(3):
        for t in out:
            t.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(out, want):
            assert torch.equal(a, b)
        binding.lfmmi_loss(num, den, x, lens, 1e-5, *out)  # eager work between the replays
        torch.cuda.synchronize()
    del graph
    num.close()
    den.close()


# Fewer than four sequences need no stream of the library's under capture: while one thread
# captures such a call, another one's eager call runs on those streams
def test_a_captured_call_of_few_sequences_stays_on_its_stream():
    import threading
    import torch
    num, den, x, lens = _setup(2, True, 6)
    eager = binding.lfmmi_graph_create(workloads.random_den_graph(np.random.default_rng(3), 500, 5, 40, 0.5))
    ex = torch.zeros((12, 400, 40), device="cuda")
    want_e = binding.lfmmi_forward_backward(eager, ex, np.full(12, 400, np.int32), 1e-5)
    want = _in_turn(num, den, x, lens)
    out = tuple(torch.empty_like(t) for t in want)
    out_e = tuple(torch.empty_like(t) for t in want_e)
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    other = torch.cuda.Stream()
    errors = []

    def eager_call():
        try:
            with torch.cuda.stream(other):
                binding.lfmmi_forward_backward(eager, ex, np.full(12, 400, np.int32), 1e-5, 1.0, False, *out_e)
        except Exception as e:  # reported below, on the test's own thread
            errors.append(e)

    with torch.cuda.stream(side):
        binding.lfmmi_loss(num, den, x, lens, 1e-5, *out)
        torch.cuda.synchronize()
        graph.capture_begin(capture_error_mode="thread_local")
        try:
            binding.lfmmi_loss(num, den, x, lens, 1e-5, *out)
            t = threading.Thread(target=eager_call)
            t.start()
            t.join()
        finally:
            graph.capture_end()
    assert not errors
    for _ in range(3):
        for t in out:
            t.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(out + out_e, want + want_e):
            assert torch.equal(a, b)
    del graph
    for h in (num, den, eager):
        h.close()


# 90 frames: one bucket by default; 330: four (500 states, 3,000 arcs); both against every count
@pytest.mark.parametrize("T", [90, 330])
def test_bucket_counts_give_the_same_bits_eager_and_replayed(T, monkeypatch):
    import torch
    rng = np.random.default_rng(T)
    den = binding.lfmmi_graph_create(workloads.random_den_graph(rng, 500, 5, 40, 0.5))
    lens = rng.integers(1, T + 1, size=12).astype(np.int32)
    lens[3] = T
    x = torch.from_numpy(rng.normal(0, 2, size=(12, T, 40)).astype(np.float32)).cuda()
    want = binding.lfmmi_forward_backward(den, x, lens, 1e-5, 1.0, False)
    out = tuple(torch.empty_like(t) for t in want)
    side = torch.cuda.Stream()
    for count in "1234":
        monkeypatch.setenv("LFMMI_BUCKETS", count)
        graph = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            binding.lfmmi_forward_backward(den, x, lens, 1e-5, 1.0, False, *out)
            torch.cuda.synchronize()
            for a, b in zip(out, want):
                assert torch.equal(a, b)
            with torch.cuda.graph(graph, stream=side, capture_error_mode="relaxed"):
                binding.lfmmi_forward_backward(den, x, lens, 1e-5, 1.0, False, *out)
        for _ in range(3):
            for t in out:
                t.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            for a, b in zip(out, want):
                assert torch.equal(a, b)
        del graph
    den.close()


# how many buckets a call takes where its longest recursion is short; `low`: half of the
# sequences have that share of T frames
@pytest.mark.parametrize("by_state,B,T,P,low,buckets", [
    (False, 47, 240, 20, 0.3, 1), (False, 48, 239, 20, 0.3, 1), (False, 48, 240, 20, 0.3, 4),
    (False, 48, 240, 20, 0.45, 1), (True, 48, 240, 20, 0.3, 1),
    (False, 15, 240, 600, 0.3, 1), (False, 16, 240, 600, 0.3, 4), (False, 16, 240, 600, 0.55, 4),
    (False, 16, 240, 600, 0.6, 1), (True, 128, 240, 600, 0.3, 1), (True, 12, 400, 20, 1.0, 4),
])
def test_bucket_count_of_short_calls(by_state, B, T, P, low, buckets):
    import torch
    rng = np.random.default_rng(B)
    g = workloads.random_den_graph(rng, 20, 2, P, 0.5)
    if by_state:
        g["pdf"] = rng.integers(0, P, 20).astype(np.int32)[g["dst"]]
    den = binding.lfmmi_graph_create(g)
    binding.lfmmi_profile_enable(den, True)
    lens = np.full(B, T, np.int32)
    lens[(B + 1) // 2:] = int(low * T)
    binding.lfmmi_forward_backward(den, torch.zeros((B, T, P), device="cuda"), lens, 1e-5)
    assert binding.lfmmi_profile_read(den)["launches"] == buckets
    den.close()
