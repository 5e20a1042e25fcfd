"""GPU parity for graphs whose initial probabilities differ from state to state, against the
fp64 CPU oracle: state values kept divided by them, in every register-resident recursion.

Tolerances as in test_gpu_parity.py: objf 1e-4 relative, gradient 1e-4 absolute."""
import numpy as np
import pytest

from oracle import lfmmi_oracle as oracle
from paper_2005_09824_amd import binding, workloads

pytestmark = pytest.mark.gpu


# slots per wave: 16 .. 28 at 16 waves, the half as many waves with more, part of a wave's
# arcs streamed with either LDS map, plain and replicated emission rows; one slice; a pdf per
# entered state in a graph too large for the recursion by state (its occupancies are by state)
@pytest.mark.parametrize("S,k,P,by_state,leak", [
    (1, 0, 3, False, 1e-5), (20, 2, 10, False, 0.3), (64, 5, 300, False, 1e-5),
    (1000, 5, 84, False, 1e-3), (1237, 6, 51, False, 1e-5), (1900, 8, 84, False, 1e-5),
    (2048, 9, 84, False, 0.0), (2000, 10, 700, False, 1e-5), (600, 30, 60, False, 1e-5),
    (5000, 9, 84, False, 1e-5), (5000, 9, 900, False, 1e-3), (9000, 5, 300, False, 1e-5),
    (4500, 9, 84, True, 1e-3),
])
def test_row_weights(S, k, P, by_state, leak):
    rng = np.random.default_rng(S + P)
    g = workloads.random_den_graph(rng, S, k, P, 0.5)
    if by_state:
        g["pdf"] = rng.integers(0, P, S).astype(np.int32)[g["dst"]]
    p = rng.uniform(0.01, 1.0, S) ** 2
    g["init_prob"] = (p / p.sum()).astype(np.float32)
    g["final_prob"] = rng.uniform(0.2, 1.0, S).astype(np.float32)
    run(g, leak, 2 if S > 1 else 0)


@pytest.mark.parametrize("kind", ["wide_range", "tiny_weights"])
def test_weights_that_leave_the_range_keep_their_factors_per_arc(kind):
    # pi[from] / pi[to] or w * pi[from] outside the normal range of fp32
    rng = np.random.default_rng(3)
    g = workloads.random_den_graph(rng, 300, 5, 20, 0.5)
    p = rng.uniform(0.5, 1.0, 300)
    if kind == "wide_range":
        p[::3] *= 1e-30
    else:
        g["logw"] = np.minimum(g["logw"], 0).astype(np.float32)
        g["logw"][::7] = -84.0
    g["init_prob"] = (p / p.sum()).astype(np.float32)
    run(g, 1e-5, 1)


def run(g, leak, kept):
    rng = np.random.default_rng(9)
    P, T = g["num_pdfs"], 14
    lengths = np.array([14, 1, 0, 7, 2], np.int32)
    x = rng.normal(0, 2, (5, T, P)).astype(np.float32)
    for b in range(5):
        x[b, lengths[b]:] = np.nan
    compare(g, x, lengths, leak, kept)


def compare(g, x, lengths, leak, kept):
    # kept: 2 state values divided by the initial probabilities, 1 a leak factor per arc
    torch = pytest.importorskip("torch")
    lengths = np.asarray(lengths, np.int32)
    h = binding.lfmmi_graph_create(g)
    assert binding.lfmmi_graph_info(h)["fp64"] == 0
    assert binding.lfmmi_graph_ordering_info(h, 0, 0)["per_arc_leak"] == kept
    objf, grad, status = binding.lfmmi_forward_backward(h, torch.from_numpy(x).cuda(), lengths, leak)
    torch.cuda.synchronize()
    h.close()
    lz, gamma = oracle.forward_backward(g, x, lengths, leak)
    assert np.all(status.cpu().numpy() == 0)
    assert np.all(np.abs(objf.cpu().numpy() - lz) <= 1e-4 * np.maximum(np.abs(lz), 1.0))
    assert np.abs(grad.cpu().numpy().astype(np.float64) - gamma).max() <= 1e-4


def _graph(S, P, arcs, init_prob, final_prob=None):
    src, dst, pdf, logw = zip(*arcs)
    return {"num_states": S, "num_pdfs": P, "src": np.array(src, np.int32), "dst": np.array(dst, np.int32),
            "pdf": np.array(pdf, np.int32), "logw": np.array(logw, np.float32),
            "init_prob": np.array(init_prob, np.float32),
            "final_prob": np.ones(S, np.float32) if final_prob is None else np.array(final_prob, np.float32)}


def _rare_state(rare, extra_arcs=(), final=1.0, arcs_out=3, copies=1):
    """State 0 starts with probability `rare` and has pdfs 0 and 1 to itself; states 1 to 8,
    which it is left for by `extra_arcs` only, take pdfs 2 to 5, `arcs_out` arcs out of each.
    Every arc stands there `copies` times, each with its share of the weight."""
    arcs = [(0, 0, 0, 0.0), (0, 0, 1, -1.0)] + list(extra_arcs)
    arcs += [(s, 1 + (s - 1 + k) % 8, 2 + (s + k) % 4, -1.1) for s in range(1, 9) for k in range(1, 1 + arcs_out)]
    arcs = [(i, j, d, w - np.log(copies)) for i, j, d, w in arcs for _ in range(copies)]
    return _graph(9, 7, arcs, [rare] + [1 / 8] * 8, [final] + [1.0] * 8)


def _noise(shape, seed=0):
    return np.random.default_rng(seed).normal(0, 1, shape).astype(np.float32)


# The rare state wins the first frames and is penalised in the following ones, so that its
# beta is small where its alpha is not: w pi beta leaves the range of fp32, w alpha beta does
# not. Both kernels that add up occupancies by arc.
@pytest.mark.parametrize("planes", ["4", "0"])
@pytest.mark.parametrize("leak", [0.0, 1e-5])
@pytest.mark.parametrize("rare", [1e-8, 1e-12, 1e-17, 1e-30])
def test_occupancies_of_a_rare_initial_state(rare, leak, planes, monkeypatch):
    monkeypatch.setenv("LFMMI_OCC_MULTI", planes)
    x = _noise((1, 10, 7))
    x[:, :5, :2] += (75 - np.log(rare)) / 5
    x[:, 5:, 2:] += 15
    compare(_rare_state(rare), x, [10], leak, 2 if rare > 1e-18 else 1)


# The rare state is left through one arc that takes a pdf far below the frame's best: the
# weight w pi[from] / pi[to] times that emission leaves the range of fp32, times the state's
# value it does not. In a wave of few slots, of more, and of more than the registers hold.
@pytest.mark.parametrize("arcs_out,copies", [(1, 1), (3, 1), (3, 20)])
@pytest.mark.parametrize("rare,below", [(1e-4, 70.0), (1e-12, 70.0), (1e-17, 60.0), (1e-17, 70.0)])
def test_recursion_out_of_a_rare_initial_state(rare, below, arcs_out, copies):
    x = _noise((1, 8, 7))
    x[0, :3, 0] += (below + 20 - np.log(rare)) / 3
    x[0, 3, 6] += below
    x[0, 3, 0] -= 30
    x[0, 3, 2:6] -= 10
    g = _rare_state(rare, [(0, 1, 1, -0.5), (0, 2, 2, -1.0)], 1.0, arcs_out, copies)
    h = binding.lfmmi_graph_pack(g)
    info = [binding.lfmmi_graph_ordering_info(h, 0, o) for o in (0, 1)]
    h.close()
    if copies > 1:
        assert all(0 < i["register_slots"] < i["max_wave_slots"] for i in info)
    else:
        assert (info[0]["max_wave_slots"] <= 4) == (arcs_out == 1)  # alpha, which holds the ratios
    compare(g, x, [8], 0.0, 2)


# What cannot be kept divided by the initial probabilities in fp32: values that would overflow
# (large weights into a rare state), final weights that vanish beside them, ratios beyond e^40.
@pytest.mark.parametrize("kind", ["overflow", "final", "ratio"])
def test_graphs_that_keep_their_factors_per_arc(kind):
    if kind == "overflow":
        S = 51
        arcs = [(0, 1, 2, 0.0), (0, 7, 3, 0.0)]
        for s in range(1, S):
            arcs += [(s, 0, s % 5, 6.0), (s, 1 + s % (S - 1), s * 3 % 5, 0.0)]
        g, x = _graph(S, 5, arcs, [1e-37] + [0.02] * (S - 1)), _noise((1, 8, 5))
    elif kind == "final":
        g, x = _rare_state(1e-17, final=1e-28), _noise((1, 10, 7))
        x[:, :, :2] += 12
    else:
        g, x = _rare_state(1e-19), _noise((1, 10, 7))
        x[:, :, :2] += 8
    for leak in (0.0, 1e-5):
        compare(g, x, [x.shape[1]], leak, 1)


def test_one_handle_of_graphs_with_equal_and_differing_initial_probabilities():
    torch = pytest.importorskip("torch")
    rng = np.random.default_rng(12)
    P, graphs = 30, []
    for S, k, varied in ((200, 4, True), (64, 3, False), (1, 0, False), (700, 5, True)):
        g = workloads.random_den_graph(rng, S, k, P, 0.5)
        if varied:
            p = rng.uniform(0.01, 1.0, S) ** 2
            g["init_prob"] = (p / p.sum()).astype(np.float32)
        graphs.append(g)
    lengths = np.array([12, 9, 14, 5], np.int32)
    x = rng.normal(0, 2, (4, 14, P)).astype(np.float32)
    for b in range(4):
        x[b, lengths[b]:] = np.nan
    h = binding.lfmmi_graph_create_batch(graphs)
    assert all(binding.lfmmi_graph_ordering_info(h, i, 0)["per_arc_leak"] == 2 for i in range(4))
    objf, grad, status = binding.lfmmi_forward_backward(h, torch.from_numpy(x).cuda(), lengths, 1e-3)
    torch.cuda.synchronize()
    h.close()
    lz, gamma = oracle.forward_backward_per_utt(graphs, x, lengths, 1e-3)
    assert np.all(status.cpu().numpy() == 0)
    assert np.all(np.abs(objf.cpu().numpy() - lz) <= 1e-4 * np.maximum(np.abs(lz), 1.0))
    assert np.abs(grad.cpu().numpy().astype(np.float64) - gamma).max() <= 1e-4
