"""GPU parity of the straight-line recursion for graphs whose arcs carry pdfs of their own,
against the fp64 CPU oracle. Tolerances as in test_gpu_parity.py."""
import numpy as np
import pytest

from oracle import lfmmi_oracle as oracle
from paper_2005_09824_amd import binding, workloads
from tests.test_gpu_by_state import parity, regular_graph
from tests.test_host_logic import graded_graph

pytestmark = pytest.mark.gpu

# around the 64 steps whose totals are stored together, and the steps that are fetched ahead
LENGTHS = [129, 128, 127, 66, 65, 64, 63, 4, 3, 2, 1, 0]


# every width of a wave's first slice that the line is laid out for, slot counts at both of its
# tests for the end of a wave's slots and in every number of slots it is built for; one and two
# staging passes of a replicated emission row (128 pdfs, 129 to 255) and plain rows
@pytest.mark.parametrize("wide,narrow,slots,P,init", [
    (2, 2, 16, 50, "uniform"), (6, 2, 16, 128, "uniform"), (8, 8, 16, 129, "uniform"), (10, 6, 16, 256, "uniform"),
    (16, 4, 24, 50, "uniform"), (11, 9, 24, 255, "uniform"), (12, 12, 24, 700, "uniform"),
    (22, 2, 24, 30, "uniform"), (14, 14, 28, 50, "uniform"), (20, 8, 28, 140, "uniform"), (14, 12, 28, 3072, "uniform"),
    (5, 3, 16, 50, "varied"), (9, 5, 16, 200, "varied"), (13, 9, 24, 128, "varied"), (13, 13, 28, 50, "varied"),
    (13, 13, 28, 230, "varied"), (13, 11, 28, 300, "varied"),
])
def test_straight_line_recursion_by_arc(wide, narrow, slots, P, init):
    rng = np.random.default_rng(wide * 40 + narrow)
    g = regular_graph(rng, 2048, wide, narrow, P, init)
    g["pdf"] = rng.integers(0, P, len(g["src"])).astype(np.int32)
    closing = 1 if init == "varied" else 0
    even = lambda d: (d + closing + 1) // 2 * 2
    h = binding.lfmmi_graph_pack(g)
    assert binding.lfmmi_graph_info(h)["emission_by_state"] == 0
    for o in (0, 1):
        c = binding.lfmmi_graph_ordering_copy(h, 0, o)
        assert c["register_slots"] == slots and c["lds_vector_rows"] == 2048
        assert c["emission_replicated"] == (1 if P <= 255 else 0)
        widths = np.diff(c["slice_off"]).reshape(16, 2)
        assert np.all(widths == [even(narrow), even(wide)])
    h.close()
    lengths = LENGTHS if P < 1000 else LENGTHS[3:]
    parity(g, lengths, max(lengths), 1e-3)


# workgroups of one wave to eleven, of which some only help to stage a row; waves with one slice
# and with two side by side
@pytest.mark.parametrize("S,k,P,init", [
    (1, 1, 3, "uniform"), (20, 2, 10, "uniform"), (64, 9, 84, "uniform"), (65, 3, 200, "varied"), (130, 5, 300, "uniform"),
    (700, 8, 84, "varied"), (1000, 9, 255, "uniform"), (1237, 6, 51, "varied"), (1900, 9, 84, "uniform"), (2048, 3, 40, "uniform"),
])
def test_straight_line_recursion_by_arc_of_random_graphs(S, k, P, init):
    rng = np.random.default_rng(S)
    g = workloads.random_den_graph(rng, S, min(k, S - 1), P, 0.5)
    if S == 1:  # two arcs on one state
        g["src"] = g["dst"] = np.zeros(2, np.int32)
        g["pdf"], g["logw"] = np.array([0, 2], np.int32), np.log(np.array([0.4, 0.3], np.float32))
    if init == "varied":
        p = rng.uniform(0.1, 1.0, S)
        g["init_prob"] = (p / p.sum()).astype(np.float32)
    h = binding.lfmmi_graph_pack(g)
    assert binding.lfmmi_graph_ordering_info(h, 0, 0)["lds_vector_rows"] == 2048
    h.close()
    parity(g, LENGTHS, 129, 1e-4)


# a handle whose graphs leave some waves of the workgroup without any slice; a dead and a NaN
# sequence beside sound ones
def test_straight_line_recursion_by_arc_of_graphs_of_different_sizes():
    torch = pytest.importorskip("torch")
    rng = np.random.default_rng(9)
    graphs = [workloads.random_den_graph(rng, S, k, 50, 0.5) for S, k in ((1100, 9), (70, 5), (5, 2), (2000, 7), (300, 4))]
    lengths = np.array([70, 65, 3, 41, 50], np.int32)
    x = rng.normal(0, 2, (5, 70, 50)).astype(np.float32)
    x[4, 20, 7] = np.nan
    h = binding.lfmmi_graph_create_batch(graphs)
    assert binding.lfmmi_graph_ordering_info(h, 0, 0)["lds_vector_rows"] == 2048
    assert [binding.lfmmi_graph_ordering_info(h, i, 0)["waves"] for i in range(5)] == [16, 2, 1, 16, 5]
    objf, grad, status = binding.lfmmi_forward_backward(h, torch.from_numpy(x).cuda(), lengths, 1e-4)
    torch.cuda.synchronize()
    h.close()
    assert status.tolist() == [0, 0, 0, 0, 3]
    assert np.isnan(objf[4].item()) and torch.all(grad[4] == 0)
    for b, g in enumerate(graphs[:4]):
        lz, gamma = oracle.forward_backward(g, x[b:b + 1], lengths[b:b + 1], 1e-4)
        assert abs(objf[b].item() - lz[0]) <= 1e-4 * max(abs(lz[0]), 1.0)
        assert np.abs(grad[b].cpu().numpy() - gamma[0]).max() <= 1e-4


# the hybrid recursion: one and two staging passes of a replicated emission row, plain rows, both
# LDS maps, waves that stream a few pairs and many; uniform and other initial probabilities
@pytest.mark.parametrize("S,k,P,init", [
    (2100, 17, 40, "uniform"), (2100, 24, 128, "varied"), (3000, 13, 129, "uniform"), (2500, 15, 255, "varied"),
    (2500, 16, 256, "uniform"), (2200, 22, 1500, "varied"), (8300, 5, 300, "uniform"), (8300, 5, 3072, "varied"),
])
def test_hybrid_recursion_by_arc(S, k, P, init):
    rng = np.random.default_rng(S + P)
    g = workloads.random_den_graph(rng, S, k, P, 0.5)
    if init == "varied":
        p = rng.uniform(0.1, 1.0, S)
        g["init_prob"] = (p / p.sum()).astype(np.float32)
    h = binding.lfmmi_graph_pack(g)
    info = binding.lfmmi_graph_ordering_info(h, 0, 0)
    h.close()
    assert info["register_slots"] == 36 < info["max_wave_slots"]
    assert info["emission_replicated"] == (1 if P <= 255 else 0)
    assert info["lds_vector_rows"] == (8192 if S <= 8192 else 12288)
    parity(g, LENGTHS[3:], 66, 1e-4)


# a handle of such graphs of different sizes, among them one whose waves stream nothing and one that
# leaves most waves without a slice; a dead and a NaN sequence beside sound ones
@pytest.mark.parametrize("init", ["uniform", "varied"])
def test_hybrid_recursion_by_arc_of_graphs_of_different_sizes(init):
    torch = pytest.importorskip("torch")
    rng = np.random.default_rng(11)
    graphs = [workloads.random_den_graph(rng, S, k, 50, 0.5)
              for S, k in ((2500, 16), (300, 4), (2100, 20), (3000, 6), (2500, 15), (2200, 17))]
    for g in graphs:
        g["num_pdfs"] = 51  # the last is on no arc
        if init == "varied":
            p = rng.uniform(0.1, 1.0, g["num_states"])
            g["init_prob"] = (p / p.sum()).astype(np.float32)
    lengths = np.array([66, 65, 30, 64, 50, 2], np.int32)
    x = rng.normal(0, 2, (6, 66, 51)).astype(np.float32)
    x[2, 11, :50] = -np.inf
    x[4, 20, 7] = np.nan
    h = binding.lfmmi_graph_create_batch(graphs)
    info = [binding.lfmmi_graph_ordering_info(h, i, 0) for i in range(6)]
    assert all(i["register_slots"] == 36 and i["lds_vector_rows"] == 8192 for i in info)
    assert info[1]["waves"] == 5 and info[3]["max_wave_slots"] < 36 < info[0]["max_wave_slots"]
    objf, grad, status = binding.lfmmi_forward_backward(h, torch.from_numpy(x).cuda(), lengths, 1e-4)
    torch.cuda.synchronize()
    h.close()
    assert status.tolist() == [0, 0, 1, 0, 3, 0]
    assert objf[2].item() == -np.inf and np.isnan(objf[4].item())
    assert torch.all(grad[2] == 0) and torch.all(grad[4] == 0)
    for b in (0, 1, 3, 5):
        lz, gamma = oracle.forward_backward(graphs[b], x[b:b + 1], lengths[b:b + 1], 1e-4)
        assert abs(objf[b].item() - lz[0]) <= 1e-4 * max(abs(lz[0]), 1.0)
        assert np.abs(grad[b].cpu().numpy() - gamma[0]).max() <= 1e-4


# graphs that two slices a wave would suit but for a hub, or for initial probabilities that keep a
# leak factor per arc: slices dealt freely, every arc in registers
@pytest.mark.parametrize("graph,registers", [
    ((1980, 24, 6, 0.2, 84, True, 1100), 26), ((1980, 12, 5, 0.45, 84, False, 1100), 20),
    ((1980, 10, 4, 0.2, 84, False, 1100, "varied"), 48), ((1600, 18, 4, 0.33, 84, False, 0, "wide"), 48),
])
def test_recursion_of_graphs_that_nearly_take_the_straight_line(graph, registers):
    g = graded_graph(*graph)
    h = binding.lfmmi_graph_pack(g)
    info = binding.lfmmi_graph_ordering_info(h, 0, 0)
    h.close()
    assert info["register_slots"] == registers and info["lds_vector_rows"] == 8192
    parity(g, LENGTHS[3:], 66, 1e-4)
