"""GPU parity for graphs whose arcs all carry the pdf-id of the state they enter, against
the fp64 CPU oracle, at the sizes where their kernels change shape.

Tolerances as in test_gpu_parity.py: objf 1e-4 relative, gradient 1e-4 absolute."""
import numpy as np
import pytest

from oracle import lfmmi_oracle as oracle
from paper_2005_09824_amd import binding, workloads

pytestmark = pytest.mark.gpu


def by_state_graph(rng, S, k, P, init="uniform", some_final=False):
    """A random graph whose pdf-ids are a function of the entered state."""
    g = workloads.random_den_graph(rng, S, k, P, 0.5)
    g["pdf"] = rng.integers(0, P, S).astype(np.int32)[g["dst"]]
    if init == "varied":
        p = rng.uniform(0.1, 1.0, S)
        g["init_prob"] = (p / p.sum()).astype(np.float32)
    if some_final:
        fin = (rng.random(S) < 0.5).astype(np.float32)
        fin[0] = 1.0
        g["final_prob"] = fin
    return g


def parity(g, lengths, T, leak=1e-5, seed=4):
    rng = np.random.default_rng(seed)
    P, B = g["num_pdfs"], len(lengths)
    lengths = np.asarray(lengths, np.int32)
    x = rng.normal(0, 2, (B, T, P)).astype(np.float32)
    for b in range(B):
        x[b, lengths[b]:] = np.nan
    h = binding.lfmmi_graph_create(g)
    torch = pytest.importorskip("torch")
    objf, grad, status = binding.lfmmi_forward_backward(h, torch.from_numpy(x).cuda(), lengths, leak)
    torch.cuda.synchronize()
    h.close()
    lz, gamma = oracle.forward_backward(g, x, lengths, leak)
    assert np.all(status.cpu().numpy() == 0)
    assert np.all(np.abs(objf.cpu().numpy() - lz) <= 1e-4 * np.maximum(np.abs(lz), 1.0))
    err = np.abs(grad.cpu().numpy().astype(np.float64) - gamma)
    assert err.max() <= 1e-4, err.max()
    for b in range(B):
        assert np.all(grad[b, lengths[b]:].cpu().numpy() == 0.0)


# occupancies added up over states: four, two and one frames per workgroup in fp32 and
# fp64, lengths around multiples of them, pdfs nothing enters, one pdf that most states carry
@pytest.mark.parametrize("S,k,P,some_final", [
    (1, 0, 1, False), (65, 3, 200, False), (1200, 2, 9, False), (1300, 2, 84, False),
    (2500, 2, 84, False), (9000, 2, 300, False),
    (64, 3, 5, True), (600, 2, 84, True), (700, 2, 84, True), (1500, 2, 30, True), (3000, 2, 84, True),
])
def test_occupancies_by_state(S, k, P, some_final):
    rng = np.random.default_rng(S)
    g = by_state_graph(rng, S, k, P, some_final=some_final)
    if P == 9:
        g["pdf"] = np.where(g["dst"] % 8 == 0, g["pdf"], 3).astype(np.int32)
    parity(g, [9, 1, 8, 0, 5], 11)


# the recursion without an emission gather: one barrier per step, scalars of a step known
# before its rows. Waves with one short slice (4, 8 slots), resident arcs up to the most
# slots that are built, uniform and other initial probabilities, fp32 and fp64; lengths
# around the two steps that are fetched ahead
@pytest.mark.parametrize("S,k,P,init,some_final,leak", [
    (1, 0, 1, "uniform", False, 1e-5), (20, 1, 7, "uniform", False, 0.3), (130, 1, 7, "varied", False, 1e-5),
    (1024, 1, 40, "uniform", False, 1e-5), (1024, 3, 40, "varied", True, 1e-3), (200, 1, 9, "varied", True, 0.0),
    (1500, 6, 40, "varied", False, 1e-3), (1900, 12, 60, "varied", False, 1e-5),
    (2000, 15, 60, "uniform", False, 1e-3), (4096, 6, 84, "uniform", False, 0.0),
    (700, 3, 84, "varied", True, 1e-3),
])
def test_recursion_by_state(S, k, P, init, some_final, leak):
    rng = np.random.default_rng(S + k)
    g = by_state_graph(rng, S, k, P, init, some_final)
    parity(g, [6, 1, 0, 2, 3, 4, 5, 23], 23, leak)


def test_recursion_by_state_flags_what_it_flagged_before():
    # a chain that cannot be left in so few frames: zero probability; a NaN logit
    K, P = 40, 6
    src = np.arange(K - 1, dtype=np.int32)
    g = {"num_states": K, "num_pdfs": P, "src": src, "dst": src + 1,
         "pdf": ((src + 1) % P).astype(np.int32), "logw": np.zeros(K - 1, np.float32),
         "init_prob": np.eye(K, dtype=np.float32)[0], "final_prob": np.eye(K, dtype=np.float32)[K - 1]}
    torch = pytest.importorskip("torch")
    x = torch.zeros((3, 60, P))
    x[1, 7, 2] = float("nan")
    h = binding.lfmmi_graph_create(g)
    lengths = np.array([39, 39, 20], np.int32)
    objf, grad, status = binding.lfmmi_forward_backward(h, x.cuda(), lengths, 0.0)
    torch.cuda.synchronize()
    h.close()
    assert status.tolist() == [0, 3, 1]
    assert objf[0].item() == 0.0 and np.isnan(objf[1].item()) and objf[2].item() == -np.inf
    assert torch.all(grad[1:] == 0)
    want = torch.zeros((39, P))
    want[torch.arange(39), (torch.arange(39) + 1) % P] = 1.0
    assert torch.equal(grad[0, :39].cpu(), want)


def regular_graph(rng, S, d_first, d_second, P, init="uniform"):
    """States of the first half have d_first arcs in and out, all within the half, the others
    d_second: every slice of a half is that many slots wide in both directions."""
    src, dst = [], []
    for at, d in ((0, d_first), (S // 2, d_second)):
        i = np.arange(S // 2)
        for q in range(d):
            src.append(at + (i * 1 + q * 7) % (S // 2))
            dst.append(at + i)
    src, dst = np.concatenate(src).astype(np.int32), np.concatenate(dst).astype(np.int32)
    p = rng.uniform(0.1, 1.0, S) if init == "varied" else np.ones(S)
    return {"num_states": S, "num_pdfs": P, "src": src, "dst": dst,
            "pdf": rng.integers(0, P, S).astype(np.int32)[dst],
            "logw": np.log(rng.uniform(0.02, 0.2, len(src))).astype(np.float32),
            "init_prob": (p / p.sum()).astype(np.float32), "final_prob": np.ones(S, np.float32)}


# the straight-line recursion: every width of a wave's first slice that it is laid out for, slot
# counts at both of its tests for the end of a wave's slots and in every number of slots it is
# built for; lengths around the 64 steps whose totals are stored together
@pytest.mark.parametrize("wide,narrow,slots,init", [
    (2, 2, 16, "uniform"), (6, 2, 16, "uniform"), (10, 6, 16, "uniform"), (14, 4, 24, "uniform"),
    (12, 10, 24, "uniform"), (12, 12, 24, "uniform"), (18, 8, 32, "uniform"), (15, 13, 32, "uniform"),
    (16, 16, 32, "uniform"), (17, 16, 36, "uniform"), (18, 18, 36, "uniform"), (34, 2, 36, "uniform"),
    (5, 3, 16, "varied"), (13, 9, 24, "varied"), (15, 13, 32, "varied"), (17, 17, 36, "varied"),
])
def test_straight_line_recursion(wide, narrow, slots, init):
    g = regular_graph(np.random.default_rng(wide * 40 + narrow), 2048, wide, narrow, 50, init)
    closing = 1 if init == "varied" else 0
    even = lambda d: (d + closing + 1) // 2 * 2
    h = binding.lfmmi_graph_pack(g)
    for o in (0, 1):
        c = binding.lfmmi_graph_ordering_copy(h, 0, o)
        assert c["register_slots"] == slots and c["lds_vector_rows"] == 2048
        widths = np.diff(c["slice_off"]).reshape(16, 2)
        assert np.all(widths == [even(narrow), even(wide)])
    h.close()
    parity(g, [129, 128, 127, 66, 65, 64, 63, 2, 1, 0, 3], 129, 1e-3)


# ... waves with one slice and with two side by side, in a handle whose graphs leave some waves
# of the workgroup without any
def test_straight_line_recursion_of_graphs_of_different_sizes():
    torch = pytest.importorskip("torch")
    rng = np.random.default_rng(8)
    graphs = [by_state_graph(rng, S, k, 50) for S, k in ((1100, 12), (70, 5), (1, 0), (2000, 7))]
    lengths = np.array([70, 65, 3, 41], np.int32)
    x = rng.normal(0, 2, (4, 70, 50)).astype(np.float32)
    h = binding.lfmmi_graph_create_batch(graphs)
    assert binding.lfmmi_graph_ordering_info(h, 0, 0)["lds_vector_rows"] == 2048
    assert [binding.lfmmi_graph_ordering_info(h, i, 0)["waves"] for i in range(4)] == [16, 2, 1, 16]
    objf, grad, status = binding.lfmmi_forward_backward(h, torch.from_numpy(x).cuda(), lengths, 1e-4)
    torch.cuda.synchronize()
    h.close()
    assert np.all(status.cpu().numpy() == 0)
    for b, g in enumerate(graphs):
        lz, gamma = oracle.forward_backward(g, x[b:b + 1], lengths[b:b + 1], 1e-4)
        assert abs(objf[b].item() - lz[0]) <= 1e-4 * max(abs(lz[0]), 1.0)
        assert np.abs(grad[b].cpu().numpy() - gamma[0]).max() <= 1e-4


# small graphs with many arcs a state: 38 to 48 slots a wave with at most 8 waves, lengths around
# the steps fetched ahead; one slice, three, six
@pytest.mark.parametrize("S,k,waves,slots", [(60, 40, 1, 48), (150, 30, 3, 44), (340, 24, 6, 38)])
def test_recursion_by_state_of_small_dense_graphs(S, k, waves, slots):
    g = by_state_graph(np.random.default_rng(S + k), S, k, 40)
    h = binding.lfmmi_graph_pack(g)
    info, fwd = binding.lfmmi_graph_info(h), binding.lfmmi_graph_ordering_info(h, 0, 0)
    bwd = binding.lfmmi_graph_ordering_info(h, 0, 1)
    h.close()
    assert info["rec_waves"] == waves and max(fwd["max_wave_slots"], bwd["max_wave_slots"]) == slots
    assert info["emission_by_state"] == 1 and fwd["register_slots"] == 48
    parity(g, [6, 1, 0, 2, 3, 4, 5, 23], 23)


# occupancies by state where the recursion has hub slices (63 padding rows each)
@pytest.mark.parametrize("init,some_final", [("uniform", False), ("varied", False), ("varied", True)])
def test_occupancies_by_state_with_hub_slices(init, some_final):
    rng = np.random.default_rng(31)
    S, P = 900, 60
    g = by_state_graph(rng, S, 6, P, init, some_final)
    into, out_of = rng.choice(S, 500, replace=False), rng.choice(S, 350, replace=False)
    g["src"] = np.concatenate([g["src"], into, np.full(350, 3)]).astype(np.int32)
    g["dst"] = np.concatenate([g["dst"], np.full(500, 5), out_of]).astype(np.int32)
    g["logw"] = np.concatenate([g["logw"], np.log(rng.uniform(0.01, 0.2, 850))]).astype(np.float32)
    g["pdf"] = rng.integers(0, P, S).astype(np.int32)[g["dst"]]
    h = binding.lfmmi_graph_pack(g)
    assert all(binding.lfmmi_graph_ordering_info(h, 0, o)["hub_slices"] == 1 for o in (0, 1))
    h.close()
    parity(g, [9, 1, 8, 0, 23], 23)
