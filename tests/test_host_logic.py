"""CPU-side tests: the C-ABI library loads and exports what include/lfmmi.h
declares, the graph packer keeps every arc exactly once in each of its three
orderings, and argument errors come back as status codes with a message.
No kernel is launched here."""
import ctypes
import os
import re

import numpy as np
import pytest

from paper_2005_09824_amd import binding, workloads

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "lfmmi.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)  # declarations only
    declared = set(re.findall(r"\b(lfmmi_[a-z_]+)\s*\(", header))
    assert declared, "no declarations found"
    lib = binding.load_library()
    for name in sorted(declared):
        assert hasattr(lib, name), name
    assert declared == set(binding.EXPORTS)


def _unpack(graph_handle, g, graph):
    """Rebuild (src, dst, pdf, w) lists from each packed ordering."""
    od = [binding.lfmmi_graph_ordering_copy(graph_handle, g, o) for o in range(3)]
    state_of = [od[0]["row_id"], od[1]["row_id"]]  # position -> state, per numbering
    out = []
    for o in range(3):
        d = od[o]
        arcs = []
        assert d["slice_off"][0] == 0 and d["slice_off"][-1] == d["total_slots"]
        assert d["wave_first"][0] == 0 and d["wave_first"][-1] == d["slices"]
        assert np.all(np.diff(d["wave_first"]) >= 0)
        per_wave = []
        for wv in range(d["waves"]):
            s0, s1 = d["wave_first"][wv], d["wave_first"][wv + 1]
            per_wave.append(int(d["slice_off"][s1] - d["slice_off"][s0]))
        assert max(per_wave) == d["max_wave_slots"]
        for s in range(d["slices"]):
            o0, o1 = d["slice_off"][s], d["slice_off"][s + 1]
            if o < 2 and d["closing_slots"]:   # it carries the row's leak-dot weight
                o1 -= 1
                for lane in range(64):
                    row = s * 64 + lane
                    st = d["row_id"][row]
                    want = 0.0 if st < 0 else (1.0 if o == 0 else float(graph["init_prob"][st]))
                    assert d["key"][o1 * 64 + lane] == 0
                    assert d["w"][o1 * 64 + lane] == np.float32(want)
            hub = o < 2 and d["slice_hub"][s]
            if hub:  # all 64 lanes hold arcs of lane 0's row; the other rows are padding
                assert d["row_id"][s * 64] >= 0 and np.all(d["row_id"][s * 64 + 1:s * 64 + 64] < 0)
            for lane in range(64):
                row = s * 64 if hub else s * 64 + lane
                for i in range(o0, o1):
                    k, w = int(d["key"][i * 64 + lane]), float(d["w"][i * 64 + lane])
                    if w == 0.0:      # padding: anywhere in the row (slots are ordered to
                        continue      # spread LDS banks); its key points at an unused bank
                    assert d["row_id"][row] >= 0
                    x, y = (k & 0xFFFF) // 4, (k >> 16) // 4
                    if o == 0:
                        arcs.append((int(state_of[0][x]), int(d["row_id"][row]), y, w))
                    elif o == 1:
                        arcs.append((int(d["row_id"][row]), int(state_of[1][x]), y, w))
                    else:
                        arcs.append((int(state_of[0][x]), int(state_of[1][y]),
                                     int(d["row_id"][row]), w))
        out.append(sorted(arcs))
    want = sorted(zip(graph["src"].tolist(), graph["dst"].tolist(), graph["pdf"].tolist(),
                      np.exp(graph["logw"].astype(np.float64)).astype(np.float32).tolist()))
    return out, want, od


@pytest.mark.parametrize("which", ["tiny", "den_scaled", "zipf"])
def test_pack_keeps_every_arc_once(which):
    if which == "tiny":
        g = workloads.make_workload(1)["den"]
    elif which == "den_scaled":
        g = workloads.make_workload(2, scale={"S": 300, "B": 2, "Tlo": 5, "Thi": 6})["den"]
    else:
        g = workloads.make_workload(3, scale={"S": 200, "P": 50, "B": 2, "Tlo": 5, "Thi": 6})["den"]
    h = binding.lfmmi_graph_pack(g)
    got, want, od = _unpack(h, 0, g)
    for o in range(3):
        assert got[o] == want, "ordering %d lost or changed arcs" % o
    S = g["num_states"]
    for o in range(2):
        ids = od[o]["row_id"]
        assert sorted(ids[ids >= 0].tolist()) == list(range(S))  # a permutation of the states
        assert od[o]["rows"] == S and od[o]["slices"] == (S + 63) // 64
    info = binding.lfmmi_graph_info(h)
    assert info["num_graphs"] == 1 and info["total_arcs"] == len(g["src"]) and info["uploaded"] == 0
    h.close()


def test_pack_batch_of_numerators():
    wl = workloads.make_workload(5, scale={"B": 5, "nlo": 3, "nhi": 9})
    h = binding.lfmmi_graph_pack_batch(wl["num"])
    assert binding.lfmmi_graph_info(h)["num_graphs"] == 5
    for g in range(5):
        got, want, _ = _unpack(h, g, wl["num"][g])
        for o in range(3):
            assert got[o] == want
    h.close()


def test_pack_waves_are_balanced():
    g = workloads.make_workload(2)["den"]
    h = binding.lfmmi_graph_pack(g)
    info = binding.lfmmi_graph_info(h)
    assert info["rec_waves"] == 16
    for o in range(3):
        oi = binding.lfmmi_graph_ordering_info(h, 0, o)
        ideal = len(g["src"]) / (64.0 * oi["waves"])
        assert oi["max_wave_slots"] <= 1.35 * ideal + 4, (o, oi, ideal)
    h.close()


def test_slot_ordering_lowers_modelled_bank_conflicts(monkeypatch):
    g = workloads.make_workload(2)["den"]
    tuned = binding.lfmmi_graph_pack(g)
    monkeypatch.setenv("LFMMI_BALANCE", "0")
    monkeypatch.setenv("LFMMI_ORDER", "0")
    plain = binding.lfmmi_graph_pack(g)
    for o in range(3):
        a = binding.lfmmi_graph_ordering_info(tuned, 0, o)
        b = binding.lfmmi_graph_ordering_info(plain, 0, o)
        floor = 2 * a["total_slots"] * (1 if o < 2 else 2)  # one cycle per half-wave gather
        assert floor <= a["gather_cycles"] <= 0.7 * b["gather_cycles"], (o, a, b)
    tuned.close(); plain.close()


@pytest.mark.parametrize("which", ["den", "hmm"])
def test_occupancy_arcs_dealt_to_rows_and_slots_keep_every_arc(which, monkeypatch):
    # the occupancy ordering may place an arc in any row of its pdf: both placements hold every
    # arc once, in a row of its pdf, and the one that is kept is never the dearer of the two
    if which == "den":
        g = workloads.make_workload(2, scale={"B": 2, "Tlo": 5, "Thi": 6})["den"]
    else:
        g = workloads.make_workload(6, scale={"B": 2, "Tlo": 5, "Thi": 6})["den"]
    both = binding.lfmmi_graph_pack(g)
    monkeypatch.setenv("LFMMI_DEAL", "0")
    ordered = binding.lfmmi_graph_pack(g)
    for h in (both, ordered):
        got, want, _ = _unpack(h, 0, g)
        assert got[2] == want
    a = binding.lfmmi_graph_ordering_info(both, 0, 2)
    b = binding.lfmmi_graph_ordering_info(ordered, 0, 2)
    assert a["total_slots"] == b["total_slots"] and a["rows"] == b["rows"]
    assert 4 * a["total_slots"] <= a["gather_cycles"] <= b["gather_cycles"]
    if which == "den":  # random pdfs on the arcs: the joint placement wins
        assert a["gather_cycles"] <= 0.95 * b["gather_cycles"], (a, b)
    both.close(); ordered.close()


def test_graph_with_no_arcs_and_isolated_states():
    g = {"num_states": 3, "num_pdfs": 2, "src": np.zeros(0, np.int32), "dst": np.zeros(0, np.int32),
         "pdf": np.zeros(0, np.int32), "logw": np.zeros(0, np.float32),
         "init_prob": np.ones(3, np.float32), "final_prob": np.ones(3, np.float32)}
    h = binding.lfmmi_graph_pack(g)
    assert binding.lfmmi_graph_ordering_info(h, 0, 0)["total_slots"] == 2  # uniform pi: no closing slot, two padding slots
    assert binding.lfmmi_graph_ordering_info(h, 0, 2)["total_slots"] == 0  # no rows at all
    h.close()


def _tiny():
    return {"num_states": 2, "num_pdfs": 2, "src": np.array([0, 1], np.int32),
            "dst": np.array([1, 0], np.int32), "pdf": np.array([0, 1], np.int32),
            "logw": np.zeros(2, np.float32), "init_prob": np.array([1, 0], np.float32),
            "final_prob": np.array([0, 1], np.float32)}


@pytest.mark.parametrize("field,value,code", [
    ("src", np.array([0, 2], np.int32), 2),
    ("dst", np.array([-1, 0], np.int32), 2),
    ("pdf", np.array([0, 2], np.int32), 2),
    ("logw", np.array([0, np.nan], np.float32), 2),
    ("logw", np.array([-np.inf, 0], np.float32), 2),
    ("init_prob", np.array([-1, 0], np.float32), 2),
    ("final_prob", np.array([np.inf, 0], np.float32), 2),
])
def test_bad_graphs_are_refused(field, value, code):
    g = _tiny()
    g[field] = value
    with pytest.raises(binding.LfmmiError) as ei:
        binding.lfmmi_graph_pack(g)
    assert ei.value.code == code and str(ei.value)


def test_unsupported_sizes_and_invalid_arguments():
    g = _tiny()
    g["num_pdfs"] = 20000
    with pytest.raises(binding.LfmmiError) as ei:
        binding.lfmmi_graph_pack(g)
    assert ei.value.code == 5
    big = {"num_states": 17000, "num_pdfs": 2, "src": np.zeros(1, np.int32),
           "dst": np.zeros(1, np.int32), "pdf": np.zeros(1, np.int32),
           "logw": np.zeros(1, np.float32), "init_prob": np.ones(17000, np.float32),
           "final_prob": np.ones(17000, np.float32)}
    with pytest.raises(binding.LfmmiError) as ei:
        binding.lfmmi_graph_pack(big)
    assert ei.value.code == 5
    lib = binding.load_library()
    out = ctypes.c_void_p()
    assert lib.lfmmi_graph_pack(0, 1, 0, None, None, None, None, None, None, ctypes.byref(out)) == 1
    assert lib.lfmmi_graph_pack(1, 1, 0, None, None, None, None, None, None, ctypes.byref(out)) == 1
    assert "null" in binding.lfmmi_last_error()
    assert lib.lfmmi_forward_backward(None, None, None, 1, 1, 1, 0.0, 1.0, 0, None, None, None, None) == 1
    # a packed-only handle cannot run
    h = binding.lfmmi_graph_pack(_tiny())
    lens = np.array([1], np.int32)
    rc = lib.lfmmi_forward_backward(h.handle, None, ctypes.c_void_p(lens.ctypes.data), 1, 1, 2,
                                    0.0, 1.0, 0, None, None, None, None)
    assert rc == 1 and "not uploaded" in binding.lfmmi_last_error()
    h.close()
    lib.lfmmi_graph_destroy(None)  # no-op


def test_fst_text_reader_round_trip_and_errors():
    from paper_2005_09824_amd import fst_text
    text = """0 1 3 3 0.5
1 1 3 3 0.25
1 2 5 5
2 0.125
"""
    g = fst_text.read_fst_text(text.splitlines())
    assert g["num_states"] == 3 and g["num_pdfs"] == 5
    assert g["src"].tolist() == [0, 1, 1] and g["dst"].tolist() == [1, 1, 2]
    assert g["pdf"].tolist() == [2, 2, 4]
    assert np.allclose(g["logw"], [-0.5, -0.25, 0.0])
    assert g["init_prob"].tolist() == [1.0, 0.0, 0.0]
    assert np.allclose(g["final_prob"], [0.0, 0.0, np.exp(-0.125)])
    # acceptor columns, explicit pdf count, another start state
    g2 = fst_text.read_fst_text(["4 2 1 0.5", "2 2 2", "2"], num_pdfs=7, acceptor=True)
    assert g2["num_states"] == 5 and g2["num_pdfs"] == 7 and g2["init_prob"][4] == 1.0
    assert g2["final_prob"][2] == 1.0 and g2["pdf"].tolist() == [0, 1]
    # what it writes it reads back
    back = fst_text.read_fst_text(fst_text.write_fst_text(g))
    for k in ("src", "dst", "pdf"):
        assert back[k].tolist() == g[k].tolist()
    assert np.allclose(back["logw"], g["logw"]) and np.allclose(back["final_prob"], g["final_prob"])
    # the packer accepts it
    h = binding.lfmmi_graph_pack(g)
    assert binding.lfmmi_graph_info(h)["total_arcs"] == 3
    h.close()
    for bad in (["0 1 0 0 1.0"], ["0 1 x 1"], ["0 1 2 2 inf"], ["3"], ["0 1 2 2 0.1 9"]):
        with pytest.raises(ValueError):
            fst_text.read_fst_text(bad)
    with pytest.raises(ValueError):
        fst_text.read_fst_text(["0 1 9 9"], num_pdfs=4)


def _hub_graph(seed=5, S=500, in_hub=300, out_hub=200):
    rng = np.random.default_rng(seed)
    g = workloads.random_den_graph(rng, S, 8, 30, 0.5)
    extra_src = rng.choice(S, size=in_hub, replace=False).astype(np.int32)       # into state 7
    extra_dst = rng.choice(S, size=out_hub, replace=False).astype(np.int32)      # out of state 11
    g["src"] = np.concatenate([g["src"], extra_src, np.full(out_hub, 11, np.int32)])
    g["dst"] = np.concatenate([g["dst"], np.full(in_hub, 7, np.int32), extra_dst])
    n = in_hub + out_hub
    g["pdf"] = np.concatenate([g["pdf"], rng.integers(0, 30, n).astype(np.int32)])
    g["logw"] = np.concatenate([g["logw"], np.log(rng.uniform(0.01, 0.2, n)).astype(np.float32)])
    return g


@pytest.mark.parametrize("nonuniform", [False, True])
def test_hub_states_get_slices_of_their_own(nonuniform):
    g = _hub_graph()
    if nonuniform:  # closing slots: the hub's leak-dot weight sits in lane 0 only
        pi = np.random.default_rng(1).uniform(0.1, 1.0, g["num_states"])
        g["init_prob"] = (pi / pi.sum()).astype(np.float32)
    h = binding.lfmmi_graph_pack(g)
    got, want, od = _unpack(h, 0, g)
    for o in range(3):
        assert got[o] == want, "ordering %d lost or changed arcs" % o
    # one hub slice per direction, a few slots wide instead of hundreds
    for o, (state, deg) in enumerate(((7, 300), (11, 200))):
        assert od[o]["hub_slices"] == 1
        s = int(np.flatnonzero(od[o]["slice_hub"])[0])
        assert od[o]["row_id"][s * 64] == state
        width = od[o]["slice_off"][s + 1] - od[o]["slice_off"][s]
        assert width <= (deg + 10 + 63) // 64 + 3 and width % 2 == 0
        assert od[o]["max_wave_slots"] < 64
    assert od[2]["hub_slices"] == 0
    h.close()


def _many_hubs(S, hubs_in, hubs_out, deg=600, seed=9, k=9, P=84):
    """Random graph plus `hubs_in` states with `deg` arcs into them and `hubs_out`
    states with `deg` arcs out of them."""
    rng = np.random.default_rng(seed)
    g = workloads.random_den_graph(rng, S, k, P, 0.5)
    src, dst = [g["src"]], [g["dst"]]
    for h in range(hubs_in):
        src.append(rng.choice(S, size=deg, replace=False).astype(np.int32))
        dst.append(np.full(deg, 10 + h, np.int32))
    for h in range(hubs_out):
        src.append(np.full(deg, 5000 % S + h, np.int32))
        dst.append(rng.choice(S, size=deg, replace=False).astype(np.int32))
    n = (hubs_in + hubs_out) * deg
    g["src"], g["dst"] = np.concatenate(src), np.concatenate(dst)
    g["pdf"] = np.concatenate([g["pdf"], rng.integers(0, P, n).astype(np.int32)])
    g["logw"] = np.concatenate([g["logw"], np.log(rng.uniform(0.001, 0.01, n)).astype(np.float32)])
    return g


@pytest.mark.parametrize("S,hubs_in,hubs_out", [
    (8000, 8, 0),     # 8000 states fit a 32 KB state vector, 8512 padded rows do not
    (8000, 20, 3),
    (12200, 0, 4),    # ... nor do 12288 + 3 * 64 the 48 KB map (P > 255: plain emission rows)
    (4000, 6, 6),     # fits: the register / hybrid kernels stay
])
def test_padded_rows_of_hub_slices_fit_the_chosen_kernels_lds_map(S, hubs_in, hubs_out):
    # every hub state gets a slice of its own, i.e. 63 padding rows: what must fit
    # the fixed LDS map of the register-resident kernels is the padded row count
    g = _many_hubs(S, hubs_in, hubs_out, P=300 if S > 12000 else 84)
    h = binding.lfmmi_graph_pack(g)
    for o in (0, 1):
        info = binding.lfmmi_graph_ordering_info(h, 0, o)
        assert info["hub_slices"] == (hubs_in, hubs_out)[o]
        assert info["slices"] * 64 >= S + 63 * info["hub_slices"]
        if info["register_slots"] > 0:
            assert info["slices"] * 64 <= info["lds_vector_rows"], info
        else:
            assert info["lds_vector_rows"] == 0
    rows = max(binding.lfmmi_graph_ordering_info(h, 0, o)["slices"] * 64 for o in (0, 1))
    resident = binding.lfmmi_graph_ordering_info(h, 0, 0)["register_slots"] > 0
    if S == 4000:
        assert resident and rows <= 8192
    elif S == 8000:   # the map with 48 KB state vectors (plain emission rows), or streamed arcs
        assert rows > 8192
        assert not resident or binding.lfmmi_graph_ordering_info(h, 0, 0)["lds_vector_rows"] == 12288
    else:
        assert rows > 12288 and not resident
    h.close()


def test_hub_slices_are_given_up_when_their_padding_rows_overflow_the_key_fields():
    # 16300 states and 5 out-degree hubs: 16640 BWD rows would not fit the 16-bit
    # (row * 4) fields of the arc records; the graph is packed without hub slices
    g = _many_hubs(16300, 0, 5, deg=300, k=2, P=40)
    h = binding.lfmmi_graph_pack(g)
    got, want, od = _unpack(h, 0, g)
    for o in range(3):
        assert got[o] == want, "ordering %d lost or changed arcs" % o
        assert od[o]["hub_slices"] == 0
    for o in (0, 1):
        assert od[o]["slices"] * 64 <= 16384
        assert int((od[o]["key"] & 0xFFFF).max()) // 4 < od[o]["slices"] * 64
    # OCC keys: both fields are row numbers
    assert int((od[2]["key"] >> 16).max()) // 4 < od[1]["slices"] * 64
    h.close()


def test_packer_finds_graphs_whose_pdf_is_a_function_of_the_entered_state(monkeypatch):
    wl6 = workloads.make_workload(6, scale={"B": 2, "Tlo": 3, "Thi": 4})
    g = wl6["den"]
    pdf_of = {}
    for d, p in zip(g["dst"].tolist(), g["pdf"].tolist()):
        assert pdf_of.setdefault(d, p) == p       # the generator's own promise
    h = binding.lfmmi_graph_pack(g)
    assert binding.lfmmi_graph_info(h)["emission_by_state"] == 1
    h.close()
    g2 = dict(g)
    pdf = g["pdf"].copy()
    pdf[5] = (pdf[5] + 1) % g["num_pdfs"]         # one arc breaks it
    g2["pdf"] = pdf
    h = binding.lfmmi_graph_pack(g2)
    assert binding.lfmmi_graph_info(h)["emission_by_state"] == 0
    h.close()
    # random pdf-ids per arc (the five named workloads' denominators): never
    h = binding.lfmmi_graph_pack(workloads.make_workload(2, scale={"S": 200, "B": 2})["den"])
    assert binding.lfmmi_graph_info(h)["emission_by_state"] == 0
    h.close()
    # phone-string numerators: yes (when asked for: with their few slots per wave the
    # variant does not pay); a batch with one graph that is not: no
    monkeypatch.setenv("LFMMI_GROUPED", "2")
    wl5 = workloads.make_workload(5, scale={"S": 100, "B": 3, "nlo": 3, "nhi": 6})
    h = binding.lfmmi_graph_pack_batch(wl5["num"])
    assert binding.lfmmi_graph_info(h)["emission_by_state"] == 1
    h.close()
    mixed = list(wl5["num"])
    bad = dict(mixed[1])
    bad["pdf"] = (mixed[1]["pdf"] + np.arange(len(mixed[1]["pdf"]))) % 84
    mixed[1] = bad
    h = binding.lfmmi_graph_pack_batch(mixed)
    assert binding.lfmmi_graph_info(h)["emission_by_state"] == 0
    h.close()


@pytest.mark.parametrize("over_pi,S,slots,leak", [
    ("1", 3000, 36, 2),   # values over init_prob: the first slots of a wave in registers
    ("0", 3000, 0, 1),    # a factor per arc: no room for any
    ("1", 1000, 16, 2), ("0", 1000, 16, 1),
])
def test_ordering_info_tells_what_runs_where_initial_probabilities_differ(over_pi, S, slots, leak, monkeypatch):
    monkeypatch.setenv("LFMMI_OVER_PI", over_pi)
    rng = np.random.default_rng(8)
    g = workloads.random_den_graph(rng, S, 14 if S == 3000 else 6, 100, 0.5)
    pi = rng.uniform(0.05, 1.0, S)
    g["init_prob"] = (pi / pi.sum()).astype(np.float32)
    h = binding.lfmmi_graph_pack(g)
    for o in (0, 1):
        info = binding.lfmmi_graph_ordering_info(h, 0, o)
        assert info["register_slots"] == slots and info["per_arc_leak"] == leak
        assert (slots == 16) == (info["max_wave_slots"] <= 16)
    h.close()


def test_bench_refuses_more_than_one_gpu():
    # one GPU is the whole target: the command says so and exits before it touches a device
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 2
    assert "one GPU" in r.stderr and r.stdout.strip() == ""


# the recursion kernel that the benchmark names is the one its workload runs
@pytest.mark.parametrize("S,k,by_state,hub,name", [
    (2000, 9, False, 0, "k_rec_line_arc"), (2000, 9, True, 0, "k_rec_line"), (2000, 14, False, 0, "k_rec_hybrid"),
    (5000, 9, False, 0, "k_rec_hybrid"), (2000, 9, False, 1500, "k_rec"), (16000, 3, False, 0, "k_rec"),
])
def test_bench_names_the_recursion_kernel(S, k, by_state, hub, name):
    import bench
    rng = np.random.default_rng(4)
    g = workloads.random_den_graph(rng, S, k, 84, 0.5)
    if by_state:
        g["pdf"] = rng.integers(0, 84, S).astype(np.int32)[g["dst"]]
    if hub:
        g["src"] = np.concatenate([g["src"], rng.choice(S, hub, replace=False).astype(np.int32)])
        for key, v in (("dst", 0), ("pdf", 0), ("logw", -3.0)):
            g[key] = np.concatenate([g[key], np.full(hub, v, g[key].dtype)])
    h = binding.lfmmi_graph_pack(g)
    assert bench.rec_kernel(binding, h) == name
    h.close()


# few rows for the occupancies: each row's sum is stored and added up again in every frame
@pytest.mark.parametrize("S,k,P,slices", [(1000, 9, 200, 8), (500, 11, 150, 8), (2000, 9, 84, 8), (300, 9, 84, 6), (100, 5, 10, 2)])
def test_occupancy_rows_are_few(S, k, P, slices):
    g = workloads.random_den_graph(np.random.default_rng(3), S, k, P, 0.5)
    h = binding.lfmmi_graph_pack(g)
    o = binding.lfmmi_graph_ordering_copy(h, 0, binding.ORD_OCC)
    h.close()
    assert o["slices"] == slices
    assert np.count_nonzero(o["w"]) == len(g["src"])


# ... and in large graphs no more of them for the few slots that one more a wave then saves: beyond 42
# slices the kernel's LDS map holds one frame a record, not two
@pytest.mark.parametrize("S,k,P,skew,slices", [(4160, 26, 1600, 2.5, 32), (4160, 25, 161, 1.0, 16)])
def test_occupancy_rows_of_large_graphs_are_few(S, k, P, skew, slices):
    rng = np.random.default_rng(1)
    src = np.repeat(np.arange(S), k).astype(np.int32)
    h = binding.lfmmi_graph_pack({
        "num_states": S, "num_pdfs": P, "src": src,
        "dst": ((src + 1 + np.tile(np.arange(k), S) * 37) % S).astype(np.int32),
        "pdf": (P * rng.random(len(src)) ** skew).astype(np.int32),
        "logw": np.full(len(src), -3, np.float32), "init_prob": np.full(S, 1 / S, np.float32),
        "final_prob": np.ones(S, np.float32)})
    o = binding.lfmmi_graph_ordering_copy(h, 0, binding.ORD_OCC)
    h.close()
    assert o["slices"] == slices
    assert np.count_nonzero(o["w"]) == len(src)


def graded_graph(S, high, low, share, P=84, by_state=False, hub=0, init="uniform"):
    """The first `share` of the states have `high` arcs in and out, all among themselves, the others
    `low`; `hub` arcs more lead into the last state."""
    rng = np.random.default_rng(1)
    n, src, dst = int(S * share), [], []
    for at, m, d in ((0, n, high), (n, S - n, low)):
        i = np.arange(m)
        for q in range(d):
            src.append(at + (i + q * 7) % m)
            dst.append(at + i)
    if hub:
        src.append(rng.choice(S, hub, replace=False))
        dst.append(np.full(hub, S - 1))
    src, dst = np.concatenate(src).astype(np.int32), np.concatenate(dst).astype(np.int32)
    p = np.ones(S) if init == "uniform" else rng.uniform(0.1, 1.0, S)
    if init == "wide":  # beyond what state values over initial probabilities can hold
        p[::3] *= 1e-30
    pdf = rng.integers(0, P, S)[dst] if by_state else rng.integers(0, P, len(src))
    return {"num_states": S, "num_pdfs": P, "src": src, "dst": dst, "pdf": pdf.astype(np.int32),
            "logw": np.log(rng.uniform(0.02, 0.2, len(src))).astype(np.float32),
            "init_prob": (p / p.sum()).astype(np.float32), "final_prob": np.ones(S, np.float32)}


# At most two slices a wave costs balance: only handles that run the straight line are dealt so. The
# others keep the slots and the kernel that they have without it (LFMMI_LINE=0).
@pytest.mark.parametrize("graphs,slots,registers,waves", [
    ([(1980, 24, 6, 0.2, 84, True, 1100)], [(24, 26)], 26, 16),
    ([(1980, 12, 5, 0.45, 84, False, 1100)], [(18, 20)], 20, 16),
    ([(1980, 10, 4, 0.2, 84, False, 1100, "varied")], [(36, 30)], 48, 8),
    ([(1600, 18, 4, 0.33, 84, False, 0, "wide")], [(40, 40)], 48, 8),
    ([(2040, 18, 4, 0.2, 4000)], [(18, 18)], 0, 16),
    # beside the graph that would take the straight line: another kind, a hub, too many rows
    ([(1980, 24, 6, 0.2, 84, True), (1000, 5, 4, 0.5)], [(24, 24), (6, 6)], 24, 16),
    ([(2040, 18, 4, 0.2), (1000, 5, 4, 0.5, 84, False, 600)], [(18, 18), (10, 6)], 20, 16),
    ([(2040, 18, 4, 0.2), (3000, 4, 4, 0.5)], [(18, 18), (12, 12)], 20, 16),
])
def test_two_slices_a_wave_only_for_the_straight_line(graphs, slots, registers, waves, monkeypatch):
    graphs = [graded_graph(*g) for g in graphs]
    taken = []
    for line in ("1", "0"):
        monkeypatch.setenv("LFMMI_LINE", line)
        h = binding.lfmmi_graph_pack_batch(graphs)
        info = [[binding.lfmmi_graph_ordering_info(h, g, o) for o in (0, 1)] for g in range(len(graphs))]
        assert all(i["lds_vector_rows"] != 2048 for pair in info for i in pair)
        assert [(f["max_wave_slots"], b["max_wave_slots"]) for f, b in info] == slots
        assert info[0][0]["register_slots"] == registers
        assert binding.lfmmi_graph_info(h)["rec_waves"] == waves
        taken.append(info)
        if line == "1":  # dealing anew has lost no arc
            for g, graph in enumerate(graphs):
                got, want, _ = _unpack(h, g, graph)
                assert all(a == want for a in got)
        h.close()
    assert taken[0] == taken[1]


def test_two_slices_a_wave_for_the_straight_line():
    h = binding.lfmmi_graph_pack(graded_graph(2040, 18, 4, 0.2))
    for o in (0, 1):
        c = binding.lfmmi_graph_ordering_copy(h, 0, o)
        assert c["lds_vector_rows"] == 2048 and c["max_wave_slots"] == 22
        widths = np.diff(c["slice_off"]).reshape(16, 2)
        assert np.all(widths[:, 0] <= widths[:, 1])
    h.close()
