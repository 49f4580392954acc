"""GPU parity of the HIP path (through the C ABI) against the fp64 oracle.

Small configs are compared in full; the full-size configs on sampled instances
(request, layer, value head), every node of each. Descriptor products (path_out,
path_len) are compared bit for bit. Invariants that hold bitwise on the GPU (policy
equivalence, commit == dumped node state, identity update, identical subtrees,
repeatability) are checked as such.
"""
from __future__ import annotations

import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU, skipped there
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
import paper_2609_23900_amd as L  # noqa: E402
from paper_2609_23900_amd.step import GdnTreeStep  # noqa: E402
from lumo_synth import configs, trees  # noqa: E402
from lumo_synth import operands as ops  # noqa: E402
import gpu_util as gu  # noqa: E402
import pins  # noqa: E402

SEQ_POLICIES = [L.LUMO_POLICY_PATHS, L.LUMO_POLICY_TWO_LEVEL, L.LUMO_POLICY_RECOMPUTE]

_WL = {}


def workload(name):
    if name not in _WL:
        _WL[name] = configs.build(name)
    return _WL[name]


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def run(wl, policy, *, with_conv=True, node_states=False, commit=True, arrays=None):
    say(f"[gpu] {wl.name} policy={policy} conv={with_conv} dump={node_states}")
    a = wl.arrays if arrays is None else arrays
    st = GdnTreeStep(n_req=wl.n_req, n_layers=wl.n_layers, h_k=wl.h_k, h_v=wl.h_v, d_k=wl.d_k,
                     d_v=wl.d_v, op_dtype=wl.op_dtype, node_off=wl.node_off,
                     parent=wl.parent_flat, n_rows=wl.n_rows,
                     arrays={k: v for k, v in a.items() if with_conv or k not in ("x", "hist", "w")},
                     policy=policy, max_path=wl.max_path, accepted=wl.accepted,
                     channels=wl.channels if with_conv else 0, with_node_states=node_states)
    if with_conv:
        st.conv()
    st.verify()
    if commit:
        st.commit()
    torch.cuda.synchronize()
    return st


# ---------------------------------------------------------------- small configs, full parity

@pytest.mark.parametrize("policy", SEQ_POLICIES)
@pytest.mark.parametrize("name", ["tiny", "layer1", "paper28"])
def test_small_config_parity(name, policy):
    wl = workload(name)
    st = run(wl, policy, node_states=(name != "layer1"))
    o = gu.to_np(st.o)
    inst = [(r, l, h) for r in range(wl.n_req) for l in range(wl.n_layers) for h in range(wl.h_v)]
    gu.check_outputs(wl, o, inst)
    ref_state, po, pl = oracle.commit(wl)
    assert np.array_equal(st.path_out.cpu().numpy(), po)
    assert np.array_equal(st.path_len.cpu().numpy(), pl)
    gu.check_states(wl, st.state.cpu().numpy(), ref_state, inst)
    # conv and conv-history publication
    y = gu.to_np(st.y)
    yref = oracle.conv_all(wl)
    rows = oracle.plan.flat_rows(wl.parents, wl.row_off)
    assert gu.max_rel(y[:, rows], yref[:, rows]) <= gu.out_tol(wl)
    href = oracle.conv_hist_publish(wl, po, pl)
    assert np.array_equal(gu.to_np(st.hist).astype(np.float64), href)


@pytest.mark.parametrize("name", ["tiny", "paper28"])
def test_commit_equals_dumped_node_state(name):
    """Publishing the path to node i reproduces the verified state of i bit for bit."""
    wl = workload(name)
    st = run(wl, L.LUMO_POLICY_PATHS, with_conv=False, node_states=True, commit=False)
    ns = st.node_states.cpu().numpy()
    rows = gu.node_rows(wl, 0)
    for node in range(len(wl.parents[0])):
        st.reset_state()
        st.accepted.fill_(node)
        st.commit()
        torch.cuda.synchronize()
        s = st.state.cpu().numpy()
        for l in range(wl.n_layers):
            for h in range(wl.h_v):
                assert np.array_equal(s[0, l, h], ns[l, rows[node], h]), (node, l, h)


def test_policies_bitwise_identical():
    wl = workload("paper28")
    outs = [gu.to_np(run(wl, p, with_conv=False, commit=False).o) for p in SEQ_POLICIES]
    rows = oracle.plan.flat_rows(wl.parents, wl.row_off)
    for o in outs[1:]:
        assert np.array_equal(o[:, rows], outs[0][:, rows])


# ---------------------------------------------------------------- full-size configs, sampled

@pytest.mark.parametrize("name,policy,n_inst", [
    ("batched", L.LUMO_POLICY_PATHS, 24),
    ("widedeep", L.LUMO_POLICY_PATHS, 12),
    ("widedeep", L.LUMO_POLICY_TWO_LEVEL, 6),
    ("chainmix", L.LUMO_POLICY_RECOMPUTE, 16),
    ("chainmix", L.LUMO_POLICY_PATHS, 8),
])
def test_full_size_sampled_parity(name, policy, n_inst):
    wl = workload(name)
    st = run(wl, policy)
    o = gu.to_np(st.o)
    inst = gu.sample_instances(wl, n_inst, seed=7)
    worst = gu.check_outputs(wl, o, inst)
    say(f"  outputs worst max-rel {worst:.3e}")
    ref_state, po, pl = oracle.commit(wl)
    assert np.array_equal(st.path_out.cpu().numpy(), po)
    assert np.array_equal(st.path_len.cpu().numpy(), pl)
    ws = gu.check_states(wl, st.state.cpu().numpy(), ref_state, inst)
    say(f"  states worst max-rel {ws:.3e}")
    # conv on two sampled layers, history on all
    y = gu.to_np(st.y)
    rows = oracle.plan.flat_rows(wl.parents, wl.row_off)
    for l in sorted({0, wl.n_layers - 1}):
        sub = {"x": wl.arrays["x"][l:l + 1], "hist": wl.arrays["hist"][:, l:l + 1],
               "w": wl.arrays["w"][l:l + 1]}
        one = configs.Workload(**{**wl.__dict__, "n_layers": 1, "arrays": sub})
        yref = oracle.conv_all(one)
        assert gu.max_rel(y[l][rows], yref[0][rows]) <= gu.out_tol(wl)
    href = oracle.conv_hist_publish(wl, po, pl)
    assert np.array_equal(gu.to_np(st.hist).astype(np.float64), href)


# ---------------------------------------------------------------- invariants and edge cases

def test_identity_update_keeps_state_bitwise():
    wl = configs.build("paper28", with_conv=False)
    a = dict(wl.arrays)
    a["beta"] = np.zeros_like(a["beta"])
    a["g"] = np.zeros_like(a["g"])  # alpha = exp(0) = 1
    st = run(wl, L.LUMO_POLICY_PATHS, with_conv=False, arrays=a)
    assert np.array_equal(st.state.cpu().numpy(), a["state0"])


def test_identical_sibling_subtrees_bitwise():
    par = np.array([-1, 0, 0, 1, 2, 3, 4, 1, 2], np.int32)
    wl = pins.make_wl([par], d_k=128, d_v=128, h_k=2, h_v=4, op_dtype=ops.BF16, max_path=4)
    wl.arrays = ops.make_gdn_operands(3, n_req=1, n_layers=1, total_rows=9, h_k=2, h_v=4,
                                      d_k=128, d_v=128, op_dtype=ops.BF16)
    rows = gu.node_rows(wl, 0)
    for x, y in ((1, 2), (3, 4), (5, 6), (7, 8)):
        for key in ("q", "k", "v", "g", "beta"):
            wl.arrays[key][:, rows[y]] = wl.arrays[key][:, rows[x]]
    for policy in SEQ_POLICIES:
        o = run(wl, policy, with_conv=False, commit=False).o.cpu()
        for x, y in ((1, 2), (3, 4), (5, 6), (7, 8)):
            assert torch.equal(o[:, rows[x]], o[:, rows[y]])


def test_pad_rows_never_read_or_written():
    wl = configs.build("paper28")
    a = {k: v.copy() for k, v in wl.arrays.items()}
    rows = set(oracle.plan.flat_rows(wl.parents, wl.row_off).tolist())
    pad = [r for r in range(wl.total_rows) if r not in rows]
    assert pad
    nan_bf16 = np.uint16(0x7FC0)
    for key in ("q", "k", "v", "x"):
        a[key][:, pad] = nan_bf16
    for key in ("g", "beta"):
        a[key][:, pad] = np.nan
    st = run(wl, L.LUMO_POLICY_TWO_LEVEL, arrays=a)
    o = gu.to_np(st.o)
    assert np.all(o[:, pad] == 0)           # untouched zero fill
    assert np.all(np.isfinite(o[:, sorted(rows)]))
    assert np.all(np.isfinite(st.state.cpu().numpy()))
    y = gu.to_np(st.y)
    assert np.all(y[:, pad] == 0) and np.all(np.isfinite(y[:, sorted(rows)]))
    gu.check_outputs(wl, o, [(0, 0, 0), (0, 0, 31)])


def test_accepted_edge_cases():
    wl = configs.build("paper28", with_conv=True)
    cases = [(-1, 0), (0, 1), (27, None), (28, -1), (-2, -1), (99, -1)]
    for acc, want_len in cases:
        st = run(wl, L.LUMO_POLICY_RECOMPUTE, with_conv=True, commit=False)
        st.accepted.fill_(acc)
        st.max_path = 12
        hist0 = st.hist.clone()
        st.commit()
        torch.cuda.synchronize()
        pl = int(st.path_len.cpu()[0])
        po = st.path_out.cpu().numpy()[0]
        # the descriptor products equal the oracle's bit for bit, invalid selections included
        path, L_ = oracle.plan.accepted_path(wl.parents[0], acc, 12)
        _, opo, opl = oracle.commit(wl, accepted=np.array([acc], np.int32), max_path=12)
        assert pl == L_ == int(opl[0]) and list(po) == path == opo[0].tolist()
        if want_len is not None:
            assert pl == want_len
        if pl <= 0:
            assert np.all(po == -1)
            assert torch.equal(st.state, st.state0)
            assert torch.equal(st.hist, hist0)
    # a path longer than max_path is refused without touching the state
    st = run(wl, L.LUMO_POLICY_RECOMPUTE, with_conv=False, commit=False)
    deep = int(np.argmax(trees.depths(wl.parents[0])))
    st.accepted.fill_(deep)
    st.max_path = 4
    st.path_out = torch.full((1, 4), -7, dtype=torch.int32, device="cuda")
    st.commit()
    torch.cuda.synchronize()
    assert int(st.path_len.cpu()[0]) == -1 and torch.equal(st.state, st.state0)
    ost, opo, opl = oracle.commit(wl, accepted=np.array([deep], np.int32), max_path=4)
    assert int(opl[0]) == -1 and st.path_out.cpu().numpy().tolist() == opo.tolist()
    assert np.array_equal(ost, wl.arrays["state0"].astype(np.float64))


def test_empty_batch_and_root_only_requests():
    parents = [np.array([-1], np.int32), np.array([-1, 0], np.int32), np.array([-1], np.int32)]
    wl = pins.make_wl(parents, d_k=64, d_v=32, h_k=1, h_v=2, op_dtype=ops.BF16, n_rows=[1, 3, 2],
                      max_path=2, n_layers=2)
    wl.arrays = ops.make_gdn_operands(5, n_req=3, n_layers=2, total_rows=6, h_k=1, h_v=2,
                                      d_k=64, d_v=32, op_dtype=ops.BF16)
    wl.accepted = np.array([0, 1, -1], np.int32)
    st = run(wl, L.LUMO_POLICY_PATHS, with_conv=False)
    inst = [(r, l, h) for r in range(3) for l in range(2) for h in range(2)]
    gu.check_outputs(wl, gu.to_np(st.o), inst)
    ref, po, pl = oracle.commit(wl)
    assert np.array_equal(st.path_len.cpu().numpy(), pl)
    gu.check_states(wl, st.state.cpu().numpy(), ref, inst)
    # n_req = 0: every entry point is a no-op
    d = L.dims(0, 1, 1, 1, 16, 16, 0)
    desc = L.TreeDesc.build(np.array([0], np.int32), np.zeros(0, np.int32), np.zeros(0, np.int32))
    e = torch.zeros(16, device="cuda")
    L.lumo_tree_gdn_verify(d, desc, e, e, e, e, e, e, e)
    L.lumo_gdn_commit(d, desc, 1, e.int(), e.int(), e.int(), e, e, e, e, e)
    torch.cuda.synchronize()


def test_repeatability_bitwise():
    wl = workload("layer1")
    o1 = run(wl, L.LUMO_POLICY_PATHS).o.cpu()
    o2 = run(wl, L.LUMO_POLICY_PATHS).o.cpu()
    assert torch.equal(o1, o2)


def test_multi_cycle_continuation():
    """verify -> commit -> verify on the next tree from the published state."""
    wl1 = configs.build("layer1", with_conv=False)
    st = run(wl1, L.LUMO_POLICY_PATHS, with_conv=False)
    wl2 = configs.build("layer1", seed=101, with_conv=False)
    ref_state, _, _ = oracle.commit(wl1)
    a2 = dict(wl2.arrays)
    a2["state0"] = ref_state.astype(np.float32)          # oracle-published state, rounded
    st2 = GdnTreeStep.from_workload(wl2, policy=L.LUMO_POLICY_PATHS, with_conv=False)
    st2.verify(state0=st.state)                          # GPU-published state
    torch.cuda.synchronize()
    gu.check_outputs(wl2, gu.to_np(st2.o), gu.sample_instances(wl2, 8), arrays=a2)


# ---------------------------------------------------------------- captured commit graph

def test_commit_graph_replays():
    wl = workload("chainmix")
    st = run(wl, L.LUMO_POLICY_RECOMPUTE, with_conv=True, commit=False)
    hist0 = st.hist.clone()
    g = st.commit_graph(with_conv=True)
    rng = np.random.default_rng(5)
    inst = gu.sample_instances(wl, 6, seed=3)
    for rep in range(24):
        lens = rng.integers(0, 17, size=wl.n_req)
        acc = np.array([configs._pick_accepted(rng, p, int(L_), int(L_)) if L_ > 0 else -1
                        for p, L_ in zip(wl.parents, lens)], np.int32)
        st.state.copy_(st.state0)
        st.hist.copy_(hist0)
        st.accepted.copy_(torch.from_numpy(acc))
        torch.cuda.synchronize()
        g.launch()
        torch.cuda.synchronize()
        ref, po, pl = oracle.commit(wl, accepted=acc)
        assert np.array_equal(st.path_out.cpu().numpy(), po), rep
        assert np.array_equal(st.path_len.cpu().numpy(), pl), rep
        gu.check_states(wl, st.state.cpu().numpy(), ref, inst)
        href = oracle.conv_hist_publish(wl, po, pl)
        assert np.array_equal(gu.to_np(st.hist).astype(np.float64), href), rep
    g.close()


def test_commit_graph_replays_prepared():
    """The captured committer with operand preparation (Sec. V-A with Sec. IV-B): 24
    replays with a changing device accepted_node, each against the oracle's prepared
    commit; the unprepared graph over the same raw operands publishes something else."""
    wl = workload("widedeep")
    a, oprep, gprep = _prep_inputs(wl, QKN | RAWG, seed=85)
    st = _prep_step(wl, a, gprep, policy=L.LUMO_POLICY_WY)
    g = st.commit_graph(with_conv=False)
    rng = np.random.default_rng(6)
    inst = gu.sample_instances(wl, 8, seed=4)
    for rep in range(24):
        lens = rng.integers(0, 17, size=wl.n_req)
        acc = np.array([configs._pick_accepted(rng, p, int(L_), int(L_)) if L_ > 0 else -1
                        for p, L_ in zip(wl.parents, lens)], np.int32)
        st.state.copy_(st.state0)
        st.accepted.copy_(torch.from_numpy(acc))
        torch.cuda.synchronize()
        g.launch()
        torch.cuda.synchronize()
        ref, po, pl = oracle.commit(wl, accepted=acc, arrays=a, prep=oprep)
        assert np.array_equal(st.path_out.cpu().numpy(), po), rep
        assert np.array_equal(st.path_len.cpu().numpy(), pl), rep
        gu.check_states(wl, st.state.cpu().numpy(), ref, inst)
    g.close()
    plain = _prep_step(wl, a, None, policy=L.LUMO_POLICY_WY)
    gp = plain.commit_graph(with_conv=False)
    plain.accepted.copy_(torch.from_numpy(acc))
    gp.launch()
    torch.cuda.synchronize()
    gp.close()
    r = int(np.argmax(pl))
    assert pl[r] > 1 and gu.max_rel(plain.state.cpu().numpy()[r], ref[r]) > 1e-2


# ---------------------------------------------------------------- negative controls

def test_negative_control_sibling_swap_detected():
    """Swapping two siblings' operand rows must break parity (the test has teeth)."""
    wl = configs.build("paper28", with_conv=False)
    a = {k: v.copy() for k, v in wl.arrays.items()}
    par = wl.parents[0]
    ch = oracle.plan.children(par)
    p = next(i for i in range(len(par)) if len(ch[i]) >= 2)
    x, y = ch[p][0], ch[p][1]
    rows = gu.node_rows(wl, 0)
    for key in ("k", "v", "g", "beta"):
        a[key][:, [rows[x], rows[y]]] = a[key][:, [rows[y], rows[x]]]
    o = gu.to_np(run(wl, L.LUMO_POLICY_PATHS, with_conv=False, commit=False, arrays=a).o)
    with pytest.raises(AssertionError):
        gu.check_outputs(wl, o, [(0, 0, h) for h in range(wl.h_v)])


def test_negative_control_zero_replay_detected():
    wl = configs.build("paper28", with_conv=False)
    st = run(wl, L.LUMO_POLICY_PATHS, with_conv=False, commit=False)
    st.accepted.fill_(-1)
    st.commit()
    torch.cuda.synchronize()
    ref, _, _ = oracle.commit(wl)
    with pytest.raises(AssertionError):
        gu.check_states(wl, st.state.cpu().numpy(), ref, [(0, 0, 0)])


# ---------------------------------------------------------------- WY form on MFMA

@pytest.mark.parametrize("name,n_inst", [("layer1", 32), ("paper28", 32), ("batched", 24),
                                          ("widedeep", 12), ("chainmix", 16)])
def test_wy_parity(name, n_inst):
    wl = workload(name)
    st = run(wl, L.LUMO_POLICY_WY)
    o = gu.to_np(st.o)
    worst = gu.check_outputs(wl, o, gu.sample_instances(wl, n_inst, seed=11))
    say(f"  wy outputs worst max-rel {worst:.3e}")
    rows = set(oracle.plan.flat_rows(wl.parents, wl.row_off).tolist())
    pad = [r for r in range(wl.total_rows) if r not in rows]
    if pad:
        assert np.all(o[:, pad] == 0)
    ref_state, po, pl = oracle.commit(wl)
    assert np.array_equal(st.path_len.cpu().numpy(), pl)
    gu.check_states(wl, st.state.cpu().numpy(), ref_state, gu.sample_instances(wl, n_inst, seed=12))


# ------------------------------------------ WY form beyond the bf16 kernel for short paths

def _wyv_case(case):
    """Shapes the bf16 matrix-core kernel for paths of up to 17 nodes does not take: fp32 at d =
    128 and bf16 paths of up to 32 nodes have matrix-core kernels of their own, heads
    below 128 run on the vector ALUs (more of those: test_gpu_wyv.py)."""
    rng = np.random.default_rng(91)
    if case == "tiny_f32":
        return configs.build("tiny", with_conv=False), [(0, 0, 0)]
    if case == "layer1_f32":  # fp32 operands at the benchmark's head shape
        wl = configs.build("layer1", with_conv=False, op_dtype=ops.F32)
        return wl, [(0, 0, h) for h in range(0, 32, 3)]
    if case == "deep_bf16":   # 30-node chain and a 25-level tree: beyond the 17-node limit
        parents = [trees.chain(30), trees.random_tree(rng, 60, 25, trees.bmax_uniform(2)), np.zeros(0, np.int32)]
        n_rows = [30, 63, 2]
        wl = pins.make_wl(parents, d_k=128, d_v=128, h_k=2, h_v=4, op_dtype=ops.BF16, n_rows=n_rows,
                          n_layers=2, max_path=30)
    elif case == "d64_group4_bf16":  # four value heads of 128 columns per key head: 8 waves, two blocks
        parents = [trees.random_tree(rng, 45, 8, trees.bmax_uniform(4)), trees.FIG1_PARENT]
        n_rows = [47, 7]
        wl = pins.make_wl(parents, d_k=64, d_v=128, h_k=1, h_v=4, op_dtype=ops.BF16, n_rows=n_rows,
                          n_layers=2, max_path=8)
    else:  # "d32_v16_f32": value columns fewer than a wave's lanes
        parents = [trees.random_tree(rng, 37, 12, trees.bmax_uniform(3))]
        n_rows = [40]
        wl = pins.make_wl(parents, d_k=32, d_v=16, h_k=2, h_v=2, op_dtype=ops.F32, n_rows=n_rows,
                          n_layers=1, max_path=12)
    wl.arrays = ops.make_gdn_operands(92, n_req=wl.n_req, n_layers=wl.n_layers, total_rows=wl.total_rows,
                                      h_k=wl.h_k, h_v=wl.h_v, d_k=wl.d_k, d_v=wl.d_v, op_dtype=wl.op_dtype)
    inst = [(r, l, h) for r in range(wl.n_req) for l in range(wl.n_layers) for h in range(wl.h_v)
            if len(wl.parents[r])]
    return wl, inst


@pytest.mark.parametrize("case", ["tiny_f32", "layer1_f32", "deep_bf16", "d64_group4_bf16", "d32_v16_f32"])
def test_wyv_parity(case):
    """The WY policy on fp32 operands, d < 128 and paths beyond 17 nodes: outputs against the oracle, NaN pad rows neither read nor
    written, and the sequential scan of the same plan shape within the output tolerance."""
    wl, inst = _wyv_case(case)
    rows = set(oracle.plan.flat_rows(wl.parents, wl.row_off).tolist())
    pad = [x for x in range(wl.total_rows) if x not in rows]
    a = dict(wl.arrays)
    nan = np.float32(np.nan) if wl.op_dtype == ops.F32 else np.uint16(0x7FC0)
    for key in ("q", "k", "v"):
        a[key] = a[key].copy()
        a[key][:, pad] = nan
    for key in ("g", "beta"):
        a[key] = a[key].copy()
        a[key][:, pad] = np.nan
    say(f"[gpu] wy {case}")
    st = run(wl, L.LUMO_POLICY_WY, with_conv=False, commit=False, arrays=a)
    o = gu.to_np(st.o)
    worst = gu.check_outputs(wl, o, inst, arrays=a)
    say(f"  outputs worst max-rel {worst:.3e}")
    if pad:
        assert np.all(o[:, pad] == 0)
    seq = gu.to_np(run(wl, L.LUMO_POLICY_RECOMPUTE, with_conv=False, commit=False, arrays=a).o)
    rl = sorted(rows)
    assert gu.max_rel(o[:, rl], seq[:, rl]) <= gu.out_tol(wl)
    # two runs give the same bits
    o2 = gu.to_np(run(wl, L.LUMO_POLICY_WY, with_conv=False, commit=False, arrays=a).o)
    assert np.array_equal(o.view(np.uint32), o2.view(np.uint32))


def test_wyv_prep_parity():
    """Operand preparation (Sec. IV-B) in the WY kernel of fp32 operands at d = 128."""
    wl, inst = _wyv_case("layer1_f32")
    rng = np.random.default_rng(93)
    a = dict(wl.arrays)
    for key in ("q", "k"):
        a[key] = (a[key] * rng.uniform(0.3, 3.0, size=a[key].shape[:-1] + (1,))).astype(np.float32)
    a["g"] = rng.standard_normal(a["g"].shape).astype(np.float32)
    a["beta"] = rng.standard_normal(a["beta"].shape).astype(np.float32)
    a_log = (0.5 * rng.standard_normal((wl.n_layers, wl.h_v))).astype(np.float32)
    dt_bias = rng.standard_normal((wl.n_layers, wl.h_v)).astype(np.float32)
    flags = QKN | RAWG
    oprep = oracle.Prep(flags, 1e-6, a_log, dt_bias)
    gprep = L.Prep(flags, 1e-6, torch.from_numpy(a_log).cuda(), torch.from_numpy(dt_bias).cuda())
    st = _prep_step(wl, a, gprep, policy=L.LUMO_POLICY_WY)
    st.verify()
    torch.cuda.synchronize()
    worst = _check_prep_outputs(wl, gu.to_np(st.o), a, oprep, inst, tol=gu.TOL_F32)
    say(f"[gpu] wy fp32 prep: outputs worst max-rel {worst:.3e}")


def test_wy_agrees_with_sequential_scan():
    """WY and the sequential scan compute the same recurrence: outputs within bf16 rounding."""
    wl = workload("layer1")
    o_seq = gu.to_np(run(wl, L.LUMO_POLICY_PATHS, with_conv=False, commit=False).o)
    o_wy = gu.to_np(run(wl, L.LUMO_POLICY_WY, with_conv=False, commit=False).o)
    rows = oracle.plan.flat_rows(wl.parents, wl.row_off)
    for h in range(wl.h_v):
        a, b = o_seq[0, rows, h], o_wy[0, rows, h]
        assert gu.max_rel(b, a) <= 2 ** -7, h


def test_wy_identical_sibling_subtrees():
    par = np.array([-1, 0, 0, 1, 2, 3, 4, 1, 2], np.int32)
    wl = pins.make_wl([par], d_k=128, d_v=128, h_k=2, h_v=4, op_dtype=ops.BF16, max_path=4)
    wl.arrays = ops.make_gdn_operands(3, n_req=1, n_layers=1, total_rows=9, h_k=2, h_v=4,
                                      d_k=128, d_v=128, op_dtype=ops.BF16)
    rows = gu.node_rows(wl, 0)
    for x, y in ((1, 2), (3, 4), (5, 6), (7, 8)):
        for key in ("q", "k", "v", "g", "beta"):
            wl.arrays[key][:, rows[y]] = wl.arrays[key][:, rows[x]]
    o = run(wl, L.LUMO_POLICY_WY, with_conv=False, commit=False).o.cpu()
    for x, y in ((1, 2), (3, 4), (5, 6), (7, 8)):
        assert torch.equal(o[:, rows[x]], o[:, rows[y]])
    gu.check_outputs(wl, gu.to_np(o.cuda()), [(0, 0, h) for h in range(4)])


@pytest.mark.parametrize("h_k,h_v", [(4, 4), (2, 8), (1, 2)])
def test_wy_head_groupings(h_k, h_v):
    """One, two and four value heads per key head (blocks of one or two value heads)."""
    rng = np.random.default_rng(17)
    parents = [trees.random_tree(rng, 45, 8, trees.bmax_uniform(4)), trees.FIG1_PARENT]
    wl = pins.make_wl(parents, d_k=128, d_v=128, h_k=h_k, h_v=h_v, op_dtype=ops.BF16,
                      n_rows=[48, 7], n_layers=2, max_path=8)
    wl.arrays = ops.make_gdn_operands(23, n_req=2, n_layers=2, total_rows=55, h_k=h_k, h_v=h_v,
                                      d_k=128, d_v=128, op_dtype=ops.BF16)
    st = run(wl, L.LUMO_POLICY_WY, with_conv=False, commit=False)
    inst = [(r, l, h) for r in range(2) for l in range(2) for h in range(h_v)]
    gu.check_outputs(wl, gu.to_np(st.o), inst)


def test_wy_deep_chain_and_ragged_requests():
    """Chains of 17 nodes (the WY depth limit), 1-node and 40-node requests, padding."""
    rng = np.random.default_rng(9)
    parents = [trees.chain(17), np.array([-1], np.int32),
               trees.random_tree(rng, 40, 9, trees.bmax_uniform(3)), trees.chain(5)]
    wl = pins.make_wl(parents, d_k=128, d_v=128, h_k=4, h_v=8, op_dtype=ops.BF16,
                      n_rows=[17, 3, 41, 5], n_layers=2, max_path=17)
    wl.arrays = ops.make_gdn_operands(21, n_req=4, n_layers=2, total_rows=66, h_k=4, h_v=8,
                                      d_k=128, d_v=128, op_dtype=ops.BF16)
    st = run(wl, L.LUMO_POLICY_WY, with_conv=False, commit=False)
    inst = [(r, l, h) for r in range(4) for l in range(2) for h in (0, 3, 7)]
    gu.check_outputs(wl, gu.to_np(st.o), inst)


# ---------------------------------------------------------------- deferred publication

def _pending_pair(h_k, h_v, seed=31):
    """Two iterations over the same 5 requests: a chain of 20 accepted whole (two staging
    rounds), a short path into a request with no nodes next time, an empty and an
    invalid pending path, and a random tree of two chunks."""
    rng = np.random.default_rng(seed)
    prev_par = [trees.chain(20), np.array([-1, 0, 0, 1], np.int32), np.array([-1], np.int32),
                trees.FIG1_PARENT, trees.random_tree(rng, 40, 8, trees.bmax_uniform(3))]
    cur_par = [trees.random_tree(rng, 30, 8, trees.bmax_uniform(3)), np.zeros(0, np.int32),
               trees.chain(5), np.zeros(0, np.int32),
               trees.random_tree(rng, 50, 9, trees.bmax_uniform(4))]
    prev = pins.make_wl(prev_par, d_k=128, d_v=128, h_k=h_k, h_v=h_v, op_dtype=ops.BF16,
                        n_rows=[20, 5, 1, 9, 40], n_layers=2, max_path=24)
    prev.arrays = ops.make_gdn_operands(seed, n_req=5, n_layers=2, total_rows=prev.total_rows,
                                        h_k=h_k, h_v=h_v, d_k=128, d_v=128, op_dtype=ops.BF16)
    deep = int(np.argmax(trees.depths(prev_par[4])))
    prev.accepted = np.array([19, 3, -1, 99, deep], np.int32)
    cur = pins.make_wl(cur_par, d_k=128, d_v=128, h_k=h_k, h_v=h_v, op_dtype=ops.BF16,
                       n_rows=[31, 2, 5, 0, 50], n_layers=2, max_path=16)
    cur.arrays = ops.make_gdn_operands(seed + 1, n_req=5, n_layers=2, total_rows=cur.total_rows,
                                       h_k=h_k, h_v=h_v, d_k=128, d_v=128, op_dtype=ops.BF16)
    return prev, cur


def _step(wl, policy, with_conv=False):
    a = {k: v for k, v in wl.arrays.items() if with_conv or k not in ("x", "hist", "w")}
    return GdnTreeStep(n_req=wl.n_req, n_layers=wl.n_layers, h_k=wl.h_k, h_v=wl.h_v, d_k=wl.d_k,
                       d_v=wl.d_v, op_dtype=wl.op_dtype, node_off=wl.node_off,
                       parent=wl.parent_flat, n_rows=wl.n_rows, arrays=a, policy=policy,
                       max_path=wl.max_path, accepted=wl.accepted,
                       channels=wl.channels if with_conv else 0)


@pytest.mark.parametrize("h_k,h_v", [(2, 4), (4, 4)])
def test_verify_pending_parity(h_k, h_v):
    """Published state = the oracle's commit of the previous iteration; outputs = the
    oracle's verification from that state; untouched requests stay bitwise."""
    prev, cur = _pending_pair(h_k, h_v)
    say(f"[gpu] verify_pending h_k={h_k} h_v={h_v}")
    sp = _step(prev, L.LUMO_POLICY_PATHS)
    sp.commit(defer=True)
    torch.cuda.synchronize()
    # the oracle refuses the invalid path of request 3; an invalid path publishes nothing,
    # as an empty one does, and reports length -1
    acc = prev.accepted.copy()
    acc[3] = -1
    ref_state, po, pl = oracle.commit(prev, accepted=acc)
    pl[3] = -1
    assert np.array_equal(sp.path_len.cpu().numpy(), pl)
    assert np.array_equal(sp.path_out.cpu().numpy(), po)
    assert torch.equal(sp.state, sp.state0)  # the deferred commit did not replay
    sc = _step(cur, L.LUMO_POLICY_WY)
    sc.verify_pending(sp, state=sp.state)
    torch.cuda.synchronize()
    st = sp.state.cpu().numpy()
    s0 = sp.state0.cpu().numpy()
    inst = [(r, l, h) for r in range(5) for l in range(2) for h in range(h_v)]
    for (r, l, h) in inst:
        if pl[r] <= 0:
            assert np.array_equal(st[r, l, h], s0[r, l, h]), (r, l, h)
    worst = gu.check_states(prev, st, ref_state, inst)
    say(f"  published state worst max-rel {worst:.3e}")
    a2 = dict(cur.arrays)
    a2["state0"] = ref_state.astype(np.float32)
    live = [(r, l, h) for (r, l, h) in inst if len(cur.parents[r]) > 0]
    worst = gu.check_outputs(cur, gu.to_np(sc.o), live, arrays=a2)
    say(f"  outputs worst max-rel {worst:.3e}")


def test_verify_pending_without_pending_is_plain_verify():
    """No pending path anywhere: bitwise the plain WY verification, state untouched."""
    wl = workload("layer1")
    s1 = run(wl, L.LUMO_POLICY_WY, with_conv=False, commit=False)
    s2 = _step(wl, L.LUMO_POLICY_WY)
    s2.accepted.fill_(-1)
    s2.commit(defer=True)
    s2.verify_pending(s2)
    torch.cuda.synchronize()
    assert int(s2.path_len.cpu()[0]) == 0
    assert torch.equal(s1.o, s2.o)
    assert torch.equal(s2.state, s2.state0)


def test_verify_pending_full_size_sampled():
    """The batched workload, its accepted paths deferred into the next verification."""
    wl = workload("batched")
    say("[gpu] verify_pending batched")
    st = GdnTreeStep.from_workload(wl, policy=L.LUMO_POLICY_WY, with_conv=False)
    st.commit(defer=True)
    st.verify_pending(st)
    torch.cuda.synchronize()
    ref_state, _, pl = oracle.commit(wl)
    assert np.array_equal(st.path_len.cpu().numpy(), pl)
    inst = gu.sample_instances(wl, 24, seed=21)
    gu.check_states(wl, st.state.cpu().numpy(), ref_state, inst)
    a2 = dict(wl.arrays)
    a2["state0"] = ref_state.astype(np.float32)
    gu.check_outputs(wl, gu.to_np(st.o), inst, arrays=a2)



@pytest.mark.parametrize("name,over", [("batched", {}), ("widedeep", dict(n_req=4, n_layers=4))])
def test_layer_calls_equal_stacked_call(name, over):
    """A call for one layer of these workloads has fewer blocks of two value heads than
    the device has CUs and runs four 32-column waves per value head; the call for all
    layers runs the 64-column pair blocks. Their outputs and published state banks must
    agree bit for bit (same operations in the same order), on the deferred verification
    of the batched workload (depth <= 8) and of four 256-node, 16-level trees."""
    wl = configs.build(name, with_conv=False, **over)
    st = GdnTreeStep.from_workload(wl, policy=L.LUMO_POLICY_WY, with_conv=False)
    d = st.dims
    assert d.n_req * d.n_layers * d.h_k >= 256 > d.n_req * d.h_k  # the two forms are taken
    say(f"[gpu] one-layer calls against the stacked call, {name} {over}")
    st.commit(defer=True)
    st.verify_pending(st)
    torch.cuda.synchronize()
    o1 = torch.zeros_like(st.o)
    s1 = st.state0.clone()
    d1 = L.dims(d.n_req, 1, d.h_k, d.h_v, d.d_k, d.d_v, d.op_dtype)
    for l in range(d.n_layers):
        sl = s1[:, l:l + 1].contiguous()
        t = {key: st.t[key][l] for key in ("q", "k", "v", "g", "beta")}
        L.lumo_tree_gdn_verify_pending(d1, st.desc, t["q"], t["k"], t["v"], t["g"], t["beta"], sl, o1[l],
                                       st.desc, st.max_path, st.path_out, st.path_len, t["k"], t["v"],
                                       t["g"], t["beta"])
        s1[:, l:l + 1] = sl
    torch.cuda.synchronize()
    assert not torch.equal(st.state, st.state0)  # paths were published
    assert torch.equal(o1.view(torch.int16), st.o.view(torch.int16)), int((o1 != st.o).sum())
    assert torch.equal(s1, st.state), int((s1 != st.state).sum())

def test_layer_calls_equal_stacked_call_prepared():
    """With the queries and keys normalised and the gates evaluated in the kernels (the
    32-column records then carry gamma_q and 1/|k|, 1/|q| factors), the 48 one-layer calls
    of the batched workload (32-column waves, each layer with its own slice of A_log and
    dt_bias) and the 48-layer call (64-column pair blocks) give the same outputs and
    published states bit for bit."""
    wl = configs.build("batched", with_conv=False)
    a, _, gprep = _prep_inputs(wl, QKN | RAWG, seed=87)
    st = _prep_step(wl, a, gprep)
    d = st.dims
    assert d.n_req * d.n_layers * d.h_k >= 256 > d.n_req * d.h_k  # the two forms are taken
    say("[gpu] prepared one-layer calls against the stacked call, batched")
    st.commit(defer=True)
    st.verify_pending(st)
    torch.cuda.synchronize()
    o1 = torch.zeros_like(st.o)
    s1 = st.state0.clone()
    d1 = L.dims(d.n_req, 1, d.h_k, d.h_v, d.d_k, d.d_v, d.op_dtype)
    preps = [L.Prep(QKN | RAWG, 1e-6, gprep.a_log[l:l + 1], gprep.dt_bias[l:l + 1]) for l in range(d.n_layers)]
    for l in range(d.n_layers):
        sl = s1[:, l:l + 1].contiguous()
        t = {key: st.t[key][l] for key in ("q", "k", "v", "g", "beta")}
        L.lumo_tree_gdn_verify_pending(d1, st.desc, t["q"], t["k"], t["v"], t["g"], t["beta"], sl, o1[l],
                                       st.desc, st.max_path, st.path_out, st.path_len, t["k"], t["v"],
                                       t["g"], t["beta"], prep=preps[l])
        s1[:, l:l + 1] = sl
    torch.cuda.synchronize()
    assert not torch.equal(st.state, st.state0)  # paths were published
    assert torch.equal(o1.view(torch.int16), st.o.view(torch.int16)), int((o1 != st.o).sum())
    assert torch.equal(s1, st.state), int((s1 != st.state).sum())


def test_deferred_loop_matches_eager_loop():
    """Three iterations: deferred publication + final flush agrees with eager commits
    (states to fp32 rounding, outputs to bf16 rounding) and with the oracle chain."""
    wls = [configs.build("layer1", seed=s, with_conv=False) for s in (101, 102, 103)]
    eager = [_step(w, L.LUMO_POLICY_WY) for w in wls]
    dfr = [_step(w, L.LUMO_POLICY_WY) for w in wls]
    bank_e = eager[0].state
    bank_d = dfr[0].state
    for i in range(3):
        eager[i].verify(state0=bank_e)
        lumo_commit_into(eager[i], bank_e)
        if i == 0:
            dfr[0].verify(state0=bank_d)
        else:
            dfr[i].verify_pending(dfr[i - 1], state=bank_d)
        dfr[i].commit(defer=True)
    lumo_commit_into(dfr[2], bank_d)  # flush the last pending path
    torch.cuda.synchronize()
    for i in range(3):
        a, b = gu.to_np(eager[i].o), gu.to_np(dfr[i].o)
        rows = oracle.plan.flat_rows(wls[i].parents, wls[i].row_off)
        assert gu.max_rel(b[:, rows], a[:, rows]) <= 2 ** -7, i
    ref = wls[0].arrays["state0"]
    for w in wls:
        ref, _, _ = oracle.commit(w, state_in=ref.astype(np.float32))
    inst = gu.sample_instances(wls[0], 16, seed=4)
    gu.check_states(wls[0], bank_d.cpu().numpy(), ref, inst)
    gu.check_states(wls[0], bank_e.cpu().numpy(), ref, inst)


def lumo_commit_into(st, bank):
    L.lumo_gdn_commit(st.dims, st.desc, st.max_path, st.accepted, st.path_out, st.path_len,
                      st.t["k"], st.t["v"], st.t["g"], st.t["beta"], bank)


# ---------------------------------------------------------------- tree convolution shapes

@pytest.mark.parametrize("case,act", [("depth_first", 1), ("runs_deep", 1), ("runs_few_blocks", 1),
                                      ("depth_first", 0), ("runs_deep", 0)])
def test_conv_tree_shapes(case, act):
    """Both conv kernels on edge shapes: paths of 16 nodes (the depth-first kernel's limit)
    or 20 (run kernel), a request without nodes, a partial channel block, bias; with the
    SiLU and without an activation (act = 0). The depth-first kernel is used when it has
    at least 1024 blocks (requests x layers x channel blocks): 4 x 52 x 5 here."""
    rng = np.random.default_rng(41)
    deep = case == "runs_deep"
    n_layers, C = (52, 8200) if case == "depth_first" else (2, 2056)
    parents = [trees.chain(20 if deep else 16), np.zeros(0, np.int32), trees.FIG1_PARENT,
               trees.random_tree(rng, 40, 8, trees.bmax_uniform(4))]
    n_rows = [len(parents[0]) + 1, 1, 7, 40]
    wl = pins.make_wl(parents, d_k=128, d_v=128, op_dtype=ops.BF16, n_rows=n_rows, n_layers=n_layers,
                      max_path=24, channels=C)
    wl.arrays = ops.make_conv_operands(43, n_req=4, n_layers=n_layers, total_rows=wl.total_rows,
                                       channels=C, op_dtype=ops.BF16)
    bias = rng.standard_normal((n_layers, C)).astype(np.float32)
    say(f"[gpu] conv shapes {case} act={act}")
    desc = L.TreeDesc.build(wl.node_off, wl.parent_flat, wl.n_rows)
    d = L.dims(4, n_layers, 1, 1, 128, 128, L.LUMO_BF16)
    x = torch.from_numpy(wl.arrays["x"]).view(torch.bfloat16).cuda()
    hist = torch.from_numpy(wl.arrays["hist"]).view(torch.bfloat16).cuda()
    w = torch.from_numpy(wl.arrays["w"]).cuda()
    b = torch.from_numpy(bias).cuda()
    y = torch.zeros((n_layers, wl.total_rows, C), dtype=torch.bfloat16, device="cuda")
    L.lumo_tree_conv_gather(d, desc, C, x, hist, w, b, act, y)
    torch.cuda.synchronize()
    got = gu.to_np(y)
    ref = oracle.conv_all(wl, bias=bias, act=act)
    rows = oracle.plan.flat_rows(wl.parents, wl.row_off)
    assert gu.max_rel(got[:, rows], ref[:, rows]) <= gu.TOL_BF16
    pad = [r for r in range(wl.total_rows) if r not in set(rows.tolist())]
    assert np.all(got[:, pad] == 0)


def _conv_wl(parents, n_rows, n_layers, C, op_dtype, seed, max_path=24):
    wl = pins.make_wl(parents, d_k=128, d_v=128, op_dtype=op_dtype, n_rows=n_rows, n_layers=n_layers,
                      max_path=max_path, channels=C)
    wl.arrays = ops.make_conv_operands(seed, n_req=len(parents), n_layers=n_layers, total_rows=wl.total_rows,
                                       channels=C, op_dtype=op_dtype)
    return wl


def _dev(a, bf):
    t = torch.from_numpy(np.ascontiguousarray(a))
    return (t.view(torch.bfloat16) if bf else t).cuda()


@pytest.mark.parametrize("bf,max_path", [(True, 24), (False, 24), (True, 4)])
def test_commit_hist_layers(bf, max_path):
    """lumo_gdn_commit_hist_layers takes each layer's x and history as buffers of their
    own (pointer tables); path_out, path_len and every layer's history must equal the
    stacked commit's bit for bit, and the oracle's publication exactly. Paths of more
    than three nodes, of two, none (-1), an invalid accepted node (99), and with
    max_path = 4 a path too long for it (length -1, nothing published); 3 layers of
    2056 channels (a partial channel block)."""
    rng = np.random.default_rng(53)
    opd = ops.BF16 if bf else ops.F32
    n_layers, C = 3, 2056
    par = [trees.random_tree(rng, 30, 8, trees.bmax_uniform(3)), trees.chain(5), trees.FIG1_PARENT,
           trees.random_tree(rng, 12, 6, trees.bmax_uniform(3))]
    deep = int(np.argmax(trees.depths(par[0])))
    acc_np = np.array([deep, 1, -1, 99], np.int32)
    wl = _conv_wl(par, [31, 5, 7, 14], n_layers, C, opd, 57, max_path=max_path)
    say(f"[gpu] commit into per-layer histories bf16={bf} max_path={max_path}")
    d = L.dims(4, n_layers, 1, 1, 128, 128, L.LUMO_BF16 if bf else L.LUMO_F32)
    desc = L.TreeDesc.build(wl.node_off, wl.parent_flat, wl.n_rows)
    acc = torch.from_numpy(acc_np).cuda()
    x = _dev(wl.arrays["x"], bf)
    hist_ref = _dev(wl.arrays["hist"], bf)
    po = torch.full((4, max_path), -7, dtype=torch.int32, device="cuda")
    pl = torch.full((4,), -7, dtype=torch.int32, device="cuda")
    L.lumo_gdn_commit(d, desc, max_path, acc, po, pl, None, None, None, None, None, C, x, hist_ref)
    xs = [x[l].clone() for l in range(n_layers)]  # separate allocations
    hs = [_dev(wl.arrays["hist"][:, l], bf) for l in range(n_layers)]
    po2 = torch.full((4, max_path), -7, dtype=torch.int32, device="cuda")
    pl2 = torch.full((4,), -7, dtype=torch.int32, device="cuda")
    L.lumo_gdn_commit_hist_layers(d, desc, max_path, acc, po2, pl2, C, xs, hs)
    torch.cuda.synchronize()
    assert torch.equal(po2, po) and torch.equal(pl2, pl)
    want0 = int(trees.depths(par[0])[deep]) + 1
    assert pl2.cpu().numpy().tolist() == [want0 if want0 <= max_path else -1, 2, 0, -1]
    iv = torch.int16 if bf else torch.int32
    for l in range(n_layers):
        assert torch.equal(hs[l].view(iv), hist_ref[:, l].view(iv)), l
    opo = np.full((4, max_path), -1, np.int32)
    opl = np.zeros(4, np.int32)
    for r in range(3):
        path, ln = oracle.plan.accepted_path(par[r], int(acc_np[r]), max_path)
        if ln > 0:
            opo[r], opl[r] = path, ln
    href = oracle.conv_hist_publish(wl, opo, opl)
    assert not np.array_equal(href, wl.arrays["hist"].astype(np.float64))  # something was published
    for l in range(n_layers):
        assert np.array_equal(gu.to_np(hs[l]).astype(np.float64), href[:, l]), l


def test_commit_hist_layers_at_the_layer_limit():
    """128 layers, the most lumo_gdn_commit_hist_layers takes (the pointer tables fill
    2 KB of kernel arguments): every layer's history equals the stacked commit's."""
    rng = np.random.default_rng(59)
    n_layers, C = 128, 16
    par = [trees.random_tree(rng, 12, 6, trees.bmax_uniform(3)), trees.chain(4)]
    wl = _conv_wl(par, [12, 4], n_layers, C, ops.BF16, 61, max_path=8)
    acc = torch.from_numpy(np.array([int(np.argmax(trees.depths(par[0]))), 3], np.int32)).cuda()
    d = L.dims(2, n_layers, 1, 1, 128, 128, L.LUMO_BF16)
    desc = L.TreeDesc.build(wl.node_off, wl.parent_flat, wl.n_rows)
    x = _dev(wl.arrays["x"], True)
    hist_ref = _dev(wl.arrays["hist"], True)
    po = torch.full((2, 8), -7, dtype=torch.int32, device="cuda")
    pl = torch.full((2,), -7, dtype=torch.int32, device="cuda")
    L.lumo_gdn_commit(d, desc, 8, acc, po, pl, None, None, None, None, None, C, x, hist_ref)
    hs = [_dev(wl.arrays["hist"][:, l], True) for l in range(n_layers)]
    po2, pl2 = torch.full_like(po, -7), torch.full_like(pl, -7)
    L.lumo_gdn_commit_hist_layers(d, desc, 8, acc, po2, pl2, C, [x[l] for l in range(n_layers)], hs)
    torch.cuda.synchronize()
    assert torch.equal(po2, po) and torch.equal(pl2, pl) and int(pl.min()) > 0
    for l in range(n_layers):
        assert torch.equal(hs[l].view(torch.int16), hist_ref[:, l].view(torch.int16)), l
    assert not torch.equal(hist_ref.cpu(), _dev(wl.arrays["hist"], True).cpu())


@pytest.mark.parametrize("case", ["depth_first", "runs", "f32"])
def test_conv_pending_history(case):
    """lumo_tree_conv_gather_pending publishes the previous iteration's accepted paths
    into the history, then convolves this iteration's tree from it. The history and y
    must equal the commit's publication followed by the plain conv, bit for bit, and the
    oracle's publication (exactly) and conv (to tolerance). The previous iteration has a
    path of more than three nodes (only x entries), one of two nodes (history and x),
    none (accepted -1), and an invalid one (accepted out of range: nothing published);
    this iteration has a request without nodes, which is still published. depth_first:
    4 requests x 64 layers x 4 channel blocks (the depth-first kernel publishes in
    place); runs: 3 layers, 2056 channels (a separate publication, then the run kernel);
    f32: the same with fp32 operands."""
    rng = np.random.default_rng(47)
    bf = case != "f32"
    opd = ops.BF16 if bf else ops.F32
    n_layers, C = (64, 8192) if case == "depth_first" else (3, 2056)
    prev_par = [trees.random_tree(rng, 30, 8, trees.bmax_uniform(3)), trees.chain(5), trees.FIG1_PARENT,
                trees.random_tree(rng, 12, 6, trees.bmax_uniform(3))]
    deep = int(np.argmax(trees.depths(prev_par[0])))
    prev_acc = np.array([deep, 1, -1, 99], np.int32)
    cur_par = [trees.random_tree(rng, 20, 8, trees.bmax_uniform(3)), np.zeros(0, np.int32), trees.chain(16),
               trees.FIG1_PARENT]
    prev = _conv_wl(prev_par, [31, 5, 7, 14], n_layers, C, opd, 51)
    cur = _conv_wl(cur_par, [20, 2, 16, 9], n_layers, C, opd, 52)
    cur.arrays["hist"] = prev.arrays["hist"]
    bias = rng.standard_normal((n_layers, C)).astype(np.float32) if case == "depth_first" else None
    say(f"[gpu] conv pending {case}")
    dt = L.LUMO_BF16 if bf else L.LUMO_F32
    d = L.dims(4, n_layers, 1, 1, 128, 128, dt)
    pdesc = L.TreeDesc.build(prev.node_off, prev.parent_flat, prev.n_rows)
    cdesc = L.TreeDesc.build(cur.node_off, cur.parent_flat, cur.n_rows)
    max_path = prev.max_path
    acc = torch.from_numpy(prev_acc).cuda()
    po = torch.full((4, max_path), -7, dtype=torch.int32, device="cuda")
    pl = torch.full((4,), -7, dtype=torch.int32, device="cuda")
    xp, xc = _dev(prev.arrays["x"], bf), _dev(cur.arrays["x"], bf)
    w = torch.from_numpy(cur.arrays["w"]).cuda()
    b = torch.from_numpy(bias).cuda() if bias is not None else None
    odt = torch.bfloat16 if bf else torch.float32
    # reference order: the commit publishes the history, then the plain conv
    hist_ref = _dev(prev.arrays["hist"], bf)
    y_ref = torch.zeros((n_layers, cur.total_rows, C), dtype=odt, device="cuda")
    L.lumo_gdn_commit(d, pdesc, max_path, acc, po, pl, None, None, None, None, None, C, xp, hist_ref)
    L.lumo_tree_conv_gather(d, cdesc, C, xc, hist_ref, w, b, 1, y_ref)
    # deferred: the commit derives the path only; the next conv publishes
    po2 = torch.full((4, max_path), -7, dtype=torch.int32, device="cuda")
    pl2 = torch.full((4,), -7, dtype=torch.int32, device="cuda")
    hist = _dev(prev.arrays["hist"], bf)
    y = torch.zeros((n_layers, cur.total_rows, C), dtype=odt, device="cuda")
    L.lumo_gdn_commit(d, pdesc, max_path, acc, po2, pl2, None, None, None, None, None, 0, None, None)
    L.lumo_tree_conv_gather_pending(d, cdesc, C, xc, hist, w, b, 1, y, pdesc, max_path, po2, pl2, xp)
    torch.cuda.synchronize()
    assert pl2.cpu().numpy().tolist() == [int(trees.depths(prev_par[0])[deep]) + 1, 2, 0, -1]
    assert torch.equal(hist.view(torch.int16 if bf else torch.int32), hist_ref.view(torch.int16 if bf else torch.int32))
    assert torch.equal(y.view(torch.int16 if bf else torch.int32), y_ref.view(torch.int16 if bf else torch.int32))
    # the oracle: paths from the parents (the invalid request publishes nothing: length 0)
    opo = np.full((4, max_path), -1, np.int32)
    opl = np.zeros(4, np.int32)
    for r in range(3):
        path, ln = oracle.plan.accepted_path(prev_par[r], int(prev_acc[r]), max_path)
        opo[r], opl[r] = path, ln
    href = oracle.conv_hist_publish(prev, opo, opl)
    assert np.array_equal(gu.to_np(hist).astype(np.float64), href)
    cur.arrays["hist"] = href.astype(np.float32) if not bf else ops.to_bf16_bits(href.astype(np.float32))
    yref = oracle.conv_all(cur, bias=bias)
    rows = oracle.plan.flat_rows(cur.parents, cur.row_off)
    assert gu.max_rel(gu.to_np(y)[:, rows], yref[:, rows]) <= (gu.TOL_BF16 if bf else gu.TOL_F32)
    pad = [r for r in range(cur.total_rows) if r not in set(rows.tolist())]
    assert np.all(gu.to_np(y)[:, pad] == 0)
    if case == "runs":
        # a batch without nodes in this iteration still publishes
        empty = L.TreeDesc.build(np.zeros(5, np.int32), np.zeros(0, np.int32), np.ones(4, np.int32))
        hist_e = _dev(prev.arrays["hist"], bf)
        L.lumo_tree_conv_gather_pending(d, empty, C, None, hist_e, None, None, 1, None, pdesc, max_path, po2,
                                        pl2, xp)
        torch.cuda.synchronize()
        assert torch.equal(hist_e.view(torch.int16), hist_ref.view(torch.int16))


# ---------------------------------------------------------------- operand preparation

QKN, RAWG = L.LUMO_PREP_QK_NORM, L.LUMO_PREP_RAW_GATES


def _prep_inputs(wl, flags, seed, eps=1e-6):
    """Raw operands for a prepared run: q and k rows rescaled by U(0.3, 3) (so the
    normalisation matters), raw gate inputs a, b ~ N(0, 1), and per-(layer, head)
    A_log ~ N(0, 0.5^2), dt_bias ~ N(0, 1). Returns (arrays, oracle Prep, device Prep)."""
    rng = np.random.default_rng(seed)
    a = dict(wl.arrays)
    if flags & QKN:
        for key in ("q", "k"):
            f = ops.bf16_bits_to_f32(a[key]) * rng.uniform(0.3, 3.0, size=a[key].shape[:-1] + (1,))
            a[key] = ops.to_bf16_bits(f.astype(np.float32))
    if flags & RAWG:
        a["g"] = rng.standard_normal(a["g"].shape).astype(np.float32)
        a["beta"] = rng.standard_normal(a["beta"].shape).astype(np.float32)
    a_log = (0.5 * rng.standard_normal((wl.n_layers, wl.h_v))).astype(np.float32)
    dt_bias = rng.standard_normal((wl.n_layers, wl.h_v)).astype(np.float32)
    oprep = oracle.Prep(flags, eps, a_log, dt_bias)
    gprep = L.Prep(flags, eps, torch.from_numpy(a_log).cuda(), torch.from_numpy(dt_bias).cuda())
    return a, oprep, gprep


def _prep_step(wl, arrays, gprep, policy=L.LUMO_POLICY_WY):
    return GdnTreeStep(n_req=wl.n_req, n_layers=wl.n_layers, h_k=wl.h_k, h_v=wl.h_v, d_k=wl.d_k,
                       d_v=wl.d_v, op_dtype=wl.op_dtype, node_off=wl.node_off,
                       parent=wl.parent_flat, n_rows=wl.n_rows,
                       arrays={k: v for k, v in arrays.items() if k not in ("x", "hist", "w")},
                       policy=policy, max_path=wl.max_path, accepted=wl.accepted, prep=gprep)


def _check_prep_outputs(wl, o, arrays, oprep, inst, tol=gu.TOL_BF16):
    worst = 0.0
    for (r, l, h) in inst:
        n = len(wl.parents[r])
        if n == 0:
            continue
        ref = oracle.verify_nodes(wl, r, l, h, list(range(n)), arrays=arrays, prep=oprep)
        got = o[l, gu.node_rows(wl, r), h, :]
        assert np.all(np.isfinite(got)), (r, l, h)
        e = gu.max_rel(got, ref)
        worst = max(worst, e)
        assert e <= tol, f"instance {(r, l, h)}: max rel err {e:.3e}"
    return worst


@pytest.mark.parametrize("flags", [QKN, RAWG, QKN | RAWG])
def test_wy_prep_parity(flags):
    """Operands prepared inside the WY kernel and the commit replay: outputs and the
    published state against the oracle with the same preparation."""
    wl = workload("layer1")
    a, oprep, gprep = _prep_inputs(wl, flags, seed=71 + flags)
    say(f"[gpu] wy prep flags={flags}")
    st = _prep_step(wl, a, gprep)
    st.verify()
    st.commit()
    torch.cuda.synchronize()
    inst = [(0, 0, h) for h in range(wl.h_v)]
    worst = _check_prep_outputs(wl, gu.to_np(st.o), a, oprep, inst)
    say(f"  outputs worst max-rel {worst:.3e}")
    ref_state, _, pl = oracle.commit(wl, arrays=a, prep=oprep)
    assert np.array_equal(st.path_len.cpu().numpy(), pl)
    ws = gu.check_states(wl, st.state.cpu().numpy(), ref_state, inst)
    say(f"  published state worst max-rel {ws:.3e}")
    # without the preparation the same raw operands give other outputs (the test has teeth)
    plain = _prep_step(wl, a, None)
    plain.verify()
    torch.cuda.synchronize()
    assert gu.max_rel(gu.to_np(plain.o)[0, gu.node_rows(wl, 0), 0], gu.to_np(st.o)[0, gu.node_rows(wl, 0), 0]) > 0.05


def test_wy_prep_deep_and_groupings():
    """Prepared operands with 17-node paths (16 path-stack registers) and one value head
    per block (h_k = h_v)."""
    rng = np.random.default_rng(73)
    parents = [trees.chain(17), trees.random_tree(rng, 40, 9, trees.bmax_uniform(3)), trees.FIG1_PARENT]
    wl = pins.make_wl(parents, d_k=128, d_v=128, h_k=4, h_v=4, op_dtype=ops.BF16,
                      n_rows=[17, 41, 7], n_layers=2, max_path=17)
    wl.arrays = ops.make_gdn_operands(74, n_req=3, n_layers=2, total_rows=65, h_k=4, h_v=4,
                                      d_k=128, d_v=128, op_dtype=ops.BF16)
    a, oprep, gprep = _prep_inputs(wl, QKN | RAWG, seed=75)
    st = _prep_step(wl, a, gprep)
    st.verify()
    torch.cuda.synchronize()
    inst = [(r, l, h) for r in range(3) for l in range(2) for h in (0, 3)]
    _check_prep_outputs(wl, gu.to_np(st.o), a, oprep, inst)


@pytest.mark.parametrize("case", ["layer1", "tiny_f32", "deep_f32"])
def test_scan_prep_parity(case):
    """Prepared operands on the sequential scan (RECOMPUTE, the schedule that needs no
    workspace): outputs against the oracle with the same preparation, for the shapes the
    WY kernel does not take (fp32 operands, d < 128, paths longer than 17 nodes)."""
    if case == "layer1":
        wl = workload("layer1")
        inst = [(0, 0, h) for h in range(0, wl.h_v, 5)]
    elif case == "tiny_f32":
        wl = workload("tiny")
        inst = [(0, 0, 0)]
    else:
        rng = np.random.default_rng(81)
        parents = [trees.chain(23), trees.random_tree(rng, 30, 20, trees.bmax_uniform(2))]
        wl = pins.make_wl(parents, d_k=64, d_v=32, h_k=2, h_v=4, op_dtype=ops.F32, n_rows=[23, 33],
                          n_layers=2, max_path=23)
        wl.arrays = ops.make_gdn_operands(82, n_req=2, n_layers=2, total_rows=56, h_k=2, h_v=4,
                                          d_k=64, d_v=32, op_dtype=ops.F32)
        wl.accepted = np.array([22, int(np.argmax(trees.depths(parents[1])))], np.int32)
        inst = [(r, l, h) for r in range(2) for l in range(2) for h in range(4)]
    flags = QKN | RAWG
    if wl.op_dtype == ops.F32:
        # fp32 operand rows rescaled for the normalisation to matter
        rng = np.random.default_rng(83)
        a = dict(wl.arrays)
        for key in ("q", "k"):
            a[key] = (a[key] * rng.uniform(0.3, 3.0, size=a[key].shape[:-1] + (1,))).astype(np.float32)
        a["g"] = rng.standard_normal(a["g"].shape).astype(np.float32)
        a["beta"] = rng.standard_normal(a["beta"].shape).astype(np.float32)
        a_log = (0.5 * rng.standard_normal((wl.n_layers, wl.h_v))).astype(np.float32)
        dt_bias = rng.standard_normal((wl.n_layers, wl.h_v)).astype(np.float32)
        oprep = oracle.Prep(flags, 1e-6, a_log, dt_bias)
        gprep = L.Prep(flags, 1e-6, torch.from_numpy(a_log).cuda(), torch.from_numpy(dt_bias).cuda())
    else:
        a, oprep, gprep = _prep_inputs(wl, flags, seed=84)
    say(f"[gpu] scan prep {case}")
    st = _prep_step(wl, a, gprep, policy=L.LUMO_POLICY_RECOMPUTE)
    st.verify()
    st.commit()
    torch.cuda.synchronize()
    worst = _check_prep_outputs(wl, gu.to_np(st.o), a, oprep, inst, tol=gu.out_tol(wl))
    say(f"  outputs worst max-rel {worst:.3e}")
    ref_state, _, pl = oracle.commit(wl, arrays=a, prep=oprep)
    assert np.array_equal(st.path_len.cpu().numpy(), pl)
    gu.check_states(wl, st.state.cpu().numpy(), ref_state, inst)
    plain = _prep_step(wl, a, None, policy=L.LUMO_POLICY_RECOMPUTE)
    plain.verify()
    torch.cuda.synchronize()
    r0, l0, h0 = inst[0]
    rows = gu.node_rows(wl, r0)
    assert gu.max_rel(gu.to_np(plain.o)[l0, rows, h0], gu.to_np(st.o)[l0, rows, h0]) > 0.05


def test_commit_prep_on_scan_plan():
    """The commit's preparation does not depend on the plan's policy."""
    wl = workload("paper28")
    a, oprep, gprep = _prep_inputs(wl, QKN | RAWG, seed=76)
    st = _prep_step(wl, a, gprep, policy=L.LUMO_POLICY_PATHS)
    st.commit()
    torch.cuda.synchronize()
    ref_state, _, _ = oracle.commit(wl, arrays=a, prep=oprep)
    gu.check_states(wl, st.state.cpu().numpy(), ref_state,
                    [(0, 0, h) for h in range(wl.h_v)])


def test_verify_pending_prep():
    """Deferred publication with prepared operands in both iterations."""
    prev, cur = _pending_pair(2, 4, seed=77)
    pa, poprep, gprep = _prep_inputs(prev, QKN | RAWG, seed=78)
    # the current iteration uses the same gate parameters (same layers and heads)
    ca, _, _ = _prep_inputs(cur, QKN | RAWG, seed=79)
    sp = _prep_step(prev, pa, gprep, policy=L.LUMO_POLICY_PATHS)
    sp.commit(defer=True)
    sc = _prep_step(cur, ca, gprep)
    sc.verify_pending(sp, state=sp.state)
    torch.cuda.synchronize()
    acc = prev.accepted.copy()
    acc[3] = -1
    ref_state, _, _ = oracle.commit(prev, accepted=acc, arrays=pa, prep=poprep)
    inst = [(r, l, h) for r in range(5) for l in range(2) for h in range(4)]
    gu.check_states(prev, sp.state.cpu().numpy(), ref_state, inst)
    c2 = dict(ca)
    c2["state0"] = ref_state.astype(np.float32)
    _check_prep_outputs(cur, gu.to_np(sc.o), c2, poprep, inst)
