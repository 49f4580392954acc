"""The vector-ALU WY kernel on the shapes it serves: heads below 128 in either dimension, with
paths up to its limit of 32 nodes and operands prepared in the kernel; fp32 trees of up to three
nodes at d = 128; and d = 128 beyond 17 nodes per path with a plan that lacks the tables of the
matrix-core forms. Also plans without the optional words of the sequential policies, which run
level by level.

Every node against the fp64 oracle under the parity tolerances."""
from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU, skipped there
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
import paper_2609_23900_amd as L  # noqa: E402
from paper_2609_23900_amd.step import GdnTreeStep  # noqa: E402
from lumo_synth import operands as ops  # noqa: E402
from lumo_synth import trees  # noqa: E402
import gpu_util as gu  # noqa: E402
import pins  # noqa: E402

QKN, RAWG = L.LUMO_PREP_QK_NORM, L.LUMO_PREP_RAW_GATES


def _trees(case):
    rng = np.random.default_rng(81)
    if case == "tiny":  # too small for a chunk of the matrix-core form
        return [trees.chain(1), np.zeros(0, np.int32), trees.chain(2), trees.chain(3), np.array([-1, 0, 0], np.int32)]
    if case == "deep":
        return [trees.chain(18), trees.chain(31), trees.chain(32), trees.random_tree(rng, 60, 25, trees.bmax_uniform(2)),
                np.zeros(0, np.int32)]
    return [trees.random_tree(rng, 45, 8, trees.bmax_uniform(4)), trees.FIG1_PARENT, trees.chain(1)]


def _setup(case, d_k, d_v, op_dtype, flags, h_k=2, h_v=4):
    parents = _trees(case)
    n_rows = [len(p) + i % 2 for i, p in enumerate(parents)]
    wl = pins.make_wl(parents, d_k=d_k, d_v=d_v, h_k=h_k, h_v=h_v, op_dtype=op_dtype, n_rows=n_rows, n_layers=2, max_path=32)
    a = ops.make_gdn_operands(82, n_req=wl.n_req, n_layers=2, total_rows=wl.total_rows, h_k=h_k, h_v=h_v, d_k=d_k, d_v=d_v,
                              op_dtype=op_dtype)
    rng = np.random.default_rng(83)
    oprep = gprep = None
    if flags:
        if flags & RAWG:
            for key in ("g", "beta"):
                a[key] = rng.standard_normal(a[key].shape).astype(np.float32)
        a_log = (0.5 * rng.standard_normal((2, h_v))).astype(np.float32)
        dt_bias = rng.standard_normal((2, h_v)).astype(np.float32)
        oprep = oracle.Prep(flags, 1e-6, a_log, dt_bias)
        gprep = L.Prep(flags, 1e-6, torch.from_numpy(a_log).cuda(), torch.from_numpy(dt_bias).cuda())
    wl.arrays = a
    st = GdnTreeStep(n_req=wl.n_req, n_layers=2, h_k=h_k, h_v=h_v, d_k=d_k, d_v=d_v, op_dtype=op_dtype, node_off=wl.node_off,
                     parent=wl.parent_flat, n_rows=wl.n_rows, arrays=a, policy=L.LUMO_POLICY_WY, max_path=32,
                     accepted=wl.accepted, prep=gprep)
    return wl, st, oprep


def _check(wl, st, oprep):
    st.verify()
    torch.cuda.synchronize()
    o = gu.to_np(st.o)
    tol = gu.out_tol(wl)
    for r, par in enumerate(wl.parents):
        for l in range(2):
            for h in range(wl.h_v):
                if len(par):
                    ref = oracle.verify_nodes(wl, r, l, h, list(range(len(par))), arrays=wl.arrays, prep=oprep)
                    assert gu.max_rel(o[l, gu.node_rows(wl, r), h], ref) <= tol, (r, l, h)
    return o


@pytest.mark.parametrize("case,d_k,d_v,op_dtype,flags", [
    ("deep", 64, 64, ops.F32, 0), ("deep", 64, 128, ops.BF16, 0), ("deep", 128, 64, ops.F32, QKN | RAWG),
    ("deep", 32, 16, ops.BF16, QKN), ("shallow", 64, 128, ops.F32, QKN | RAWG), ("shallow", 64, 128, ops.BF16, QKN | RAWG),
    ("shallow", 128, 64, ops.BF16, RAWG), ("shallow", 16, 64, ops.F32, QKN)])
def test_vector_alu_wy(case, d_k, d_v, op_dtype, flags):
    print(f"[gpu] wyv {case} d={d_k}x{d_v} dtype={op_dtype} prep={flags}", flush=True)
    wl, st, oprep = _setup(case, d_k, d_v, op_dtype, flags)
    _check(wl, st, oprep)


@pytest.mark.parametrize("flags,h_k,h_v", [(0, 2, 4), (QKN | RAWG, 2, 4), (QKN, 16, 48)])
def test_vector_alu_wy_of_tiny_trees(flags, h_k, h_v):
    print(f"[gpu] wyv tiny trees d=128 fp32 heads={h_k}/{h_v} prep={flags}", flush=True)
    wl, st, oprep = _setup("tiny", 128, 128, ops.F32, flags, h_k, h_v)
    o = _check(wl, st, oprep)
    rows = set(oracle.plan.flat_rows(wl.parents, wl.row_off).tolist())
    assert np.all(o[:, [x for x in range(wl.total_rows) if x not in rows]] == 0)


@pytest.mark.parametrize("op_dtype,flags", [(ops.F32, 0), (ops.BF16, 0), (ops.F32, QKN | RAWG), (ops.BF16, QKN)])
def test_wy_plans_without_the_deep_tables(op_dtype, flags):
    print(f"[gpu] wyv d=128 without deep tables dtype={op_dtype} prep={flags}", flush=True)
    wl, st, oprep = _setup("deep", 128, 128, op_dtype, flags)
    with_tables = _check(wl, st, oprep)
    plan = st.desc.desc.plan
    plan.n_words = plan.o_vis + 2 * plan.total_nodes  # a blob that ends with the last named section
    st.o.zero_()
    without = _check(wl, st, oprep)
    assert not np.array_equal(with_tables, without)  # another kernel, another order of sums


@pytest.mark.parametrize("policy", [L.LUMO_POLICY_PATHS, L.LUMO_POLICY_TWO_LEVEL, L.LUMO_POLICY_RECOMPUTE])
def test_sequential_plans_without_the_traversal(policy):
    """The same bits level by level, in a call large enough for the single launch."""
    print(f"[gpu] scan without traversal words policy={policy}", flush=True)
    rng = np.random.default_rng(84)
    parents = [trees.random_tree(rng, 40, 8, trees.bmax_uniform(3)), trees.chain(9)]
    node_off = np.array([0, 40, 49], np.int32)
    layers, h, d = 70, 2, 64
    a = ops.make_gdn_operands(85, n_req=2, n_layers=layers, total_rows=49, h_k=h, h_v=h, d_k=d, d_v=d, op_dtype=ops.BF16)
    assert 2 * layers * h * (d // 16) > 1024
    out = []
    for strip in (False, True):
        st = GdnTreeStep(n_req=2, n_layers=layers, h_k=h, h_v=h, d_k=d, d_v=d, op_dtype=ops.BF16, node_off=node_off,
                         parent=np.concatenate(parents), n_rows=np.array([40, 9], np.int32), arrays=a, policy=policy)
        plan = st.desc.desc.plan
        if strip:
            plan.n_words = plan.o_vis + 2 * plan.total_nodes
        st.verify()
        torch.cuda.synchronize()
        out.append(st.o.view(torch.int16).cpu())
    assert torch.equal(*out) and bool(out[0].any())
