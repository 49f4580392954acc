"""The WY verification of fp32 operands on the matrix cores (d = 128), and the isolation of
non-finite values in it and in the bf16 form for paths of 18 to 32 nodes.

Every node against the fp64 oracle at the edges of the path registers (9 / 10, 17 / 18 and 32
nodes per path), of the 32-node chunks and their halves, with path stacks that reach back
over several chunks, plain and with operands prepared in the kernel. Besides the parity
tolerance of fp32 operands, the root mean square error over all outputs must stay within 2^-21
of their root mean square: fp32 rounds by 2^-24, and a value is the end of at most 32
updates and of sums whose rounding errors add up like random steps (sqrt(32) < 8).
"""
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
    rng = np.random.default_rng(51)
    if case == "nine":
        return [trees.chain(9), np.zeros(0, np.int32), trees.random_tree(rng, 33, 9, trees.bmax_uniform(3)), trees.chain(1)]
    if case == "seventeen":
        return [trees.chain(10), trees.random_tree(rng, 64, 17, trees.bmax_uniform(2)), trees.chain(17), trees.chain(16)]
    # a 31-deep spine with leaves at every level, visited last: deep stacks in every chunk
    return [np.array(list(range(-1, 30)) + [i % 31 for i in range(50)], np.int32), trees.chain(32), trees.chain(18)]


def _workload(parents, h_k, h_v, op_dtype):
    n_rows = [len(p) + i % 2 for i, p in enumerate(parents)]
    wl = pins.make_wl(parents, d_k=128, d_v=128, h_k=h_k, h_v=h_v, op_dtype=op_dtype, n_rows=n_rows, n_layers=2,
                      max_path=32)
    wl.arrays = ops.make_gdn_operands(53, n_req=wl.n_req, n_layers=2, total_rows=wl.total_rows, h_k=h_k, h_v=h_v,
                                      d_k=128, d_v=128, op_dtype=op_dtype)
    return wl


def _verify(wl, a, prep=None):
    st = GdnTreeStep(n_req=wl.n_req, n_layers=2, h_k=wl.h_k, h_v=wl.h_v, d_k=128, d_v=128, op_dtype=wl.op_dtype,
                     node_off=wl.node_off, parent=wl.parent_flat, n_rows=wl.n_rows, arrays=a, policy=L.LUMO_POLICY_WY,
                     max_path=32, accepted=wl.accepted, prep=prep)
    st.verify()
    torch.cuda.synchronize()
    return gu.to_np(st.o)


@pytest.mark.parametrize("case,h_k,h_v,flags", [("nine", 1, 1, 0), ("nine", 2, 4, QKN | RAWG), ("seventeen", 1, 3, 0),
                                                ("seventeen", 2, 2, QKN), ("deep", 2, 2, 0), ("deep", 1, 2, QKN | RAWG)])
def test_fp32_wy_against_oracle(case, h_k, h_v, flags):
    wl = _workload(_trees(case), h_k, h_v, ops.F32)
    a = dict(wl.arrays)
    rng = np.random.default_rng(54)
    oprep = gprep = None
    if flags:
        if flags & RAWG:
            for key in ("g", "beta"):
                a[key] = rng.standard_normal(a[key].shape).astype(np.float32)
        a_log = (0.5 * rng.standard_normal((2, h_v))).astype(np.float32)
        dt_bias = rng.standard_normal((2, h_v)).astype(np.float32)
        oprep = oracle.Prep(flags, 1e-6, a_log, dt_bias)
        gprep = L.Prep(flags, 1e-6, torch.from_numpy(a_log).cuda(), torch.from_numpy(dt_bias).cuda())
    print(f"[gpu] fp32 wy {case} heads={h_k}/{h_v} prep={flags}", flush=True)
    o = _verify(wl, a, gprep)
    off = size = 0.0
    for r, par in enumerate(wl.parents):
        for l in range(2):
            for h in range(h_v):
                if len(par) == 0:
                    continue
                ref = oracle.verify_nodes(wl, r, l, h, list(range(len(par))), arrays=a, prep=oprep)
                got = o[l, gu.node_rows(wl, r), h]
                assert gu.max_rel(got, ref) <= gu.TOL_F32, (r, l, h)
                off += float(np.sum((got - ref) ** 2))
                size += float(np.sum(np.asarray(ref, np.float64) ** 2))
    assert np.sqrt(off / size) <= 2.0 ** -21, np.sqrt(off / size)
    pad = [x for x in range(wl.total_rows) if x not in set(oracle.plan.flat_rows(wl.parents, wl.row_off).tolist())]
    assert np.all(o[:, pad] == 0)


@pytest.mark.parametrize("case,op_dtype", [("nine", ops.F32), ("seventeen", ops.F32), ("deep", ops.F32),
                                           ("deep", ops.BF16)])
def test_non_finite_values_stay_in_their_subtree(case, op_dtype):
    """NaN and infinity in single value entries spoil the outputs of that node and its
    descendants in that column; every other output keeps its bits."""
    wl = _workload(_trees(case), 1, 2, op_dtype)
    clean = _verify(wl, wl.arrays)
    a = dict(wl.arrays)
    a["v"] = a["v"].copy()
    bad = {}  # (row, column): the rows of the subtree
    for r, par in enumerate(wl.parents):
        if len(par) < 4:
            continue
        rows = gu.node_rows(wl, r)
        for node, col, f32 in ((2, 5 + r, np.nan), (len(par) // 2, 77 + r, np.inf)):
            a["v"][0, rows[node], 1, col] = f32 if op_dtype == ops.F32 else (0x7FC0 if np.isnan(f32) else 0x7F80)
            sub = [rows[i] for i in range(len(par)) if node in oracle.plan.ancestry(par, i)]
            bad.setdefault(col, []).extend(sub)
    print(f"[gpu] non-finite values {case} dtype={op_dtype}", flush=True)
    o = _verify(wl, a)
    keep = np.ones(o.shape, bool)
    for col, rows in bad.items():
        keep[0, rows, 1, col] = False
        assert not np.any(np.isfinite(o[0, rows, 1, col]))
    assert np.array_equal(o[keep].view(np.uint32), clean[keep].view(np.uint32))


@pytest.mark.parametrize("length", [9, 17, 32])  # the three widths of path registers
def test_fp32_wy_products_keep_24_bits(length):
    """A single term decides each output: one-hot keys and queries against the state (beta 0),
    and against each other (state 0, value 1, each node its own index). The output is one
    product of two fp32 numbers: at most 2^-24 of it is dropped by the three-part split, and
    it is rounded by 2^-24 (the small partial products round 2^-7 times finer). The values
    include the one that loses most when the first part is cut off (0x3f80ff80)."""
    parents = [trees.chain(length), np.array([-1] + [0] * 40, np.int32)]
    wl = _workload(parents, 2, 2, ops.F32)
    rng = np.random.default_rng(55)
    a = {k: np.zeros_like(x) for k, x in wl.arrays.items()}

    def factor(shape):
        x = (1 + rng.random(shape)).astype(np.float32)
        x.flat[::3] = np.uint32(0x3F80FF80).view(np.float32)
        return x

    index = np.concatenate([np.arange(len(p)) for p in parents])
    rows = np.concatenate([gu.node_rows(wl, r) for r in range(2)])
    key, query = factor((2, len(rows), 2)), factor((2, len(rows), 2))
    print(f"[gpu] fp32 wy single products, paths of {length}", flush=True)
    for part in ("state", "gram"):
        b = {k: x.copy() for k, x in a.items()}
        for l in range(2):
            for h in range(2):
                b["q"][l, rows, h, index] = query[l, :, h]
                b["k"][l, rows, h, index] = key[l, :, h]
        if part == "state":
            b["state0"][:] = factor(b["state0"].shape)
            want = np.zeros((2, wl.total_rows, 2, 128))
            for r in range(2):
                at = slice(0, length) if r == 0 else slice(length, None)
                for l in range(2):
                    for h in range(2):
                        want[l, rows[at], h] = (query[l, at, h].astype(np.float64)[:, None]
                                                * b["state0"][r, l, h][index[at]].astype(np.float64))
        else:
            b["beta"][:], b["v"][:] = 1.0, 1.0
            want = np.zeros((2, wl.total_rows, 2, 128))
            want[:, rows] = (query.astype(np.float64) * key)[..., None]
        o = _verify(wl, b)[:, rows]
        want = want[:, rows]
        assert np.max(np.abs(o - want) / np.abs(want)) <= 2.0 ** -23 + 2.0 ** -27, part


def _wy_form(q, k, v, g, beta, state, par):
    """The WY form of one head in 64 bits, nodes in storage order (parents first)."""
    path, out, delta = [], [], []
    for t, p in enumerate(par):
        anc = oracle.plan.ancestry(par, t)
        gam = np.exp(sum(g[m] for m in anc))
        d = beta[t] * (v[t] - gam * (k[t] @ state))
        o = gam * (q[t] @ state)
        for j, m in enumerate(anc[:-1]):
            decay = np.exp(sum(g[x] for x in anc[j + 1:]))
            d = d - (beta[t] * decay * (k[m] @ k[t])) * delta[m]
            o = o + (decay * (k[m] @ q[t])) * delta[m]
        delta.append(d)
        out.append(o + (k[t] @ q[t]) * d)
    return np.array(out)


def _kind(x):
    return np.where(np.isnan(x), 2, np.where(np.isinf(x), np.sign(x), 0))


@pytest.mark.parametrize("case,op_dtype,where", [(c, ops.F32, w) for c in ("nine", "seventeen", "deep")
                                                 for w in ("state0", "k", "q", "state0 k")]
                         + [("deep", ops.BF16, w) for w in ("state0", "k", "q")])
def test_infinities_pass_as_in_a_dot_product(case, op_dtype, where):
    """An infinite entry of the state, a key or a query (and two of them that meet) gives the
    outputs that whole fp32 factors give: the same infinities with the same sign, NaN only
    where two of them meet, and finite values everywhere else. Values of every fourth node are
    exact in bf16, so that an infinity meets zero parts. Finite outputs are held to the
    parity tolerance per instance."""
    wl = _workload(_trees(case), 1, 2, op_dtype)
    a = {k: x.copy() for k, x in wl.arrays.items()}
    f32 = op_dtype == ops.F32
    for name in ("q", "k"):
        if f32:
            a[name][:, ::4] = ops.bf16_bits_to_f32(ops.to_bf16_bits(a[name][:, ::4]))
    for r, par in enumerate(wl.parents):
        rows = gu.node_rows(wl, r)
        if len(par) < 4:
            continue
        if "state0" in where:
            a["state0"][r, 0, 1, 3 + r, 40] = np.inf
            a["state0"][r, 0, 1, 90, 41 + r] = -np.inf
        for name in ("k", "q"):
            if name in where:
                for node, entry, neg in ((0, 60, False), (len(par) // 2, 17, False), (len(par) - 1, 3 + r, True)):
                    x = -np.inf if neg else np.inf
                    a[name][0, rows[node], 0, entry] = x if f32 else (0xFF80 if neg else 0x7F80)
    print(f"[gpu] infinities {case} dtype={op_dtype} in {where}", flush=True)
    o = _verify(wl, a)
    val = {n: (x if x.dtype == np.float32 else ops.bf16_bits_to_f32(x)).astype(np.float64) for n, x in a.items()}
    seen = set()
    with np.errstate(all="ignore"):
        for r, par in enumerate(wl.parents):
            rows = gu.node_rows(wl, r)
            for l in range(2):
                for h in range(2):
                    if len(par) == 0:
                        continue
                    ref = _wy_form(val["q"][l, rows, 0], val["k"][l, rows, 0], val["v"][l, rows, h], val["g"][l, rows, h],
                                   val["beta"][l, rows, h], val["state0"][r, l, h], par)
                    got = o[l, rows, h]
                    assert np.array_equal(_kind(got), _kind(ref)), (r, l, h)
                    seen |= set(np.unique(_kind(ref)).tolist())
                    ok = np.isfinite(ref)
                    tol = gu.TOL_F32 if f32 else gu.TOL_BF16
                    assert np.max(np.abs(got - ref)[ok], initial=0.0) <= tol * np.max(np.abs(ref[ok]), initial=1e-30), (r, l, h)
    assert len(seen) >= 3, seen
