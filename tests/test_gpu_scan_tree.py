"""The sequential policies' single-launch scan against the level-by-level scan, bit for bit.

A call that asks for the node states runs level by level; the same call without them
takes the single launch (the layers are chosen so that it does: more than 1,024 column
tiles, below which calls with wide trees stay level by level; only RECOMPUTE of the complete tree
at d_k = 32 is level by level both times). Both must leave the same output bits at every node row and touch
no pad row, for every key and value dimension, both operand types, grouped heads, trees that
end on and around the 16-node chunks, zero to four saved states, and trees that need more
(which stay level by level).
"""
from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU, skipped there
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2609_23900_amd as L  # noqa: E402
from lumo_synth import operands as ops  # noqa: E402
from lumo_synth import trees  # noqa: E402


def _complete(levels):
    """A complete binary tree: `levels` - 1 saved states."""
    return np.array([-1] + [(i - 1) // 2 for i in range(1, 2 ** levels - 1)], np.int32)


def _slots(plan, blob):
    at = plan.o_vis + 2 * plan.total_nodes
    return int(blob[at + at % 2])


TREES = {
    "chunks": lambda rng: [trees.chain(n) for n in (1, 15, 16, 17, 32, 33)],
    "random": lambda rng: [trees.random_tree(rng, 64, 8, trees.bmax_uniform(4)), np.zeros(0, np.int32),
                           trees.random_tree(rng, 47, 24, trees.bmax_uniform(3))],
    "four": lambda rng: [_complete(5), trees.chain(3)],
    "five": lambda rng: [_complete(6), trees.FIG1_PARENT],
}


@pytest.mark.parametrize("tree,dtype,h_k,h_v,d_k,d_v", [
    ("chunks", ops.BF16, 2, 4, 128, 128), ("chunks", ops.F32, 1, 1, 16, 16), ("random", ops.BF16, 2, 2, 128, 64),
    ("random", ops.F32, 2, 6, 128, 128), ("random", ops.BF16, 1, 2, 32, 16), ("random", ops.F32, 1, 3, 64, 32),
    ("four", ops.BF16, 1, 2, 128, 128), ("four", ops.F32, 2, 4, 32, 128), ("five", ops.BF16, 1, 2, 64, 64),
])
def test_single_launch_scan_equals_level_by_level(tree, dtype, h_k, h_v, d_k, d_v):
    rng = np.random.default_rng(31)
    parents = TREES[tree](rng)
    n_rows = np.array([len(p) + 1 + i % 2 for i, p in enumerate(parents)], np.int32)
    node_off = np.concatenate([[0], np.cumsum([len(p) for p in parents])]).astype(np.int32)
    n_layers, rows = 1024 // (len(parents) * h_v * (d_v // 16)) + 1, int(n_rows.sum())
    a = ops.make_gdn_operands(7, n_req=len(parents), n_layers=n_layers, total_rows=rows, h_k=h_k, h_v=h_v, d_k=d_k,
                              d_v=d_v, op_dtype=dtype)
    bf = dtype == ops.BF16
    t = {k: torch.from_numpy(x).cuda() for k, x in a.items()}
    if bf:
        t.update({k: t[k].view(torch.bfloat16) for k in "qkv"})
    row_off = np.concatenate([[0], np.cumsum(n_rows)])
    pad = [int(row_off[r]) + i for r, p in enumerate(parents) for i in range(len(p), int(n_rows[r]))]
    for k in ("q", "k", "v", "g", "beta"):
        t[k][:, pad] = float("nan")
    dims = L.dims(len(parents), n_layers, h_k, h_v, d_k, d_v, L.LUMO_BF16 if bf else L.LUMO_F32)
    for policy in (L.LUMO_POLICY_PATHS, L.LUMO_POLICY_TWO_LEVEL, L.LUMO_POLICY_RECOMPUTE):
        plan, blob = L.lumo_tree_plan(node_off, np.concatenate(parents), n_rows, policy)
        if tree in ("four", "five"):
            assert _slots(plan, blob) == (4 if tree == "four" else 5)
        desc = L.TreeDesc(plan, blob)
        need = L.lumo_tree_gdn_workspace_bytes(dims, plan)
        ws = torch.empty(max(need // 4, 4), dtype=torch.float32, device="cuda")
        out = []
        for dump in (False, True):
            print(f"[gpu] scan {tree} policy={policy} d={d_k}x{d_v} heads={h_k}/{h_v} bf16={bf} dump={dump}", flush=True)
            o = torch.full((n_layers, rows, h_v, d_v), 3.0, dtype=torch.bfloat16 if bf else torch.float32, device="cuda")
            ns = torch.zeros((n_layers, rows, h_v, d_k, d_v), device="cuda") if dump else None
            L.lumo_tree_gdn_verify(dims, desc, t["q"], t["k"], t["v"], t["g"], t["beta"], t["state0"], o, node_states=ns,
                                   workspace=ws if need else None)
            torch.cuda.synchronize()
            assert bool((o[:, pad] == 3.0).all())
            out.append(o.view(torch.int16 if bf else torch.int32).cpu())
        assert torch.equal(*out)
        assert bool(torch.isfinite(o.float()).all())
