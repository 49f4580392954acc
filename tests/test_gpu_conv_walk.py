"""The tree conv's walk over runs (large grids) against the run kernel, bit for bit.

A batch large enough for the walk is convolved in one call and request by request (calls too
small for it): every output must have the same bits, and pad rows (NaN) are neither read
nor written. Trees end on and around the runs (16 nodes fp32, 64 bf16), have paths up to the
walk's limit of 17 nodes, and their runs start deep in a branch and leave it again; channel
counts include a partial last chunk.
"""
from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU, skipped there
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2609_23900_amd as L  # noqa: E402
from lumo_synth import trees  # noqa: E402


@pytest.mark.parametrize("bf16,channels,n_layers,act,with_bias", [(False, 2056, 10, 1, True), (False, 1024, 20, 0, False),
                                                                 (True, 4104, 24, 1, False), (True, 4096, 24, 0, True)])
def test_walk_equals_run_kernel(bf16, channels, n_layers, act, with_bias):
    rng = np.random.default_rng(61)
    # full trees beside the edge sizes: the walk is for batches whose runs are mostly full
    sizes = (1, 15, 16, 17, 0, 33, 63, 64, 65, 128, 129, 200) + (256,) * 8
    parents = [trees.random_tree(rng, n, 17, trees.bmax_uniform(2 + i % 3)) if n > 1 else trees.chain(n)
               for i, n in enumerate(sizes)] + [trees.chain(17)]
    n_rows = np.array([len(p) + 1 for p in parents], np.int32)
    node_off = np.concatenate([[0], np.cumsum([len(p) for p in parents])]).astype(np.int32)
    row_off = np.concatenate([[0], np.cumsum(n_rows)])
    nodes, rows, n_req = int(node_off[-1]), int(row_off[-1]), len(parents)
    per, lane = (64, 8) if bf16 else (16, 4)
    runs = sum(-(-len(p) // per) for p in parents)  # the walk's lines
    assert nodes // per * n_layers * -(-channels // (64 * lane)) >= 2048
    assert 4 * nodes >= 3 * per * runs and 2 * runs >= n_req * -(-256 // per)
    dt = torch.bfloat16 if bf16 else torch.float32
    g = torch.Generator(device="cuda").manual_seed(62)

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda").to(dt)

    x, hist = normal(n_layers, rows, channels), normal(n_req, n_layers, 3, channels)
    w = torch.randn((n_layers, channels, 4), generator=g, device="cuda")
    bias = torch.randn((n_layers, channels), generator=g, device="cuda") if with_bias else None
    x[:, [int(o) - 1 for o in row_off[1:]]] = float("nan")  # each request's pad row
    code = L.LUMO_BF16 if bf16 else L.LUMO_F32

    def conv(lo, hi):
        par = np.concatenate(parents[lo:hi]).astype(np.int32)
        desc = L.TreeDesc.build(node_off[lo:hi + 1] - node_off[lo], par, n_rows[lo:hi], L.LUMO_POLICY_RECOMPUTE)
        xs = x[:, int(row_off[lo]):int(row_off[hi])].contiguous()
        y = torch.full_like(xs, 5.0)
        L.lumo_tree_conv_gather(L.dims(hi - lo, n_layers, 1, 1, 128, 128, code), desc, channels, xs,
                                hist[lo:hi].contiguous(), w, bias, act, y)
        torch.cuda.synchronize()
        return y

    print(f"[gpu] conv walk bf16={bf16} channels={channels} layers={n_layers}", flush=True)
    whole = conv(0, n_req)
    apart = torch.cat([conv(r, r + 1) for r in range(n_req)], 1)
    bits = torch.int16 if bf16 else torch.int32
    assert torch.equal(whole.view(bits), apart.view(bits))
    assert bool(torch.isfinite(whole.float()).all())
    assert bool((whole[:, [int(o) - 1 for o in row_off[1:]]] == 5.0).all())
