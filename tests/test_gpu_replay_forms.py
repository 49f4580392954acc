"""The commit's two replay forms (16-column tiles; 64-column tiles for state banks beyond 256
MB) publish the same bits: the layers of one large call against the same layers committed one
by one, with paths around the 16 staged entries (1, 15, 16, 17 and 33 nodes), none and an
invalid one, ragged requests, and operands prepared in the kernel."""
from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU, skipped there
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2609_23900_amd as L  # noqa: E402
from lumo_synth import trees  # noqa: E402


@pytest.mark.parametrize("bf16,d_k,d_v,h_k,h_v,flags", [(True, 128, 128, 2, 6, 0), (True, 128, 128, 4, 4, 3),
                                                       (False, 128, 128, 2, 4, 3), (False, 16, 64, 8, 16, 0),
                                                       (True, 64, 16, 16, 16, 0), (False, 32, 128, 4, 8, 1)])
def test_replay_forms_publish_the_same_bits(bf16, d_k, d_v, h_k, h_v, flags):
    parents = [trees.chain(33), trees.chain(17), trees.chain(16), trees.FIG1_PARENT, trees.chain(15)]
    accepted = torch.tensor([32, 16, 15, 99, 0], dtype=torch.int32, device="cuda")
    n_rows = np.array([len(p) + 1 for p in parents], np.int32)
    node_off = np.concatenate([[0], np.cumsum([len(p) for p in parents])]).astype(np.int32)
    n_req, rows = len(parents), int(n_rows.sum())
    bank = n_req * h_v * d_k * d_v * 4  # of one layer
    n_layers = (256 << 20) // bank + 2  # beyond the line
    dt = torch.bfloat16 if bf16 else torch.float32
    g = torch.Generator(device="cuda").manual_seed(71)

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda")

    k = torch.nn.functional.normalize(normal(n_layers, rows, h_k, d_k), dim=-1).to(dt)
    v = normal(n_layers, rows, h_v, d_v).to(dt)
    gate, beta = -torch.nn.functional.softplus(normal(n_layers, rows, h_v)), torch.sigmoid(normal(n_layers, rows, h_v))
    a_log, dt_bias = 0.5 * normal(n_layers, h_v), normal(n_layers, h_v)
    state = normal(n_req, n_layers, h_v, d_k, d_v)
    desc = L.TreeDesc.build(node_off, np.concatenate(parents).astype(np.int32), n_rows, L.LUMO_POLICY_RECOMPUTE)
    path = torch.zeros((n_req, 40), dtype=torch.int32, device="cuda")
    plen = torch.zeros(n_req, dtype=torch.int32, device="cuda")
    code = L.LUMO_BF16 if bf16 else L.LUMO_F32

    def commit(lo, hi):
        prep = L.Prep(flags, 1e-6, a_log[lo:hi].clone(), dt_bias[lo:hi].clone()) if flags else None
        s = state[:, lo:hi].clone(memory_format=torch.contiguous_format)
        L.lumo_gdn_commit_prep(L.dims(n_req, hi - lo, h_k, h_v, d_k, d_v, code), desc, prep, 40, accepted, path, plen,
                               k[lo:hi].clone(), v[lo:hi].clone(), gate[lo:hi].clone(), beta[lo:hi].clone(), s)
        torch.cuda.synchronize()
        return s

    print(f"[gpu] replay forms bf16={bf16} d={d_k}x{d_v} heads={h_k}/{h_v} prep={flags} layers={n_layers}", flush=True)
    whole = commit(0, n_layers)
    assert plen.tolist() == [33, 17, 16, -1, 1]
    for l in sorted({0, 1, n_layers // 2, n_layers - 1}):
        assert torch.equal(whole[:, l:l + 1].view(torch.int32), commit(l, l + 1).view(torch.int32)), l
    assert torch.equal(whole[3].view(torch.int32), state[3].view(torch.int32))  # the invalid selection
    assert not torch.equal(whole[0], state[0])


@pytest.mark.parametrize("bf16,d_k,d_v,h_v,longest", [(True, 64, 128, 8, 33), (False, 32, 64, 8, 17), (True, 128, 128, 4, 3),
                                                      (False, 16, 16, 8, 2), (True, 128, 64, 4, 1)])
def test_large_grids_publish_the_bits_of_single_layers(bf16, d_k, d_v, h_v, longest):
    """Shapes that take 64-column tiles within 256 MB (more than 1,536 tiles of short keys, and
    trees of up to three levels), against the same layers one by one, which take 16 columns."""
    parents = [trees.chain(1), trees.chain(longest), trees.chain(max(1, longest - 1)), trees.chain(longest)]
    accepted = torch.tensor([0, longest - 1, 0, 99], dtype=torch.int32, device="cuda")
    n_rows = np.array([len(p) for p in parents], np.int32)
    node_off = np.concatenate([[0], np.cumsum(n_rows)]).astype(np.int32)
    n_req, rows = len(parents), int(n_rows.sum())
    n_layers = 1536 // (n_req * h_v * ((d_v + 63) // 64)) + 2
    dt = torch.bfloat16 if bf16 else torch.float32
    g = torch.Generator(device="cuda").manual_seed(72)

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda")

    k = torch.nn.functional.normalize(normal(n_layers, rows, 2, d_k), dim=-1).to(dt)
    v = normal(n_layers, rows, h_v, d_v).to(dt)
    gate, beta = -torch.nn.functional.softplus(normal(n_layers, rows, h_v)), torch.sigmoid(normal(n_layers, rows, h_v))
    state = normal(n_req, n_layers, h_v, d_k, d_v)
    desc = L.TreeDesc.build(node_off, np.concatenate(parents).astype(np.int32), n_rows, L.LUMO_POLICY_RECOMPUTE)
    path = torch.zeros((n_req, 40), dtype=torch.int32, device="cuda")
    plen = torch.zeros(n_req, dtype=torch.int32, device="cuda")

    def commit(lo, hi):
        s = state[:, lo:hi].clone(memory_format=torch.contiguous_format)
        L.lumo_gdn_commit(L.dims(n_req, hi - lo, 2, h_v, d_k, d_v, L.LUMO_BF16 if bf16 else L.LUMO_F32), desc, 40, accepted,
                          path, plen, k[lo:hi].clone(), v[lo:hi].clone(), gate[lo:hi].clone(), beta[lo:hi].clone(), s)
        torch.cuda.synchronize()
        return s

    print(f"[gpu] replay large grid bf16={bf16} d={d_k}x{d_v} heads={h_v} longest={longest} layers={n_layers}", flush=True)
    whole = commit(0, n_layers)
    assert plen.tolist() == [1, longest, 1, -1]
    for l in (0, n_layers - 1):
        assert torch.equal(whole[:, l:l + 1].view(torch.int32), commit(l, l + 1).view(torch.int32)), l
    assert not torch.equal(whole[0], state[0])
