"""The WY verification of paths of 18 to 32 nodes on the matrix cores (bf16, d = 128).

Every node against the fp64 oracle, at the edges of the path registers (18, 31 and 32
nodes), of the 32-node chunks and their halves, with path stacks that reach back over
several chunks; plain and with operands prepared in the kernel. Outputs are bf16: besides
the tolerance of the other parity tests, the state keeps all its fp32 bits here, so an output
may be off by its own rounding (bf16 has 8 significant bits, so half a unit in the last place
is at most 2^-8 of the value) plus fp32 arithmetic over at most 32
updates (bounded by 2^-12 of the head's largest output).
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
    rng = np.random.default_rng(41)
    if case == "chains":  # chunk and half-chunk edges, the depth limits
        return [trees.chain(n) for n in (18, 31, 32, 1)]
    if case == "stacks":  # a 31-deep spine with leaves at every level, visited last: deep stacks in every chunk
        spine = list(range(-1, 30))
        return [np.array(spine + [i % 31 for i in range(62)], np.int32), np.zeros(0, np.int32)]
    return [trees.random_tree(rng, n, d, trees.bmax_uniform(2)) for n, d in ((49, 18), (64, 32), (97, 25))]


@pytest.mark.parametrize("case,h_k,h_v,flags", [("chains", 1, 1, 0), ("chains", 2, 4, QKN | RAWG), ("stacks", 1, 3, 0),
                                                ("random", 2, 2, 0), ("random", 2, 4, QKN)])
def test_deep_paths_against_oracle(case, h_k, h_v, flags):
    parents = _trees(case)
    n_rows = [len(p) + i % 2 for i, p in enumerate(parents)]
    wl = pins.make_wl(parents, d_k=128, d_v=128, h_k=h_k, h_v=h_v, op_dtype=ops.BF16, n_rows=n_rows, n_layers=2,
                      max_path=32)
    a = ops.make_gdn_operands(43, n_req=wl.n_req, n_layers=2, total_rows=wl.total_rows, h_k=h_k, h_v=h_v, d_k=128,
                              d_v=128, op_dtype=ops.BF16)
    rng = np.random.default_rng(44)
    oprep = gprep = None
    if flags:
        a["g"] = rng.standard_normal(a["g"].shape).astype(np.float32) if flags & RAWG else a["g"]
        a["beta"] = rng.standard_normal(a["beta"].shape).astype(np.float32) if flags & RAWG else a["beta"]
        a_log = (0.5 * rng.standard_normal((2, h_v))).astype(np.float32)
        dt_bias = rng.standard_normal((2, h_v)).astype(np.float32)
        oprep = oracle.Prep(flags, 1e-6, a_log, dt_bias)
        gprep = L.Prep(flags, 1e-6, torch.from_numpy(a_log).cuda(), torch.from_numpy(dt_bias).cuda())
    wl.arrays = a
    print(f"[gpu] deep paths {case} heads={h_k}/{h_v} prep={flags}", flush=True)
    st = GdnTreeStep(n_req=wl.n_req, n_layers=2, h_k=h_k, h_v=h_v, d_k=128, d_v=128, op_dtype=ops.BF16,
                     node_off=wl.node_off, parent=wl.parent_flat, n_rows=wl.n_rows, arrays=a,
                     policy=L.LUMO_POLICY_WY, max_path=32, accepted=wl.accepted, prep=gprep)
    st.verify()
    torch.cuda.synchronize()
    o = gu.to_np(st.o)
    for r, par in enumerate(parents):
        for l in range(2):
            for h in range(h_v):
                if len(par) == 0:
                    continue
                ref = oracle.verify_nodes(wl, r, l, h, list(range(len(par))), arrays=a, prep=oprep)
                got = o[l, gu.node_rows(wl, r), h]
                err = np.abs(got - ref) - np.abs(ref) * 2.0 ** -8
                assert err.max() <= 2.0 ** -12 * np.abs(ref).max(), (r, l, h, float(err.max()))
