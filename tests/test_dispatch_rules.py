"""The host rules that choose between two forms of a kernel (csrc/dispatch.h), compiled with the
host compiler and evaluated on plans: the form that was measured faster is the one taken."""
from __future__ import annotations

import ctypes
import os
import subprocess

import numpy as np
import pytest

import paper_2609_23900_amd as L
from lumo_synth import trees

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src = d / "rules.cpp"
    src.write_text('''#include "dispatch.h"
extern "C" int scan_tree(const lumo_gdn_dims* d, const lumo_plan* p, const int32_t* b) {
    return lumo::scan_tree_faster(*d, *p, b);
}
extern "C" int conv_run(const lumo_gdn_dims* d, const lumo_plan* p, const int32_t* b, int channels) {
    return lumo::conv_walk(*d, *p, b, channels).run_nodes;
}
extern "C" int wy_vector(const lumo_gdn_dims* d, const lumo_plan* p, const int32_t* b) {
    return lumo::wy_vector_faster(*d, *p, b);
}
extern "C" int replay(const lumo_gdn_dims* d, const lumo_plan* p, int max_path) {
    return lumo::replay_narrow(*d, *p, max_path);
}
''')
    lib = d / "rules.so"
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2609_23900_amd", "csrc"), str(src), "-o", str(lib)], check=True)
    return ctypes.CDLL(str(lib))


def _plan(parents, policy):
    off = np.concatenate([[0], np.cumsum([len(p) for p in parents])]).astype(np.int32)
    return L.lumo_tree_plan(off, np.concatenate(parents).astype(np.int32), np.diff(off).astype(np.int32), L.POLICIES[policy])


def _star(n):
    return np.array([-1] + [0] * (n - 1), np.int32)


def _levels(n, levels):
    return trees.random_tree(np.random.default_rng(5), n, levels, trees.bmax_uniform(4))


ONE = (1, 16, 32, 128, 128)  # one layer of 16 key and 32 value heads


@pytest.mark.parametrize("policy,tree,n_req,shape,single", [
    # measured at both forms: level by level first, then the single launch, us
    ("two_level", _star(256), 1, ONE, 0),          # 47, 143
    ("paths", _star(256), 1, ONE, 0),              # 48, 142
    ("paths", _star(64), 2, ONE, 0),               # 32, 40
    ("recompute", _star(256), 2, ONE, 0),          # 90, 144
    ("two_level", _levels(256, 8), 1, ONE, 0),     # 109, 143
    ("recompute", _levels(64, 8), 1, ONE, 0),      # 30, 37
    ("two_level", _levels(64, 8), 8, (2, 2, 4, 32, 128), 0),   # 18, 35
    ("two_level", _levels(200, 16), 8, (2, 4, 4, 16, 16), 0),  # 24, 46
    ("paths", _levels(256, 8), 1, ONE, 1),         # 178, 143
    ("paths", _levels(64, 8), 1, ONE, 1),          # 99, 39
    ("two_level", _levels(64, 8), 2, ONE, 1),      # 57, 39
    ("recompute", trees.chain(64), 1, ONE, 1),     # 153, 36
    ("paths", _star(256), 8, ONE, 1),              # 269, 167
    ("two_level", _levels(64, 8), 8, (2, 8, 8, 128, 16), 1),   # 43, 37
    ("two_level", _star(100), 64, (1, 16, 32, 64, 64), 1),     # beyond 1,024 column tiles
    ("paths", trees.chain(1), 64, (4, 16, 32, 128, 128), 0),   # 97, 154
    ("recompute", trees.chain(3), 64, (4, 16, 32, 128, 128), 0),   # 123, 179
    ("paths", trees.chain(16), 64, (4, 16, 32, 128, 128), 1),  # 427, 362
    ("paths", trees.chain(1), 64, (1, 8, 16, 64, 128), 0),     # 6.4, 10.9
    ("paths", trees.chain(2), 64, (4, 8, 8, 32, 128), 0),      # 8.7, 16.3
    ("recompute", trees.chain(8), 64, (4, 8, 16, 128, 16), 1),     # 63, 30
    ("recompute", _star(16), 1, ONE, 0),           # 7.6, 12.3
    ("paths", _star(33), 2, (1, 8, 16, 128, 16), 0),           # 14.9, 21.4
    ("paths", _levels(64, 8), 8, (6, 16, 32, 128, 128), 1),    # 1,175, 280
])
def test_scan_form_is_the_faster_one(rules, policy, tree, n_req, shape, single):
    plan, blob = _plan([tree] * n_req, policy)
    layers, h_k, h_v, d_k, d_v = shape
    d = L.dims(n_req, layers, h_k, h_v, d_k, d_v, L.LUMO_BF16)
    assert rules.scan_tree(ctypes.byref(d), ctypes.byref(plan), L._hptr(blob)) == single


def test_scan_rule_takes_empty_and_tiny_plans(rules):
    for parents in ([np.zeros(0, np.int32)], [trees.chain(1), np.zeros(0, np.int32)]):
        for policy in ("paths", "two_level", "recompute"):
            plan, blob = _plan(parents, policy)
            d = L.dims(len(parents), 1, 1, 1, 16, 16, L.LUMO_F32)
            assert rules.scan_tree(ctypes.byref(d), ctypes.byref(plan), L._hptr(blob)) in (0, 1)


@pytest.mark.parametrize("sizes,bf16,layers,channels,run", [
    ([2048] + [8] * 31, False, 1, 8192, 0),       # run kernel 36 us, walk 157
    ([2048] + [8] * 31, True, 4, 8192, 0),        # 93, 130
    ([65] * 64, True, 2, 8192, 0),                # 77, 96
    ([17] * 128, False, 2, 8192, 0),              # 88, 99
    ([65] * 64, False, 1, 8192, 16),              # 76, 60
    ([64] * 8, False, 12, 8192, 16),              # 125, 82
    ([64] * 8, False, 1, 8192, 0),                # too few blocks
    ([256] * 32, True, 1, 8192, 64),              # 64, 56
    ([16, 128] * 32, True, 2, 8192, 64),          # 93, 91
    ([16, 128] * 32, False, 1, 8192, 16),         # 96, 85
    ([28] * 64, False, 3, 8192, 16),              # 110, 76
    ([33] * 32, False, 4, 8192, 16),              # 84, 63
    ([512] * 4 + [64] * 28, False, 6, 2304, 16),  # 168, 112
    ([512] * 4 + [64] * 28, True, 4, 8192, 0),    # 135, 232
    ([256] + [32] * 31, False, 2, 8192, 0),       # 35, 48
    ([256, 32] * 8, False, 2, 8192, 16),          # 96, 74
    ([512] * 4 + [64] * 28, False, 1, 8192, 0),   # 48, 131: an XCD takes all the large trees
    ([64] * 28 + [512] * 4, False, 2, 8192, 0),
    ([512] * 4 + [64] * 28, False, 4, 8192, 16),  # 303, 298
    ([512], False, 8, 8192, 16),                  # one request is spread by its channels
])
def test_conv_walk_is_taken_where_it_is_faster(rules, sizes, bf16, layers, channels, run):
    rng = np.random.default_rng(9)
    parents = [trees.random_tree(rng, n, 17, trees.bmax_uniform(4)) if n > 17 else trees.chain(n) for n in sizes]
    plan, blob = _plan(parents, "recompute")
    d = L.dims(len(sizes), layers, 1, 1, 128, 128, L.LUMO_BF16 if bf16 else L.LUMO_F32)
    assert rules.conv_run(ctypes.byref(d), ctypes.byref(plan), L._hptr(blob), channels) == run


def test_conv_walk_refuses_long_paths(rules):
    plan, blob = _plan([trees.chain(18)] * 64, "recompute")
    d = L.dims(64, 48, 1, 1, 128, 128, L.LUMO_F32)
    assert rules.conv_run(ctypes.byref(d), ctypes.byref(plan), L._hptr(blob), 8192) == 0


@pytest.mark.parametrize("heads,d_k,d_v,bf16,depth,max_path,narrow", [
    # measured with 64 and with 16 columns, us
    ((1, 1, 32), 128, 128, True, 32, 32, 1),      # 8 steps 18.5, 10.0
    ((64, 1, 32), 128, 128, True, 32, 32, 1),     # 63.7, 54.0
    ((64, 1, 32), 64, 128, True, 32, 32, 0),      # 33.0, 39.4
    ((16, 1, 32), 64, 128, True, 32, 32, 1),      # 16.5, 14.2
    ((16, 1, 48), 64, 128, True, 32, 32, 1),      # 18.4, 18.4; 32 steps 46, 36
    ((16, 1, 48), 64, 128, False, 32, 32, 0),     # 16.9, 18.5
    ((64, 4, 32), 64, 128, False, 32, 32, 0),     # 101, 141: at the 256 MB
    ((64, 1, 32), 32, 128, False, 32, 32, 0),     # 21.6, 26.0
    ((64, 4, 48), 32, 128, False, 32, 32, 0),     # 88, 109
    ((16, 1, 32), 64, 64, False, 32, 32, 1),      # 12.9, 10.3
    ((64, 1, 32), 64, 64, False, 32, 32, 0),      # 23.5, 24.4
    ((64, 4, 48), 128, 16, True, 32, 32, 1),      # 115, 52
    ((64, 4, 32), 16, 16, False, 32, 32, 1),      # 17.7, 15.4
    ((16, 1, 32), 128, 128, True, 1, 16, 0),      # one step 14.3, 17.2
    ((16, 1, 32), 128, 128, True, 16, 2, 0),      # two steps, 1.12 times
    ((16, 1, 32), 128, 128, True, 16, 4, 1),      # four steps, 0.99 times
    ((64, 1, 32), 128, 128, False, 1, 16, 1),     # 51.3, 48.0
    ((4, 1, 32), 128, 128, True, 1, 16, 1),       # 9.2, 8.4
    ((18, 8, 32), 128, 128, True, 32, 32, 0),     # beyond the cache: 122, 136
])
def test_replay_form_is_the_faster_one(rules, heads, d_k, d_v, bf16, depth, max_path, narrow):
    n_req, layers, h_v = heads
    plan, _ = _plan([trees.chain(depth)] * n_req, "recompute")
    d = L.dims(n_req, layers, 1, h_v, d_k, d_v, L.LUMO_BF16 if bf16 else L.LUMO_F32)
    assert rules.replay(ctypes.byref(d), ctypes.byref(plan), max_path) == narrow


def _deep(n, depth):
    """A chain of `depth` nodes, the others under the root."""
    return np.array(list(range(-1, depth - 1)) + [0] * (n - depth), np.int32)


@pytest.mark.parametrize("sizes,layers,h_v,bf16,vector", [
    # (nodes, levels) per request; measured on the matrix cores and on the vector ALUs, us
    ([(1, 1)], 1, 32, False, 1),                          # 10.0, 5.4
    ([(3, 3)] * 4, 1, 32, False, 1),                      # 10.0, 9.5
    ([(4, 4)], 1, 32, False, 0),                          # 10.0, 11.5
    ([(4, 4)] * 64, 1, 32, False, 1),                     # 47, 37
    ([(1, 1)] * 64, 4, 32, False, 1),                     # 185, 97
    ([(7, 7)] * 64, 1, 32, False, 0),                     # 47, 51
    ([(8, 4)] * 64, 4, 32, False, 0),
    ([(12, 12)] * 64, 1, 32, False, 0),                   # 60, 78
    ([(18, 18)] * 64, 1, 32, False, 1),                   # 141, 115
    ([(18, 18)] * 16, 1, 32, False, 0),                   # 38, 52
    ([(24, 24)] * 64, 1, 32, False, 0),                   # 134, 151
    ([(64, 8)] * 8, 12, 32, False, 0),
    ([(64, 18)] * 64, 4, 32, False, 0),
    ([(1, 1)] * 63 + [(18, 18)], 4, 32, False, 1),        # 363, 136
    ([(1, 1)] * 63 + [(64, 20)], 4, 32, False, 1),        # 378, 268
    ([(1, 1)] * 63 + [(64, 20)], 1, 32, False, 0),
    ([(1, 1)] * 63 + [(64, 8)], 4, 32, False, 0),         # 194, 242
    ([(4, 4)] * 63 + [(18, 18)], 4, 32, True, 0),         # 172, 188
    ([(0, 0)] * 63 + [(1, 1)], 1, 32, False, 1),
    ([(1, 1)] * 63 + [(18, 18)], 4, 32, True, 1),         # 171, 137
    ([(18, 18)] * 64, 4, 32, True, 0),
    ([(96, 32)] * 16, 4, 32, True, 0),
    ([(1, 1)] * 64, 4, 32, True, 0),                      # paths of up to 17 nodes: always the matrix cores
])
def test_wy_form_is_the_faster_one(rules, sizes, layers, h_v, bf16, vector):
    plan, blob = _plan([_deep(*s) if s[0] else np.zeros(0, np.int32) for s in sizes], "wy")
    d = L.dims(len(sizes), layers, 1, h_v, 128, 128, L.LUMO_BF16 if bf16 else L.LUMO_F32)
    assert rules.wy_vector(ctypes.byref(d), ctypes.byref(plan), L._hptr(blob)) == vector
