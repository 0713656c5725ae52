"""The terms of the fp64 sweeps at the edges of the range in which they may be referenced to 0 (|s| <= 600): values
beyond it on either side, masked and broken rows, temperatures at which the 16-bit tables cannot be used, and
ragged vocabularies, for chains and for trees, against the oracle."""
import numpy as np
import pytest
import torch

from paper_2512_16273_amd import workloads as W
from tests import _parity as P

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def t32(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def edge_rows(t):
    """Rows that leave the range, one way per sequence or node (t [n, V] fp32)."""
    t[0, ::7] = -700.0                        # far below: exp is 0 beside the rest of the row
    t[1] += 650.0                             # the whole row above the range
    t[2, 100:] = -float("inf")                # mostly masked
    t[3] -= 640.0                             # the whole row below the range
    t[4, 3::5] = -float("inf")
    t[5, 0] = -599.0                          # just inside, and just outside
    t[5, -1] = -601.0
    return t


@pytest.mark.parametrize("dtype,V,T", [("f32", 9001, 1.0), ("f32", 4096, 0.7), ("f32", 1000, 1.0), ("bf16", 9001, 0.15),
                                       ("f16", 9001, 0.05), ("f16", 9001, 1.0), ("f16", 120000, 1.0)])
def test_chain_terms(tslt, dtype, V, T):
    w = W.scaled(W.WORKLOADS["chain_topk"], B=7, V=V, gamma=3, dtype=dtype, T=T)
    if T < 0.5:                               # scaled values as at T = 1
        w = W.scaled(w, sigma=w.sigma * T, zipf=w.zipf * T, noise_t=w.noise_t * T)
    chain = W.make_chain(w, 19, DEV)
    target = chain["target"].float()
    target[:6, 0] = edge_rows(target[:6, 0].clone())
    target[:6, 3] = edge_rows(target[:6, 3].clone())        # the bonus rows
    chain["target"] = target.to(W.torch_dtype(dtype))
    u_acc = chain["u_accept"].clone()
    u_acc[:, 0] = 0.9995
    u_acc[:2] = 0.0
    chain["u_accept"] = u_acc
    ref = P.oracle_chain(P.to_np(chain["draft"]), P.to_np(chain["target"]), w.T, w.top_k, w.top_p, w.k_cap,
                         P.to_np(chain["u_sample"]), P.to_np(u_acc), P.to_np(chain["u_resample"]))
    out = tslt.verify(chain["target"], w.T, t32(ref["q_idx"]), t32(ref["q_logit"]), t32(ref["q_count"]), t32(ref["tokens"]),
                      u_acc, chain["u_resample"])
    torch.cuda.synchronize()
    # a rate below fp32's range cannot be told from 0 in the fp32 output
    ref["verify"]["beta_hat"] = ref["verify"]["beta_hat"].astype(np.float32)
    print(P.compare_verify(out, ref["verify"], label=f"{dtype} {V} {T}"), ref["verify"]["accept_len"])


@pytest.mark.parametrize("dtype,V,T", [("f32", 9001, 1.0), ("f32", 4097, 0.6), ("f16", 9001, 0.9), ("bf16", 9001, 0.15)])
def test_tree_terms(tslt, dtype, V, T):
    w = W.scaled(W.WORKLOADS["tree"], B=2, V=V, expansion=(3, 2), top_k=8, k_cap=8, dtype=dtype, T=T)
    if T < 0.5:
        w = W.scaled(w, sigma=w.sigma * T, zipf=w.zipf * T, noise_t=w.noise_t * T)
    tree = W.make_tree(w, 23, DEV)
    target = tree["target"].float()
    target[0, 4:10] = edge_rows(target[0, 4:10].clone())             # the leaves
    rows = target[1, :6].clone()                                     # the non-leaf nodes (the shifted rows among them:
    rows[[0, 4, 2, 1, 3, 5]] = edge_rows(rows[[0, 4, 2, 1, 3, 5]])   # test_tree_terms_at_every_inner_node)
    target[1, :4] = torch.stack([rows[0], rows[4], rows[2], rows[5]])
    tree["target"] = target.to(W.torch_dtype(dtype))
    ref = P.oracle_tree(P.to_np(tree["draft"]), P.to_np(tree["target"]), w.T, w.top_k, w.top_p, w.k_cap, w.expansion,
                        P.to_np(tree["u_sample"]), P.to_np(tree["u_accept"]), P.to_np(tree["u_resample"]), False, False)
    args = [tree["target"], w.T, w.expansion, t32(ref["q_idx"]), t32(ref["q_logit"]), t32(ref["q_count"]), t32(ref["cands"]),
            tree["u_accept"], tree["u_resample"]]
    out = tslt.verify_tree(*args, all_nodes=True)
    path = tslt.verify_tree(*args, all_nodes=False)
    torch.cuda.synchronize()
    print(P.compare_tree(out, ref, w.expansion, all_nodes=True, label=f"{dtype} {V} {T}"))
    assert torch.equal(path["seq"], out["seq"]) and torch.equal(path["len"], out["len"])


@pytest.mark.parametrize("dtype,B,gamma,V", [
    ("bf16", 64, 7, 1203),     # 512 rows: two per compute unit in one pass (one through the bit table)
    ("bf16", 103, 4, 2500),    # beyond that: acceptance and resampling apart
    ("f32", 64, 3, 1203),      # 256 rows: the largest batch in one pass for the other types
    ("f16", 65, 3, 1203),
    ("f16", 300, 1, 1100),     # more sequences than compute units
    ("f32", 1, 70, 700),       # more positions than a wave has lanes
    ("bf16", 2, 130, 130),     # ... with V as wide as the set
])
def test_batches_on_either_side_of_the_dispatch(tslt, dtype, B, gamma, V):
    w = W.scaled(W.WORKLOADS["chain_topk"], B=B, V=V, gamma=gamma, dtype=dtype, top_k=32, k_cap=130)
    chain = W.make_chain(w, 29, DEV)
    u_acc = chain["u_accept"].clone()
    u_acc[0] = 0.0                             # everything accepted wherever the token can be
    chain["u_accept"] = u_acc
    ref = P.oracle_chain(P.to_np(chain["draft"]), P.to_np(chain["target"]), w.T, w.top_k, w.top_p, w.k_cap,
                         P.to_np(chain["u_sample"]), P.to_np(u_acc), P.to_np(chain["u_resample"]))
    args = [chain["target"], w.T, t32(ref["q_idx"]), t32(ref["q_logit"]), t32(ref["q_count"]), t32(ref["tokens"]), u_acc,
            chain["u_resample"]]
    out = tslt.verify(*args)
    torch.cuda.synchronize()
    print(P.compare_verify(out, ref["verify"], label=f"{dtype} {B}x{gamma} {V}"))
    ws = torch.empty(tslt.workspace_bytes(tslt.OP_VERIFY, B, gamma, V, w.k_cap), dtype=torch.uint8, device=DEV)
    halves = {k: torch.empty_like(v) for k, v in out.items()}
    tslt.verify(*args, out=halves, workspace=ws, phase="accept")
    tslt.verify(*args, out=halves, workspace=ws, phase="resample")
    torch.cuda.synchronize()
    for k in out:
        assert torch.equal(out[k], halves[k]), k


@pytest.mark.parametrize("dtype,B,expansion,V", [
    ("f32", 34, (2, 2, 2), 2000),      # 510 nodes: every node at once, then the walk
    ("f32", 35, (2, 2, 2), 2000),      # 525: node after node
    ("f16", 19, (4, 2), 1500),         # 247 nodes of a tree of two layers
    ("f16", 20, (4, 2), 1500),         # 260
    ("f32", 35, (2, 2, 2), 100001),    # two layers at once, then node after node
    ("f16", 30, (3, 3), 100000),       # the same of a tree of two layers
    ("bf16", 170, (1, 1), 900),        # 510
    ("bf16", 171, (1, 1), 900),        # 513
])
def test_path_on_either_side_of_the_dispatch(tslt, dtype, B, expansion, V):
    """The verified path alone gives what the evaluation of every node gives along it, and NaN off it."""
    w = W.scaled(W.WORKLOADS["tree"], B=B, V=V, expansion=expansion, top_k=8, k_cap=8, dtype=dtype)
    tree = W.make_tree(w, 31, DEV)
    offsets, width = [0], 1
    for k in expansion + (0,):
        offsets.append(offsets[-1] + width)
        width *= k
    n_int, n = offsets[-2], offsets[-1]
    draft = tree["draft"].reshape(B * n_int, V)
    u = W.uniforms((B * n_int, max(expansion)), 5, 2, 3, DEV)
    sets = tslt.truncate(draft, w.T, 8, 0.0, 8, u=u)
    token = sets["token"].view(B, n_int, -1)
    cands = torch.cat([token[:, lo:hi, :k].reshape(B, -1) for k, lo, hi in zip(expansion, offsets, offsets[1:])], 1).contiguous()
    args = [tree["target"], w.T, expansion, sets["idx"].view(B, n_int, 8), sets["logit"].view(B, n_int, 8),
            sets["count"].view(B, n_int), cands, tree["u_accept"], tree["u_resample"]]
    out = {k: P.to_np(v) for k, v in tslt.verify_tree(*args, all_nodes=True).items()}
    path = {k: P.to_np(v) for k, v in tslt.verify_tree(*args, all_nodes=False).items() if v is not None}
    assert np.array_equal(path["seq"], out["seq"]) and np.array_equal(path["len"], out["len"])
    lengths = set()
    for b in range(B):
        on = np.zeros(n - 1, bool)
        node = 0
        for layer, k in enumerate(expansion):
            child = offsets[layer + 1] + (node - offsets[layer]) * k
            on[child - 1:child - 1 + k] = True
            if out["node_slot"][b, node] < 0:
                break
            node = child + out["node_slot"][b, node]
        lengths.add(int(out["len"][b]))
        for k in ("ratio", "beta"):
            assert np.isnan(path[k][b][~on]).all()
            # fp64 sums of terms within 1.5 ulp by either table, rounded to fp32
            np.testing.assert_allclose(path[k][b][on], out[k][b][on], rtol=2.5e-7)
    assert len(lengths) > 1 and (path["status"] == 0).all()


def mask_rows(t, low):
    """Rows masked with a finite value far below the range, one way per sequence or node (t [n, V] fp32)."""
    V = t.shape[1]
    t[0, -5:] = low                            # the vocabulary's padding
    t[1, V // 10:] = low                       # whole runs
    t[2, ::97] = low                           # a few elements of nearly every vector's neighbourhood
    t[3, :V // 2] = -float("inf")              # masks of both kinds
    t[3, V // 2:V - 40] = low
    t[4] = low                                 # nothing but masks: every token alike
    t[5, :V - 9] = low                         # ... and a few tokens that are not in whole vectors
    t[5, V - 9:] -= 700.0                      # below the range as well: the row by its maximum
    return t


@pytest.mark.parametrize("dtype,V,B", [("f32", 9001, 7), ("bf16", 9001, 7), ("f16", 9001, 7), ("f32", 2003, 300), ("bf16", 2003, 300),
                                       ("f16", 2003, 300)])
def test_chain_finite_masks(tslt, dtype, V, B):
    low = -60000.0 if dtype == "f16" else -1.0e9
    w = W.scaled(W.WORKLOADS["chain_topk"], B=B, V=V, gamma=2, dtype=dtype, T=0.9, top_k=16, k_cap=16)
    chain = W.make_chain(w, 47, DEV)
    target = chain["target"].float()
    target[:6, 0] = mask_rows(target[:6, 0].clone(), low)
    target[:6, 2] = mask_rows(target[:6, 2].clone(), low)       # the bonus rows
    chain["target"] = target.to(W.torch_dtype(dtype))
    u_acc = chain["u_accept"].clone()
    u_acc[:, 0] = 0.9995
    chain["u_accept"] = u_acc
    ref = P.oracle_chain(P.to_np(chain["draft"]), P.to_np(chain["target"]), w.T, w.top_k, w.top_p, w.k_cap,
                         P.to_np(chain["u_sample"]), P.to_np(u_acc), P.to_np(chain["u_resample"]))
    out = tslt.verify(chain["target"], w.T, t32(ref["q_idx"]), t32(ref["q_logit"]), t32(ref["q_count"]), t32(ref["tokens"]),
                      u_acc, chain["u_resample"])
    # the bonus rows: the same positions with nearly everything accepted (a token whose p is 0 is not)
    u0 = torch.full_like(u_acc, 1e-3)
    ref0 = P.oracle_chain(P.to_np(chain["draft"]), P.to_np(chain["target"]), w.T, w.top_k, w.top_p, w.k_cap,
                          P.to_np(chain["u_sample"]), P.to_np(u0), P.to_np(chain["u_resample"]))
    out0 = tslt.verify(chain["target"], w.T, t32(ref0["q_idx"]), t32(ref0["q_logit"]), t32(ref0["q_count"]), t32(ref0["tokens"]),
                       u0, chain["u_resample"])
    torch.cuda.synchronize()
    for o, r in ((out, ref), (out0, ref0)):
        r["verify"]["beta_hat"] = r["verify"]["beta_hat"].astype(np.float32)
        print(P.compare_verify(o, r["verify"], label=f"{dtype} {V} {B}"), r["verify"]["accept_len"][:7])


@pytest.mark.parametrize("dtype,B", [("f32", 2), ("bf16", 2), ("f16", 2), ("f32", 60), ("bf16", 60), ("f16", 60)])
def test_tree_finite_masks(tslt, dtype, B):
    """Leaves and non-leaf nodes; 60 trees of 10 nodes are walked node after node."""
    low = -60000.0 if dtype == "f16" else -1.0e9
    w = W.scaled(W.WORKLOADS["tree"], B=B, V=3001, expansion=(3, 2), top_k=8, k_cap=8, dtype=dtype, T=0.9)
    tree = W.make_tree(w, 53, DEV)
    target = tree["target"].float()
    target[0, 4:10] = mask_rows(target[0, 4:10].clone(), low)
    rows = mask_rows(target[1, :6].clone(), low)
    target[1, :4] = rows[[0, 1, 5, 4]]
    target[0, :4] = rows[[2, 3, 4, 5]]
    tree["target"] = target.to(W.torch_dtype(dtype))
    ref = P.oracle_tree(P.to_np(tree["draft"]), P.to_np(tree["target"]), w.T, w.top_k, w.top_p, w.k_cap, w.expansion,
                        P.to_np(tree["u_sample"]), P.to_np(tree["u_accept"]), P.to_np(tree["u_resample"]), False, False)
    args = [tree["target"], w.T, w.expansion, t32(ref["q_idx"]), t32(ref["q_logit"]), t32(ref["q_count"]), t32(ref["cands"]),
            tree["u_accept"], tree["u_resample"]]
    out = tslt.verify_tree(*args, all_nodes=True)
    path = tslt.verify_tree(*args, all_nodes=False)
    torch.cuda.synchronize()
    print(P.compare_tree(out, ref, w.expansion, all_nodes=True, label=f"{dtype} {B}"))
    assert torch.equal(path["seq"], out["seq"]) and torch.equal(path["len"], out["len"])


@pytest.mark.parametrize("dtype,B,wor", [("f32", 2, False), ("f32", 90, True), ("bf16", 90, False), ("f16", 2, True), ("f16", 90, False)])
def test_tree_terms_at_every_inner_node(tslt, dtype, B, wor):
    """The rows of edge_rows at non-leaf nodes: candidates tested, updates made and tokens drawn on a row that was swept again by
    its maximum, and the walk going on from such a node (90 trees of 6 nodes are walked node after node)."""
    w = W.scaled(W.WORKLOADS["tree"], B=B, V=4097, expansion=(2, 1), top_k=8, k_cap=8, dtype=dtype, T=1.0, without_replacement=wor)
    tree = W.make_tree(w, 71, DEV)
    target = tree["target"].float()
    for first, b in ((0, 0), (3, 1)):                                # tree 0: nodes 0, 1, 2 get rows 0 to 2, tree 1 rows 3 to 5
        six = edge_rows(target[b, :3].repeat(2, 1).clone())
        target[b, :3] = six[first:first + 3]
    if B > 2:
        for b in range(2, 50):                                       # the shifted rows at every node, in every order
            target[b, :3] = target[b, :3] + torch.tensor([[650.0, 0.0, -640.0], [0.0, -640.0, 650.0], [-640.0, 650.0, 0.0]],
                                                         device=DEV)[b % 3][:, None]
    tree["target"] = target.to(W.torch_dtype(dtype))
    tree["u_accept"] = tree["u_accept"] * 0.9
    ref = P.oracle_tree(P.to_np(tree["draft"]), P.to_np(tree["target"]), w.T, w.top_k, w.top_p, w.k_cap, w.expansion,
                        P.to_np(tree["u_sample"]), P.to_np(tree["u_accept"]), P.to_np(tree["u_resample"]), wor, wor)
    args = [tree["target"], w.T, w.expansion, t32(ref["q_idx"]), t32(ref["q_logit"]), t32(ref["q_count"]), t32(ref["cands"]),
            tree["u_accept"], tree["u_resample"]]
    out = tslt.verify_tree(*args, all_nodes=True, without_replacement=wor)
    path = tslt.verify_tree(*args, all_nodes=False, without_replacement=wor)
    torch.cuda.synchronize()
    print(P.compare_tree(out, ref, w.expansion, all_nodes=True, label=f"{dtype} {B}"), np.bincount(ref["verify"]["len"]))
    assert torch.equal(path["seq"], out["seq"]) and torch.equal(path["len"], out["len"])
