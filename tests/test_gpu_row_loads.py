"""fp32 rows that the fp64 sweeps load in other ways than the rest: through the caches where an earlier launch of a large batch has
read them (sampled rows of chains, last rows of quick walks), by address in walks over short rows.  The same batch in parts that
stay below those lines, and every node of the same trees, have to give the same, with broken rows among them."""
import pytest
import torch

from paper_2512_16273_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("B,gamma,V", [(260, 1, 130001), (135, 3, 130001), (100, 5, 120001)])      # two rows a compute unit, one, shared ones
def test_sampled_rows_of_batches_beyond_the_cache(tslt, B, gamma, V):
    K = 16
    assert B * (gamma + 1) * V * 4 > 256 << 20 and (B // 2) * (gamma + 1) > 256
    w = W.scaled(W.WORKLOADS["chain_topk"], B=B, V=V, gamma=gamma, dtype="f32", top_k=K, k_cap=K, T=0.8)
    c = W.make_chain(w, 17, DEV)
    tr = tslt.truncate(c["draft"].view(B * gamma, V), w.T, K, 0.0, K, u=c["u_sample"].view(B * gamma, 1))
    target, u_accept = c["target"], c["u_accept"]
    target[0, gamma, 77] = float("nan")          # bonus rows that are reached
    target[1, gamma] += 650.0
    target[2, gamma] = -float("inf")
    target[3, gamma, ::3] = torch.finfo(torch.float32).min
    u_accept[:4] = 0.0
    args = [target, tr["idx"].view(B, gamma, K), tr["logit"].view(B, gamma, K), tr["count"].view(B, gamma), tr["token"].view(B, gamma),
            u_accept, c["u_resample"]]
    whole = tslt.verify(args[0], w.T, *args[1:])
    for i, j in ((0, B // 2), (B // 2, B)):
        part = [a[i:j].contiguous() for a in args]
        out = tslt.verify(part[0], w.T, *part[1:])
        torch.cuda.synchronize()
        for k, v in out.items():
            assert torch.equal(v.nan_to_num(nan=-7.0), whole[k][i:j].nan_to_num(nan=-7.0)) if v.is_floating_point() else torch.equal(v, whole[k][i:j]), k
    assert whole["accept_len"][:4].tolist() == [gamma] * 4 and whole["status"][:4].tolist() == [1, 0, 2, 0]
    assert (whole["tokens"][:4, gamma] < 0).tolist() == [True, False, True, False]


@pytest.mark.parametrize("B,expansion,V", [
    (64, (4, 2), 200001),                        # a quick walk, its last rows shared and cached
    (300, (2, 2), 110001),                       # the same, a workgroup to each
    (200, (2, 2), 9001), (200, (2, 2), 47999), (200, (2, 2), 48001),      # a walk from the root: by address, and streamed from 48000 on
])
def test_paths_against_every_node(tslt, B, expansion, V):
    K = 16
    w = W.scaled(W.WORKLOADS["tree"], B=B, V=V, expansion=expansion, top_k=K, k_cap=K, dtype="f32", without_replacement=False)
    tree = W.make_tree(w, 29, DEV)
    n = tree["target"].shape[1]
    sets = tslt.truncate(tree["draft"].reshape(-1, V), w.T, K, 0.0, K)
    n_int = sets["idx"].shape[0] // B
    g = torch.Generator().manual_seed(5)
    idx = sets["idx"].view(B, n_int, K)
    cand, node, width = [], 0, 1
    for k in expansion:
        pick = torch.randint(0, 6, (B, width, k), generator=g).to(DEV)
        cand.append(idx[:, node:node + width].gather(2, pick).reshape(B, -1))
        node, width = node + width, width * k
    rows = tree["target"].view(-1, V)
    rows[0, 77] = float("nan")
    rows[n] += 650.0
    rows[2 * n] = -float("inf")
    rows[3 * n, ::3] = torch.finfo(torch.float32).min
    args = (tree["target"], w.T, list(expansion), idx.contiguous(), sets["logit"].view(B, n_int, K), sets["count"].view(B, n_int),
            torch.cat(cand, 1).contiguous(), tree["u_accept"], tree["u_resample"])
    path = tslt.verify_tree(*args, all_nodes=False)
    every = tslt.verify_tree(*args, all_nodes=True)
    torch.cuda.synchronize()
    assert torch.equal(every["seq"], path["seq"]) and torch.equal(every["len"], path["len"])
    tested = ~path["ratio"].isnan()
    assert tested.any() and torch.allclose(every["ratio"][tested], path["ratio"][tested], rtol=1e-6, atol=0)
    assert (path["status"][:3] & 3).tolist() == [1, 0, 2] and (path["seq"][:3, 0] < 0).tolist() == [True, False, True]
