"""Rejections that leave no residual: rows with a few allowed tokens, all of them in the received set with q_hat equal to p,
and a draft token outside it (reported, and rejected).  max(0, p - q_hat) is zero but for rounding, and what is drawn is a
token of p itself, never none."""
import numpy as np
import pytest
import torch

from oracle import tslt_oracle as O
from tests import _parity as P

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}


def masked_rows(n, V, allowed, dtype, T, seed):
    """Target rows [n, V] with `allowed` tokens each, their sets (width 4), a token outside each set and the token at
    which the cumulative p passes u, with u well inside its bucket."""
    rng = np.random.default_rng(seed)
    z = torch.full((n, V), -float("inf"))
    ids = np.stack([rng.choice(V - 1, allowed, replace=False) for _ in range(n)])
    vals = torch.from_numpy(rng.normal(0.0, 2.0, (n, allowed)).astype(np.float32))
    z.scatter_(1, torch.from_numpy(ids), vals)
    z = z.to(DTYPES[dtype])
    rows = z.float().numpy()
    q_idx = np.full((n, 4), -1, np.int32)
    q_logit = np.full((n, 4), -np.inf, np.float32)
    tr = O.truncate(rows, T, allowed, 0.0, 4)
    q_idx[:], q_logit[:] = tr["idx"], tr["logit"]
    outside = np.full(n, V - 1, np.int32)
    u = rng.random(n).astype(np.float32)
    want = np.empty(n, np.int64)
    for r in range(n):
        p = O.dense_probs(rows[r], T)
        want[r], margin = O.inverse_cdf(p, u[r])
        while margin < 1e-9:
            u[r] = np.float32(rng.random())
            want[r], margin = O.inverse_cdf(p, u[r])
    return z, q_idx, q_logit, np.full(n, allowed, np.int32), outside, u, want


@pytest.mark.parametrize("dtype,T,B", [("f32", 0.9, 200), ("bf16", 0.9, 200), ("bf16", 0.1, 200), ("f16", 0.9, 200),
                                       ("f32", 0.9, 300), ("bf16", 0.9, 300), ("f16", 0.9, 300)])
@pytest.mark.parametrize("allowed", [1, 2, 3])
def test_chain_without_residual(tslt, dtype, T, B, allowed):
    V = 2003
    z, q_idx, q_logit, q_count, outside, u, want = masked_rows(B, V, allowed, dtype, T, 100 * allowed + B)
    target = torch.stack([z, z], 1).contiguous().to(DEV)                     # [B, 2, V]
    u_res = torch.from_numpy(np.stack([u, u], 1)).to(DEV)
    args = [target, T, torch.from_numpy(q_idx[:, None]).contiguous().to(DEV), torch.from_numpy(q_logit[:, None]).contiguous().to(DEV),
            torch.from_numpy(q_count[:, None]).contiguous().to(DEV), torch.from_numpy(outside[:, None]).contiguous().to(DEV),
            torch.full((B, 1), 0.5, device=DEV), u_res]
    out = tslt.verify(*args)
    ws = torch.empty(tslt.workspace_bytes(tslt.OP_VERIFY, B, 1, V, 4), dtype=torch.uint8, device=DEV)
    halves = tslt.verify(*args, workspace=ws, phase="accept", out={k: torch.empty_like(v) for k, v in out.items()})
    tslt.verify(*args, out=halves, workspace=ws, phase="resample")
    torch.cuda.synchronize()
    for o in (out, halves):
        assert np.all(P.to_np(o["accept_len"]) == 0) and np.all(P.to_np(o["status"]) == 4)
        got = P.to_np(o["tokens"])[:, 0]
        wrong = np.nonzero(got != want)[0]
        assert wrong.size == 0, (wrong.size, got[wrong[:5]], want[wrong[:5]])


@pytest.mark.parametrize("dtype,B", [("f32", 30), ("bf16", 30), ("f16", 30), ("f32", 180), ("bf16", 180), ("f16", 180)])
@pytest.mark.parametrize("allowed,rule", [(1, False), (2, True), (3, False)])
def test_tree_without_residual(tslt, dtype, B, allowed, rule):
    """The root rejects a token outside its set, then, with nothing left to subtract from, tests its second candidate
    against p as it was: the set's first token, whose ratio is 1.  Its child rejects two such tokens and draws."""
    V, T = 1203, 0.9
    z, q_idx, q_logit, q_count, outside, u, want = masked_rows(B, V, allowed, dtype, T, 7 * allowed + B)
    n, n_int = 7, 3                                                           # expansion (2, 2)
    target = z[:, None].expand(B, n, V).contiguous().to(DEV)
    sets = [torch.from_numpy(np.repeat(a[:, None], n_int, 1)).contiguous().to(DEV) for a in (q_idx, q_logit, q_count)]
    cands = np.repeat(outside[:, None], n - 1, 1)
    cands[:, 1] = q_idx[:, 0]
    u_res = torch.from_numpy(np.repeat(u[:, None], n, 1)).contiguous().to(DEV)
    args = [target, T, (2, 2), *sets, torch.from_numpy(cands).to(DEV), torch.full((B, n - 1), 0.5, device=DEV), u_res]
    for all_nodes in (True, False):
        out = tslt.verify_tree(*args, all_nodes=all_nodes, without_replacement=rule)
        torch.cuda.synchronize()
        seq, ratio = P.to_np(out["seq"]), P.to_np(out["ratio"])
        assert np.all(P.to_np(out["len"]) == 2) and np.all(P.to_np(out["status"]) == 4)
        assert np.array_equal(seq[:, 0], q_idx[:, 0]) and np.array_equal(seq[:, 1], want), (all_nodes, seq[:5], want[:5])
        assert np.all(ratio[:, 0] == -1.0)
        np.testing.assert_allclose(ratio[:, 1], 1.0, rtol=1e-6)


@pytest.mark.parametrize("dtype,B", [("f32", 120), ("bf16", 120), ("f16", 120), ("f32", 300), ("f16", 300)])
def test_draw_at_the_start_of_the_residual(tslt, dtype, B):
    """A uniform of 0 takes the first token with residual mass, also where the run before it holds nothing but a token at
    which q_hat is above p: what rounding leaves of that run's mass is not drawn from."""
    V, T = 9001, 0.9
    rng = np.random.default_rng(B)
    ids = np.stack([rng.integers(lo, lo + 900, B) for lo in (0, 2048, 4100, 7000)], 1)           # runs of their own
    z = torch.full((B, V), -float("inf"))
    z.scatter_(1, torch.from_numpy(ids), torch.from_numpy(rng.normal(0.0, 1.0, (B, 4)).astype(np.float32)))
    z = z.to(DTYPES[dtype])
    p = np.stack([O.dense_probs(r, T) for r in z.float().numpy()])
    # the set: the first two tokens, each with more mass than p has there; the last two are the residual
    q_logit = np.log(np.take_along_axis(p, ids[:, :2], 1)).astype(np.float32)
    q_idx = np.where(q_logit[:, :1] >= q_logit[:, 1:], ids[:, :2], ids[:, 1::-1]).astype(np.int32)
    q_logit = -np.sort(-q_logit, 1)
    target = torch.stack([z, z], 1).contiguous().to(DEV)
    args = [target, T, torch.from_numpy(q_idx[:, None]).contiguous().to(DEV), torch.from_numpy(q_logit[:, None]).contiguous().to(DEV),
            torch.full((B, 1), 2, dtype=torch.int32, device=DEV), torch.full((B, 1), V - 1, dtype=torch.int32, device=DEV),
            torch.full((B, 1), 0.5, device=DEV), torch.zeros(B, 2, device=DEV)]
    out = tslt.verify(*args)
    torch.cuda.synchronize()
    assert np.array_equal(P.to_np(out["tokens"])[:, 0], ids[:, 2])
