"""The native fast path of the Python binding against the step-by-step one: same outputs, same errors."""
import pytest
import torch

from paper_2512_16273_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


class Declines:
    """Stands for the native module and never takes a call."""
    def __getattr__(self, name):
        return lambda *a: None


class Recorder:
    """The native module, and which calls it has taken."""
    def __init__(self, native):
        self.native, self.taken = native, []

    def __getattr__(self, name):
        def call(*a):
            made = getattr(self.native, name)(*a)
            self.taken.append(made is not None)
            return made
        return call


def both(tslt, monkeypatch, call, taken=True):
    """The call's outcome by either path: its outputs, or the error's type and text.  `taken`: whether the native module takes it."""
    assert tslt._fast is not None
    native, got = Recorder(tslt._fast), []
    for fast in (native, Declines()):
        with monkeypatch.context() as m:
            m.setattr(tslt, "_fast", fast)
            try:
                got.append({k: None if v is None else v.clone() for k, v in call().items()})
            except Exception as e:  # noqa: BLE001  (whatever it is, it has to be the same)
                got.append((type(e), str(e)))
    assert native.taken and set(native.taken) == {taken}
    a, b = got
    if isinstance(a, tuple) or isinstance(b, tuple):
        assert a == b
        return a
    assert a.keys() == b.keys()
    for k in a:
        if a[k] is None:
            assert b[k] is None
        else:
            assert a[k].dtype == b[k].dtype and a[k].shape == b[k].shape
            assert torch.equal(a[k].view(torch.uint8), b[k].view(torch.uint8)), k
    return a


def unwritten(out):
    """Outputs as they are handed over, with what no call writes in them."""
    return {k: None if v is None else torch.full_like(v, 77) for k, v in out.items()}


def test_calls_by_either_path(tslt, monkeypatch):
    B, G, V, K = 3, 4, 4099, 16
    w = W.scaled(W.WORKLOADS["chain_topk"], B=B, V=V, gamma=G, dtype="bf16", top_k=K, k_cap=K)
    c = W.make_chain(w, 5, DEV)
    rows = c["draft"].reshape(B * G, V)
    wide = torch.zeros(B * G, V + 5, dtype=rows.dtype, device=DEV)
    wide[:, :V] = rows
    u = c["u_sample"].view(B * G, 1)
    made = tslt.truncate(rows, 0.7, K, 0.0, K, u=u)
    fresh = lambda: unwritten(made)  # noqa: E731
    def draft(z, top_k=K, u=u, out=None, taken=True):
        return both(tslt, monkeypatch, lambda: tslt.truncate(z, 0.7, top_k, 0.0, K, u=u, out=dict(out) if out else fresh()), taken)
    out = draft(rows)
    assert torch.equal(out["idx"], made["idx"]) and torch.equal(out["token"], made["token"])
    draft(wide[:, :V])                                                   # a stride
    draft(rows.view(B, G, V))
    draft(rows, out={**fresh(), "prob": None, "mass": None, "status": None, "slot": None})
    draft(rows, out={k: v for k, v in fresh().items() if k not in ("token", "slot")}, taken=False)
    assert torch.equal(draft(rows, top_k=(1 << 64) + K, taken=False)["idx"], made["idx"])      # (cut to 32 bits, as ctypes does)
    assert draft(rows, out={k: v for k, v in fresh().items() if k != "idx"}, taken=False)[0] is KeyError
    assert draft(rows, top_k=-1)[0] is tslt.TsltError
    for z, bad in ((rows, dict(u=u.cpu())), (rows, dict(u=u.double())), (wide.view(B, G, V + 5)[:, :, :V], {}), (rows.int(), {}), (rows.t(), {})):
        assert draft(z, taken=False, **bad)[0] is tslt.TsltError

    sets = (out["idx"].view(B, G, K), out["logit"].view(B, G, K), out["count"].view(B, G))
    ws = torch.empty(tslt.workspace_bytes(tslt.OP_VERIFY, B, G, V, K), dtype=torch.uint8, device=DEV)
    vf = tslt.verify(c["target"], 0.7, *sets, out["token"].view(B, G), c["u_accept"], c["u_resample"])
    def chain(target, s=sets, ws=ws, T=0.7, taken=True, phases=("both",), **o):
        def call():
            got = {**unwritten(vf), **o}
            for phase in phases:
                tslt.verify(target, T, *s, out["token"].view(B, G), c["u_accept"], c["u_resample"], out=got, workspace=ws, phase=phase)
            return got
        return both(tslt, monkeypatch, call, taken)
    for phases in (("both",), ("accept", "resample")):
        got = chain(c["target"], phases=phases)
        assert torch.equal(got["tokens"], vf["tokens"]) and torch.equal(got["accept_len"], vf["accept_len"])
        assert torch.equal(got["ratio"], vf["ratio"])
    chain(c["target"], ratio=None, beta=None, status=None)
    for bad in (dict(ws=ws[:64]), dict(T=0.0)):
        assert chain(c["target"], **bad)[0] is tslt.TsltError
    for target, bad in ((c["target"], dict(s=(sets[0].long(), *sets[1:]))), (c["target"], dict(s=(sets[0][:2], *sets[1:]))),
                        (c["target"][:, :, ::2], {}), (c["target"].view(-1, V), {})):
        assert chain(target, taken=False, **bad)[0] is tslt.TsltError

    pack = lambda i, pay="bf16", taken=True: both(tslt, monkeypatch, lambda: tslt.pack(i, out["logit"], out["count"], V, pay), taken)  # noqa: E731
    sent = pack(out["idx"])
    assert pack(out["idx"], "f32")[0] is tslt.TsltError and pack(out["idx"].t(), taken=False)[0] is tslt.TsltError
    pack(out["idx"][:0], taken=False)
    for rows_in, cap in ((B * G, K), (0, K), (B * G, 0)):
        both(tslt, monkeypatch, lambda: tslt.unpack(sent["words"], sent["row_offset"], rows_in, cap, V, "bf16"), rows_in > 0 and cap > 0)


def test_trees_by_either_path(tslt, monkeypatch):
    B, V, K, expansion = 2, 3001, 16, (2, 2)
    w = W.scaled(W.WORKLOADS["tree"], B=B, V=V, expansion=expansion, top_k=K, k_cap=K, dtype="f16", without_replacement=True)
    t = W.make_tree(w, 3, DEV)
    n = t["target"].shape[1]
    sets = tslt.truncate(t["draft"].reshape(-1, V), w.T, K, 0.0, K)
    n_int = sets["idx"].shape[0] // B
    idx = sets["idx"].view(B, n_int, K)
    cand = idx[:, :, :2].reshape(B, -1).contiguous()
    args = (idx.contiguous(), sets["logit"].view(B, n_int, K), sets["count"].view(B, n_int), cand, t["u_accept"], t["u_resample"])
    for every in (True, False):
        first = tslt.verify_tree(t["target"], w.T, expansion, *args, all_nodes=every, without_replacement=True)
        op = tslt.OP_VERIFY_TREE if every else tslt.OP_VERIFY_TREE_PATH
        ws = torch.empty(tslt.workspace_bytes(op, B, n, V, K), dtype=torch.uint8, device=DEV)
        call = lambda e, target=t["target"], ws=ws, taken=True: both(tslt, monkeypatch, lambda: tslt.verify_tree(  # noqa: E731
            target, w.T, e, *args, all_nodes=every, out=unwritten(first), workspace=ws, without_replacement=True), taken)
        for e in (expansion, list(expansion)):
            got = call(e)
            assert torch.equal(got["seq"], first["seq"]) and torch.equal(got["len"], first["len"])
            assert torch.equal(got["ratio"].nan_to_num(nan=-7.0), first["ratio"].nan_to_num(nan=-7.0))
        for bad in ((2, 99), [], (0, 2)):
            assert call(bad)[0] is tslt.TsltError
        assert call(expansion, ws=ws[:64])[0] is tslt.TsltError and call(expansion, t["target"][0], taken=False)[0] is tslt.TsltError
