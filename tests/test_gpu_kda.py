"""GPU parity of KDA over packed rollout trees (Sec. 2.2, eq. chunk-state;
handoffs of Sec. 3.4) against the fp64 trajectory-wise oracle, through the
C ABI: o, S_final, dq, dk, dv, dg, dbeta and dS0_tree on small forests,
the edge-case forests of the linear-attention tests, seeded random forests
and plans of three and four rounds, and strong decays (every element); on the 64k-token agentic
microbatch at 16 heads of 128 (the benchmark's launch configuration), two
heads: o and dq of sampled rows from their trajectory prefixes, S_final of
sampled leaves, and dk, dv, dg, dbeta of rows near the end of leaf segments
(only the rest of their own trajectory depends on them) by reverse mode over
that suffix.  Tolerances: max relative error per tensor, 1e-4 for float32,
2e-2 for bf16 (q, k, v, dO rounded to bf16; g, beta float32)."""
import numpy as np
import pytest
import torch

from oracle.forest import SegTree
from oracle.kda import kda_forest, kda_recurrent
from tests.harness import TOL, max_rel, phys_index, record
from tests.test_kda_tables import CASES
from workloads.tensors import to_bf16_roundtrip
from workloads.trees import forest_for_config

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    from paper_2608_28158_amd import _lib
    _lib.lib()


def draw(Cn, H, d, n_trees, n_leaves, seed, bf16, strong=False):
    r = np.random.default_rng(seed)
    f32 = lambda a: a.astype(np.float32)
    q = f32(r.standard_normal((Cn, H, d)))
    k = r.standard_normal((Cn, H, d))
    k = f32(k / np.linalg.norm(k, axis=-1, keepdims=True))
    v = f32(r.standard_normal((Cn, H, d)))
    g = f32(r.uniform(-0.3, 0.0, (Cn, H, d)))
    if strong:
        # every fifth channel decays by up to 12 per row (about 96 over 16
        # rows), the next by up to 7.5 (about 56 +- 8 over 16 rows)
        g[:, :, 0::5] = r.uniform(-12.0, 0.0, g[:, :, 0::5].shape)
        g[:, :, 1::5] = r.uniform(-7.5, 0.0, g[:, :, 1::5].shape)
    beta = f32(r.uniform(0.05, 1.0, (Cn, H)))
    dO = f32(r.standard_normal((Cn, H, d)))
    S0 = f32(r.standard_normal((n_trees, H, d, d)) * 0.5)
    dSf = f32(r.standard_normal((n_leaves, H, d, d)) * 0.1)
    if bf16:
        q, k, v, dO = (to_bf16_roundtrip(a) for a in (q, k, v, dO))
    return q, k, v, g, beta, dO, S0, dSf


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 128)])
@pytest.mark.parametrize("label,parent,seg_len", CASES, ids=[c[0] for c in CASES])
def test_kda_matches_oracle(label, parent, seg_len, dtype, d):
    check_forest(label, parent, seg_len, dtype, d, 2)


@pytest.mark.parametrize("dtype,d", [("f32", 128), ("bf16", 64)])
def test_kda_other_dtype_and_width(dtype, d):
    label, parent, seg_len = CASES[2]
    check_forest(label, parent, seg_len, dtype, d, 2)


# A root of 70 rows with 18 leaves of 3..63 rows at 32 heads: the round of
# the leaves runs 17 state chains per head, 544 in all, enough for the state
# pass's 64-column slabs (the small forests above take its 32-column slabs).
STAR = ("star of 18 leaves", [-1] + [0] * 18, [70] + [3 + (9 * i + 5) % 61 for i in range(18)])


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 128)])
def test_kda_wide_state_slabs(dtype, d):
    run = check_forest(*STAR, dtype, d, 32)
    assert max(s1 - s0 for s0, s1, *_ in run.rounds) * 32 * (d // 64) >= 512


@pytest.mark.parametrize("dtype,d,H", [("f32", 64, 10), ("bf16", 128, 4)])
def test_kda_middle_state_slabs(dtype, d, H):
    """The star at head counts whose leaf round takes 32-column slabs: too many
    chains for all 16-column workgroups to run at once, too few for 64."""
    run = check_forest(*STAR, dtype, d, H)
    chains = max(s1 - s0 for s0, s1, *_ in run.rounds) * H
    assert chains * (d // 16) > (512 if d == 64 else 256) and chains * (d // 64) < 512


# The edge-case forests of the linear-attention parity tests (forks on,
# before and after chunk boundaries, replay across several ancestors, chains
# of one-row segments, a star, two trees, exact chunk multiples).
from tests.test_gpu_parity import EDGE_FORESTS  # noqa: E402
from tests.test_gpu_rounds import random_k3_forests  # noqa: E402


@pytest.mark.parametrize("label,parent,seg_len", EDGE_FORESTS, ids=[e[0] for e in EDGE_FORESTS])
def test_kda_edge_forests(label, parent, seg_len):
    check_forest(label, parent, seg_len, "f32", 64, 2)


# Seeded random forests whose plans have three or more rounds: sequences
# that start from a requested state and request states themselves.
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 128)])
def test_kda_random_k3_forests(dtype, d):
    for i, (parent, seg_len) in enumerate(random_k3_forests(31 + d, 3, 150)):
        run = check_forest(f"random K>=3 #{i}", parent, seg_len, dtype, d, 2)
        assert len(run.rounds) >= 3


# Channels whose log-decay falls by more than 60 over a 16-row block take the
# exact per-pair exponentials inside the block; the others factor through
# the block's first row.  Strong decays put both kinds, and channels close
# to the boundary, into every chunk.
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 128)])
def test_kda_strong_decays(dtype, d):
    label, parent, seg_len = CASES[2]
    check_forest(label + " strong decays", parent, seg_len, dtype, d, 2, strong=True)


def check_forest(label, parent, seg_len, dtype, d, H, strong=False):
    """Every element of o, S_final and the gradients against the oracle."""
    from paper_2608_28158_amd.kda import KdaRunner
    from paper_2608_28158_amd.plan import HartsPlan
    plan = HartsPlan(parent, seg_len, 64, heads=H)
    Cn = int(np.sum(seg_len))
    print(f"[gpu] kda {label} K={plan['n_rounds']} {dtype} d={d} H={H}", flush=True)
    q, k, v, g, beta, dO, S0, dSf = draw(Cn, H, d, plan["n_trees"], plan["n_leaves"], Cn + d, dtype == "bf16",
                                         strong)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    phys = phys_index(seg_len, plan["seg_row"])

    def dev(a, dt):
        out = np.empty_like(a)
        out[phys] = a
        return torch.from_numpy(out).to("cuda", dt).contiguous()

    run = KdaRunner(plan, H, d, tdt)
    scale = d ** -0.5
    o, Sf = run.forward(dev(q, tdt), dev(k, tdt), dev(v, tdt), dev(g, torch.float32), dev(beta, torch.float32),
                        torch.from_numpy(S0).cuda(), scale)
    grads = run.backward(dev(dO, tdt), torch.from_numpy(dSf).cuda())
    torch.cuda.synchronize()
    ref = kda_forest(parent, seg_len, q, k, v, g, beta, scale, S0, dO=dO, dS_final=dSf)
    host = lambda x: x.float().cpu().numpy()
    errs = {"o": max_rel(host(o)[phys], ref["o"]), "S_final": max_rel(host(Sf), ref["S_final"])}
    for n in ("dq", "dk", "dv", "dg", "dbeta"):
        errs[n] = max_rel(host(grads[n])[phys], ref[n])
    errs["dS0_tree"] = max_rel(host(grads["dS0_tree"]), ref["dS0_tree"])
    print(f"[gpu] kda {label} {dtype} d={d}: " + ", ".join(f"{a}={b:.2e}" for a, b in errs.items()), flush=True)
    record(f"kda {label} K={plan['n_rounds']} d={d} H={H}", dtype, errs)
    assert all(e <= TOL[dtype] for e in errs.values()), errs
    return run


def test_kda_64k_workload_sampled():
    from paper_2608_28158_amd.kda import KdaRunner
    from paper_2608_28158_amd.plan import HartsPlan
    f, _, cfg = forest_for_config(2)
    H, d = cfg["H"], cfg["d"]
    plan = HartsPlan(f.parent, f.seg_len, 64, heads=H)
    Cn = f.n_rows
    print(f"[gpu] kda 64k workload C={Cn} H={H} d={d} K={plan['n_rounds']}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(13)
    rnd = lambda *s: torch.randn(s, device="cuda", generator=gen)
    q = rnd(Cn, H, d).to(torch.bfloat16)
    k = rnd(Cn, H, d)
    k = (k / k.norm(dim=-1, keepdim=True)).to(torch.bfloat16)
    v = rnd(Cn, H, d).to(torch.bfloat16)
    g = -0.3 * torch.rand((Cn, H, d), device="cuda", generator=gen)
    beta = 0.05 + 0.95 * torch.rand((Cn, H), device="cuda", generator=gen)
    dO = rnd(Cn, H, d).to(torch.bfloat16)
    S0 = 0.5 * rnd(plan["n_trees"], H, d, d)
    dSf = 0.1 * rnd(plan["n_leaves"], H, d, d)
    run = KdaRunner(plan, H, d, torch.bfloat16)
    scale = d ** -0.5
    o, Sf = run.forward(q, k, v, g, beta, S0, scale)
    grads = run.backward(dO, dSf)
    torch.cuda.synchronize()
    r = np.random.default_rng(13)
    hs = torch.tensor(np.sort(r.choice(H, 2, replace=False))).cuda()
    phys = phys_index(f.seg_len, plan["seg_row"])
    host = lambda x: torch.from_numpy(x.index_select(1, hs).float().cpu().numpy()[phys]).double()
    Q, K, V, Gd, Bt, DO = (host(x) for x in (q, k, v, g, beta, dO))
    got = {n: host(grads[n]) for n in ("dq", "dk", "dv", "dg", "dbeta")}
    got["o"] = host(o)
    S0h = S0.index_select(1, hs).double().cpu()
    Sfh = Sf.index_select(1, hs).double().cpu()
    dSfh = dSf.index_select(1, hs).double().cpu()
    t = SegTree(f.parent, f.seg_len)
    ref, val = {n: [] for n in ("o", "dq", "dk", "dv", "dg", "dbeta", "S_final")}, None
    val = {n: [] for n in ref}
    leaves = [(li, u) for li, u in enumerate(t.leaves) if t.len[u] >= 8]
    for li, u in (leaves[int(i)] for i in r.choice(len(leaves), 5, replace=False)):
        rows = t.trajectory_rows(u)
        n = len(rows)
        cut = n - int(r.integers(2, min(48, t.len[u])))         # suffix inside the leaf segment
        with torch.no_grad():
            S = S0h[t.tree[u]]
            picks = set(int(x) for x in r.choice(cut, 4, replace=False))
            for j in range(cut):
                ot, S = kda_recurrent(Q[[rows[j]]], K[[rows[j]]], V[[rows[j]]], Gd[[rows[j]]], Bt[[rows[j]]],
                                      scale, S)
                if j in picks:                                   # o and dq from the prefix state
                    c = rows[j]
                    ref["o"].append(ot[0])
                    ref["dq"].append(scale * torch.einsum("hkv,hv->hk", S, DO[c]))
                    val["o"].append(got["o"][c])
                    val["dq"].append(got["dq"][c])
        suf = rows[cut:]
        xs = [x[suf].clone().requires_grad_(True) for x in (K, V, Gd, Bt)]
        os_, Sn = kda_recurrent(Q[suf], xs[0], xs[1], xs[2], xs[3], scale, S)
        ((os_ * DO[suf]).sum() + (Sn * dSfh[li]).sum()).backward()
        ref["S_final"].append(Sn.detach())
        val["S_final"].append(Sfh[li])
        for name, x in zip(("dk", "dv", "dg", "dbeta"), xs):
            ref[name].append(x.grad[0])
            val[name].append(got[name][suf[0]])
    errs = {n: max_rel(torch.stack(val[n]).numpy(), torch.stack(ref[n]).numpy()) for n in ref}
    print("[gpu] kda 64k workload: " + ", ".join(f"{a}={b:.2e}" for a, b in errs.items()), flush=True)
    record("kda 68k x 16 heads of 128 (sampled)", "bf16", errs)
    assert all(e <= TOL["bf16"] for e in errs.values()), errs


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_kda_backward_unaligned_rows(dtype):
    """v, dO, dv and the dv slots one element off a 16-byte boundary (element
    by element stores, row loads through registers): the same bits as aligned."""
    import ctypes as C
    from paper_2608_28158_amd import _lib
    from paper_2608_28158_amd.kda import KdaRunner, _p
    from paper_2608_28158_amd.plan import HartsPlan
    label, parent, seg_len = CASES[2]
    H, d = 2, 128
    plan = HartsPlan(parent, seg_len, 64, heads=H)
    Cn = int(np.sum(seg_len))
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    q, k, v, g, beta, dO, S0, dSf = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in draw(
        Cn, H, d, plan["n_trees"], plan["n_leaves"], 5, dtype == "bf16"))
    q, k, v, dO = (t.to(tdt) for t in (q, k, v, dO))

    def off(t):
        return torch.cat([t.new_zeros(1), t.reshape(-1)])[1:].view(t.shape)

    code = _lib.HARTS_BF16 if dtype == "bf16" else _lib.HARTS_F32
    scale, outs = d ** -0.5, []
    for shift in (lambda t: t, off):
        run = KdaRunner(plan, H, d, tdt)
        v_, dO_ = shift(v), shift(dO)
        run.forward(q, k, v_, g, beta, S0, scale)
        sz, st = run.sizes, run._stream()
        dbank = torch.zeros((plan["n_bank"], H, d, d), device="cuda")
        dS0 = torch.empty((sz.n_seq, H, d, d), device="cuda")
        # (rows with slots are not written: NaN stays)
        dq, dk, dg, dbeta = (torch.full_like(t, float("nan")) for t in (q, k, g, beta))
        dv = shift(torch.full_like(v, float("nan")))
        ns = max(sz.n_slots, 1)
        sq, sk, sg = (torch.full((ns, H, d), float("nan"), device="cuda") for _ in range(3))
        sv = shift(torch.full((ns, H, d), float("nan"), device="cuda"))
        sb = torch.full((ns, H), float("nan"), device="cuda")
        assert sz.n_slots > 0 and (dv.data_ptr() % 16 != 0) == (shift is off)
        for s0, s1, c0, c1, g0, g1 in reversed(run.rounds):
            _lib.check(run.L.harts_kda_bwd(
                _p(run.d_rows), _p(run.d_seq), _p(run.d_req), _p(run.d_slot), c0, c1 - c0, s0, s1 - s0, code, H, d,
                C.c_float(scale), _p(q), _p(k), _p(v_), _p(g), _p(beta), _p(dO_), _p(dSf), _p(dbank), _p(dS0),
                _p(run.ws), _p(dq), _p(dk), _p(dv), _p(dg), _p(dbeta), _p(sq), _p(sk), _p(sv), _p(sg), _p(sb), st),
                "harts_kda_bwd")
            _lib.check(run.L.harts_kda_bank_add(_p(run.d_group), g0, g1 - g0, _p(run.d_gseq), H * d * d, _p(dS0),
                                                _p(dbank), st), "harts_kda_bank_add")
        torch.cuda.synchronize()
        outs.append(dict(dq=dq, dk=dk, dv=dv.clone(), dg=dg, dbeta=dbeta, dbank=dbank, dS0=dS0, sq=sq, sk=sk,
                         sv=sv.clone(), sg=sg, sb=sb))
    for n, a in outs[0].items():
        b = outs[1][n]
        assert torch.equal(torch.isnan(a), torch.isnan(b)), n
        assert torch.equal(torch.nan_to_num(a), torch.nan_to_num(b)), n
    for out in outs:
        # rows replayed elsewhere go to the slots (all of them written), all others to the gradients
        for n in ("dq", "dk", "dv", "dg"):
            nan = torch.isnan(out[n])
            assert int(nan.any(-1).any(-1).sum()) == int(nan.all(-1).all(-1).sum()) == sz.n_multi, n
        assert int(torch.isnan(out["dbeta"]).all(-1).sum()) == sz.n_multi
        for n in ("dbank", "dS0", "sq", "sk", "sv", "sg", "sb"):
            assert torch.isfinite(out[n]).all(), n


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 128)])
def test_kda_non_finite_beta_leaves_earlier_queries(dtype, d, bad):
    """A query's gradient depends on no later row: with a beta that is not
    finite in a chunk's first 16 rows, the rows before it keep their dq (0
    times that beta must not reach them); so do a fork's other branch and the
    other head.  (In later 16-row blocks the products of whole blocks with
    L^-1 spread it over the block.)"""
    from paper_2608_28158_amd.kda import KdaRunner
    from paper_2608_28158_amd.plan import HartsPlan
    parent, seg_len, H = [-1, 0, 0], [100, 90, 70], 2
    plan = HartsPlan(parent, seg_len, 64, heads=H)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    q, k, v, g, beta, dO, S0, dSf = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in draw(
        260, H, d, 1, 2, 9, dtype == "bf16"))
    q, k, v, dO = (t.to(tdt) for t in (q, k, v, dO))
    run, outs = KdaRunner(plan, H, d, tdt), []
    row = int(plan["seg_row"][1]) + 41          # position 141 of its trajectory: chunk row 13
    for x in (None, bad):
        b = beta.clone()
        if x is not None:
            b[row, 1] = x
        run.forward(q, k, v, g, b, S0, d ** -0.5)
        outs.append(run.backward(dO, dSf)["dq"].clone())
    keep = torch.ones(260, dtype=torch.bool, device="cuda")
    keep[row:int(plan["seg_row"][1]) + 90] = False
    assert torch.equal(outs[0][:, 0], outs[1][:, 0]) and torch.equal(outs[0][keep], outs[1][keep])
    assert not torch.isfinite(outs[1][row + 1:row + 30, 1]).any()
