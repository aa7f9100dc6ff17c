"""Edges of the kernels' launch rules: sizes at which a kernel variant, a tile or a remainder begins, each against the
oracle or against the library's other form of the same computation."""
import sys

import numpy as np
import pytest

import oracle
import synth
from gpu_support import GATE_TOL, backward_error_bounds, grouped_gap_bound, higham_bound, to_dev, upload

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2602_05711_amd as P  # noqa: E402
from paper_2602_05711_amd import binding as B  # noqa: E402


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def _random_routing(w, seed=3):
    """Distinct random experts per (token, head) and gates that sum to one."""
    rng = np.random.default_rng(seed)
    idx = np.argsort(rng.random((w.T, w.H, w.N)), axis=-1)[..., :w.K].astype(np.int32)
    g = rng.random((w.T, w.H, w.K)).astype(np.float32)
    return np.ascontiguousarray(idx), g / g.sum(-1, keepdims=True)


# (T, d, H, K, dtype): the routed sum with four v rows in flight (at most 4096 rows of 1 KiB over the tokens' v rows) and
# just past it; slots that four do not divide, more than 64 of them; column splits of one, two and four; whole and
# partial rows.
ACC_CASES = [(1024, 512, 2, 13, "bf16"), (1025, 2048, 2, 3, "bf16"), (600, 1024, 5, 13, "bf16"),
             (1100, 200, 1, 3, "bf16"), (300, 2048, 3, 23, "bf16"), (1024, 2048, 2, 2, "bf16"),
             (4096, 64, 2, 1, "bf16"), (1030, 264, 2, 9, "f32"), (600, 512, 1, 17, "f32")]


@pytest.mark.parametrize("case", ACC_CASES, ids=[str(c) for c in ACC_CASES])
def test_routed_sum_rows_in_flight(case):
    T, d, H, K, dtype = case
    say(f"[routed sum] {case}")
    w = synth.Workload("acc", T=T, d=d, n_rows=9, n_cols=11, d_key=8, H=H, K=K, dtype=dtype)
    inp = synth.make_inputs(w)
    f = {k: synth.as_f32(v) for k, v in inp.items()}
    idx, g = _random_routing(w)
    dsc = oracle.desc(w)
    perm = oracle.schedule(dsc, idx)[0]
    ref = oracle.expert_forward(dsc, f["x"], f["u"], f["v"], idx, g.astype(np.float64))
    dev, D = upload(inp), B.make_desc(w)
    y = torch.full((T, d), float("nan"), device="cuda")
    y_tc = torch.full((T, d), float("nan"), device="cuda")
    P.omnimoe_expert_forward(D, dev["x"], dev["u"], dev["v"], to_dev(idx), to_dev(g), to_dev(perm), y)
    P.omnimoe_expert_forward_token_centric(D, dev["x"], dev["u"], dev["v"], to_dev(idx), to_dev(g), y_tc)
    torch.cuda.synchronize()
    # Stored values are exact in fp32 and all sums are fp32, so each result lies within Higham's bound of the exact one:
    # the dot products' error (gamma_d sum |x u|, through act' <= 1.13 and the gate) and the slot sum's. A relative bound
    # on the row does not hold: with one slot whose x . u nearly cancels, all of the row carries that dot's error.
    gap = np.abs(y.cpu().numpy().astype(np.float64) - ref)
    assert np.all(gap <= grouped_gap_bound(f, idx, g, d, dsc.act))
    # every form sums a token's slots one after another, so the bits agree
    assert np.array_equal(y.cpu().numpy().view(np.uint8), y_tc.cpu().numpy().view(np.uint8))


# (T, d, n_rows, n_cols, H, K, dtype): row pieces of 256 elements, whole and partial, one to sixteen per lane; segments longer
# than the 64 positions of a wave's window and of every remainder; one and two experts per wave (from 32768 rows on).
BWD_CASES = [(300, 200, 2, 3, 1, 4, "bf16"), (131, 256, 3, 4, 2, 5, "bf16"), (90, 512, 5, 7, 1, 3, "bf16"),
             (77, 1024, 6, 6, 2, 3, "bf16"), (40, 1032, 4, 9, 1, 7, "bf16"), (67, 2048, 5, 8, 1, 6, "bf16"),
             (33, 4096, 4, 4, 1, 5, "bf16"), (150, 264, 3, 3, 1, 2, "f32"), (50, 2048, 5, 5, 2, 3, "f32"),
             (700, 64, 190, 190, 4, 13, "bf16")]


@pytest.mark.parametrize("case", BWD_CASES, ids=[str(c) for c in BWD_CASES])
def test_expert_backward_segments(case):
    T, d, nr, nc, H, K, dtype = case
    say(f"[expert backward] {case}")
    w = synth.Workload("bwd", T=T, d=d, n_rows=nr, n_cols=nc, d_key=8, H=H, K=K, dtype=dtype)
    inp = synth.make_inputs(w)
    f = {k: synth.as_f32(v) for k, v in inp.items()}
    if w.N <= 4096:
        idx, g = _random_routing(w)
    else:
        rng = np.random.default_rng(5)
        idx = np.stack([rng.choice(w.N, K, replace=False) for _ in range(T * H)]).reshape(T, H, K).astype(np.int32)
        g = rng.random((T, H, K)).astype(np.float32)
    dsc = oracle.desc(w)
    perm, act, off, _ = oracle.schedule(dsc, idx)
    dy = np.random.default_rng(11).standard_normal((T, d)).astype(np.float32)
    ref = oracle.expert_backward(dsc, f["x"], f["u"], f["v"], idx, g.astype(np.float64), dy.astype(np.float64))
    bnd = backward_error_bounds(f["x"], f["u"], f["v"], idx, g, dy, np.vectorize(lambda z: oracle.act(0, z)),
                                np.vectorize(lambda z: oracle.act_grad(0, z)))
    A, n = min(w.M, w.N), len(act)
    out = {k: torch.full(shape, float("nan"), device="cuda") for k, shape in
           [("dx", (T, d)), ("du", (A, d)), ("dv", (A, d)), ("dgates", (T, H, K)), ("dscores", (T, H, K))]}
    offd = torch.full((A + 1,), -1, dtype=torch.int32, device="cuda")
    offd[:n + 1] = to_dev(off)
    dev = upload(inp)
    P.omnimoe_expert_backward(B.make_desc(w), dev["x"], dev["u"], dev["v"], to_dev(idx), to_dev(g), to_dev(perm), offd,
                              torch.tensor([n], dtype=torch.int32, device="cuda"), to_dev(dy), out["dx"], out["du"],
                              out["dv"], out["dgates"], out["dscores"])
    torch.cuda.synchronize()
    for k, rk in (("dx", "dx"), ("du", "du_rows"), ("dv", "dv_rows"), ("dgates", "dgates"), ("dscores", "dscores")):
        got = out[k].cpu().numpy()[:n if k in ("du", "dv") else None]
        err = np.abs(got.astype(np.float64) - ref[rk])
        say(f"  {k}: max err / bound {(err / (2 * bnd[k] + 1e-30)).max():.2f}")
        assert np.all(err <= 2 * bnd[k] + 1e-30), k
    # rows past the active experts are not written
    assert torch.isnan(out["du"][n:]).all() and torch.isnan(out["dv"][n:]).all()


# (tasks of each expert in id order, d, dtype): segments of a piece of tasks (16 here, 32 from 32769 tasks on), one more, several,
# that begin on a piece's edge and off it, one after the other and at the end; one and two experts per wave; every token
# with one expert.
PIECE_CASES = [((16, 17, 1, 33, 64, 2, 130), 200, "bf16"), ((300,), 2048, "bf16"), ((50, 16, 14, 20), 4096, "bf16"),
               ((3, 3, 3, 3, 3, 47, 1, 1, 15, 16, 17, 18), 1032, "f32"), ((15,), 64, "bf16"), ((17, 15, 32, 16), 64, "f32"),
               ((1,) * 36000 + (2000, 1, 1999), 16, "bf16")]


@pytest.mark.parametrize("case", PIECE_CASES, ids=[f"{len(c[0])} experts, {c[1:]}" for c in PIECE_CASES])
def test_expert_backward_pieces(case):
    counts, d, dtype = case
    T, nr = sum(counts), 192 if len(counts) > 1000 else 4
    say(f"[expert backward, pieces] {len(counts)} experts, {T} tokens, d {d} {dtype}")
    w = synth.Workload("piece", T=T, d=d, n_rows=nr, n_cols=nr, d_key=8, H=1, K=1, dtype=dtype)
    inp = synth.make_inputs(w)
    f = {k: synth.as_f32(v) for k, v in inp.items()}
    rng = np.random.default_rng(T)
    idx = rng.permutation(np.repeat(np.arange(len(counts)), counts)).reshape(T, 1, 1).astype(np.int32)
    g = rng.random((T, 1, 1)).astype(np.float32)
    dsc = oracle.desc(w)
    perm, act, off, _ = oracle.schedule(dsc, idx)
    dy = rng.standard_normal((T, d)).astype(np.float32)
    ref = oracle.expert_backward(dsc, f["x"], f["u"], f["v"], idx, g.astype(np.float64), dy.astype(np.float64))
    bnd = backward_error_bounds(f["x"], f["u"], f["v"], idx, g, dy, np.vectorize(lambda z: oracle.act(0, z)),
                                np.vectorize(lambda z: oracle.act_grad(0, z)))
    A, n = min(w.M, w.N), len(act)
    offd = torch.full((A + 1,), -1, dtype=torch.int32, device="cuda")
    offd[:n + 1] = to_dev(off)
    dev, D = upload(inp), B.make_desc(w)
    ws = P.workspace(D, B.STAGE_EXPERT_BACKWARD)
    outs = []
    for fill in (0, 255):  # the workspace's contents do not matter
        ws.fill_(fill)
        out = {k: torch.full(shape, float("nan"), device="cuda") for k, shape in
               [("dx", (T, d)), ("du", (A, d)), ("dv", (A, d)), ("dgates", (T, 1, 1)), ("dscores", (T, 1, 1))]}
        P.omnimoe_expert_backward(D, dev["x"], dev["u"], dev["v"], to_dev(idx), to_dev(g), to_dev(perm), offd,
                                  torch.tensor([n], dtype=torch.int32, device="cuda"), to_dev(dy), out["dx"], out["du"],
                                  out["dv"], out["dgates"], out["dscores"], ws=ws)
        torch.cuda.synchronize()
        assert torch.isnan(out["du"][n:]).all() and torch.isnan(out["dv"][n:]).all()
        outs.append({k: v.cpu().numpy()[:n if k in ("du", "dv") else None] for k, v in out.items()})
    for k, rk in (("dx", "dx"), ("du", "du_rows"), ("dv", "dv_rows"), ("dgates", "dgates"), ("dscores", "dscores")):
        err = np.abs(outs[0][k].astype(np.float64) - ref[rk])
        say(f"  {k}: max err / bound {(err / (2 * bnd[k] + 1e-30)).max():.2f}")
        assert np.all(err <= 2 * bnd[k] + 1e-30), k
        assert np.array_equal(outs[0][k].view(np.uint8), outs[1][k].view(np.uint8)), k


def test_expert_backward_time_under_skew():
    """One expert with a quarter of all tasks: its tasks are shared out, so the call takes a few times what it takes with
    the tasks spread evenly (1.5 times here) and not the time of 16384 tasks one after another (30 times)."""
    w = synth.Workload("hot", T=16384, d=512, n_rows=64, n_cols=64, d_key=8, H=1, K=4)
    rng = np.random.default_rng(1)
    even = torch.from_numpy((rng.permutation(w.M) % (w.N - 4) + 4).astype(np.int32).reshape(w.T, 1, 4))
    hot = even.clone()
    hot[:, 0, 0] = 1
    dev = {k: torch.randn(s, device="cuda").to(torch.bfloat16) for k, s in
           (("x", (w.T, w.d)), ("u", (w.N, w.d)), ("v", (w.N, w.d)))}
    dy, D = torch.randn((w.T, w.d), device="cuda"), B.make_desc(w)
    g = torch.full((w.T, 1, 4), 0.25, device="cuda")
    ws = P.workspace(D, B.STAGE_EXPERT_BACKWARD)
    out = [torch.empty(s, device="cuda") for s in ((w.T, w.d), (w.N, w.d), (w.N, w.d), (w.T, 1, 4), (w.T, 1, 4))]
    ms = {}
    for name, idx in (("even", even), ("hot", hot)):
        idx = idx.cuda()
        perm, act, off, na = (torch.empty(n, dtype=torch.int32, device="cuda") for n in (w.M, w.N, w.N + 1, 1))
        P.omnimoe_schedule(D, idx, perm, act, off, na)
        runs = []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            P.omnimoe_expert_backward(D, dev["x"], dev["u"], dev["v"], idx, g, perm, off, na, dy, *out, ws=ws)
            b.record()
            torch.cuda.synchronize()
            runs.append(a.elapsed_time(b))
        ms[name] = sorted(runs)[3]
    say(f"[expert backward] even {ms['even']:.3f} ms, one expert with a quarter of the tasks {ms['hot']:.3f} ms")
    assert ms["hot"] <= 6 * ms["even"]


# (T, d, d_key, n_rows, n_cols, H, K, query, dtype): blocks of 1, 2, 8 and 16 slots with partial ones, more than 64 picks per
# token, a sub-key with hundreds of picks, tables of one row and of 4096; d_key pieces of 256 elements, whole and
# partial, one to sixteen of them (combinations that eight divides and that it does not).
ROUTE_BWD_CASES = [(1, 16, 8, 3, 4, 1, 5, "split", "bf16"), (70, 64, 24, 5, 6, 2, 1, "split", "bf16"),
                   (300, 2048, 1024, 6, 9, 2, 13, "split", "bf16"), (90, 1544, 768, 8, 7, 1, 17, "split", "bf16"),
                   (129, 264, 264, 12, 3, 3, 30, "shared", "bf16"), (33, 256, 64, 4096, 2, 1, 64, "split", "bf16"),
                   (700, 128, 64, 1, 40, 5, 2, "split", "f32"), (50, 2048, 2048, 9, 9, 1, 8, "shared", "f32"),
                   (17, 4096, 4096, 5, 5, 2, 20, "shared", "bf16"), (5000, 64, 32, 16, 16, 4, 16, "split", "bf16")]


@pytest.mark.parametrize("case", ROUTE_BWD_CASES, ids=[str(c) for c in ROUTE_BWD_CASES])
def test_route_backward_picks(case):
    T, d, dk, nr, nc, H, K, query, dtype = case
    say(f"[route backward] {case}")
    w = synth.Workload("rbwd", T=T, d=d, n_rows=nr, n_cols=nc, d_key=dk, H=H, K=K, query_mode=query, dtype=dtype)
    rng = np.random.default_rng(K + T)
    idx = np.stack([rng.choice(w.N, K, replace=False) for _ in range(T * H)]).reshape(T, H, K).astype(np.int32)
    kr, kc = synth.make_keys(w)
    x = synth.make_x(w)
    fx, fr, fc = synth.as_f32(x), synth.as_f32(kr), synth.as_f32(kc)
    ds = rng.standard_normal((T, H, K)).astype(np.float32)
    dx0 = rng.standard_normal((T, d)).astype(np.float32)
    dsc = oracle.desc(w)
    ref = oracle.route_backward(dsc, fx, fr, fc, idx, ds, dx=dx0)
    absb = oracle.route_backward(dsc, np.abs(fx), np.abs(fr), np.abs(fc), idx, np.abs(ds), dx=np.abs(dx0))
    outs = []
    for _ in range(2):
        dx = to_dev(dx0.copy())
        dkr = torch.full((H, nr, dk), float("nan"), device="cuda")
        dkc = torch.full((H, nc, dk), float("nan"), device="cuda")
        P.omnimoe_route_backward(B.make_desc(w), to_dev(x), to_dev(kr), to_dev(kc), to_dev(idx), to_dev(ds), dx, dkr, dkc)
        torch.cuda.synchronize()
        outs.append([v.cpu().numpy() for v in (dx, dkr, dkc)])
    # Every element is a fp32 sum of n terms (and of products): gamma_n times the sum of their absolute values (Higham),
    # whatever the order, with two more roundings for the block sums of the weights and the products.
    u = 2.0 ** -24
    hd = np.arange(H)[None, :, None]
    n_r = np.bincount((hd * nr + idx // nc).ravel(), minlength=H * nr).reshape(H, nr, 1) + 3
    n_c = np.bincount((hd * nc + idx % nc).ravel(), minlength=H * nc).reshape(H, nc, 1) + 3
    for k, got, rv, ab, n in zip(("dx", "dkeys_row", "dkeys_col"), outs[0], ref, absb, (2 * H * K + 3, n_r, n_c)):
        bound = (n * u / (1 - n * u)) * ab + 1e-30
        err = np.abs(got.astype(np.float64) - rv)
        say(f"  {k}: max err / bound {(err / bound).max():.3f}")
        assert np.all(err <= bound), k
    for x0, x1 in zip(*outs):
        assert np.array_equal(x0.view(np.uint8), x1.view(np.uint8))


def test_route_backward_one_half_at_a_time():
    """2^30 tasks, whose picks of both halves 32 bits do not number: each half in a round of its own. Every token picks every
    cell of the grid; the weights are whole numbers, zero but for a few tokens, so that every sum is exact."""
    T, n, dk = 1 << 18, 64, 8
    w = synth.Workload("half", T=T, d=2 * dk, n_rows=n, n_cols=n, d_key=dk, H=1, K=n * n)
    say(f"[route backward] {w.M} tasks")
    rng = np.random.default_rng(3)
    x = torch.from_numpy(rng.integers(-4, 5, (T, 2 * dk)).astype(np.float32)).to(torch.bfloat16)
    kr, kc = (torch.from_numpy(rng.integers(-4, 5, (1, n, dk)).astype(np.float32)).to(torch.bfloat16) for _ in range(2))
    order = torch.from_numpy(rng.permutation(n * n).astype(np.int32))
    idx = order.cuda().repeat(T, 1).view(T, 1, n * n)
    slot = torch.from_numpy(rng.integers(-3, 4, n * n).astype(np.float32))
    tok = torch.zeros(T)
    tok[torch.tensor([0, 1, 77777, T // 2, T - 2, T - 1])] = torch.tensor([1.0, -2.0, 3.0, 1.0, 2.0, -1.0])
    ds = (tok.cuda()[:, None] * slot.cuda()[None]).view(T, 1, n * n)
    dx = torch.zeros((T, 2 * dk), device="cuda")
    dkr, dkc = (torch.full((1, n, dk), float("nan"), device="cuda") for _ in range(2))
    P.omnimoe_route_backward(B.make_desc(w), x.cuda(), kr.cuda(), kc.cuda(), idx, ds, dx, dkr, dkc)
    torch.cuda.synchronize()
    for half, got, keys in ((order.long() // n, dkr, kr), (order.long() % n, dkc, kc)):
        q = 0 if got is dkr else dk
        per_key = torch.zeros(n).scatter_add_(0, half, slot)
        assert torch.equal(got[0].cpu(), per_key[:, None] * (tok @ x[:, q:q + dk].float())[None])
        want = tok[:, None] * (per_key @ keys[0].float())[None]
        assert torch.equal(dx[:, q:q + dk].cpu(), want)


# (T, d, d_key, n_rows, n_cols, H, query): fp32 logits on tiles of 64 x 64 with k steps of 32: one k step and several, whole and
# partial, tokens and keys at a tile's edge and past it.
F32_LOGIT_CASES = [(1, 16, 8, 1, 3, 1, "split"), (64, 64, 32, 32, 64, 2, "split"), (65, 80, 40, 64, 65, 1, "split"),
                   (130, 264, 264, 21, 43, 3, "shared"), (63, 1024, 512, 63, 5, 1, "split")]


@pytest.mark.parametrize("case", F32_LOGIT_CASES, ids=[str(c) for c in F32_LOGIT_CASES])
def test_f32_logits(case):
    T, d, dk, nr, nc, H, query = case
    say(f"[fp32 logits] {case}")
    w = synth.Workload("f32l", T=T, d=d, n_rows=nr, n_cols=nc, d_key=dk, H=H, K=1, query_mode=query, dtype="f32")
    x, (kr, kc) = synth.make_x(w), synth.make_keys(w)
    hs = torch.full((T, H, nr + nc), float("nan"), device="cuda")
    idx = torch.empty((T, H, 1), dtype=torch.int32, device="cuda")
    g = torch.empty((T, H, 1), device="cuda")
    P.omnimoe_route(B.make_desc(w), to_dev(x), to_dev(kr), to_dev(kc), idx, g, half_scores=hs)
    torch.cuda.synchronize()
    c0 = dk if query == "split" else 0
    for keys, xq, got in ((kr, x[:, :dk], hs[..., :nr]), (kc, x[:, c0:c0 + dk], hs[..., nr:])):
        ref = np.einsum("tm,hjm->thj", xq.astype(np.float64), keys.astype(np.float64))
        assert np.all(np.abs(got.cpu().numpy() - ref) <= higham_bound(xq, keys) + 1e-30)


# (T, d, n_rows, n_cols, H, K, dtype, act, one kernel?): the expert stage by tokens in the layer: both sides of its line (400
# tokens, or six per slot), slots that four waves do not share evenly and more than one batch of 256, rows of one to
# eight chunks a lane, whole and partial; sums of one part, of four and of sixteen (up to 1023 tokens of sixteen slots or
# 64); short rows with one wave per token from 2048 tokens on; tables past 128 MiB on
# both sides of six tasks per expert.
STAGE_CASES = [(48, 64, 16, 17, 1, 8, "f32", "gelu", True), (47, 64, 16, 17, 1, 8, "f32", "gelu", False),
               (400, 520, 12, 13, 3, 13, "f32", "silu", True), (399, 512, 30, 40, 3, 27, "bf16", "gelu", False),
               (401, 1024, 20, 21, 2, 150, "bf16", "gelu", True), (2048, 200, 10, 10, 2, 5, "bf16", "gelu", True),
               (2047, 200, 10, 10, 2, 5, "bf16", "silu", True), (500, 2048, 9, 10, 5, 3, "bf16", "gelu", True),
               (430, 4096, 5, 6, 1, 3, "f32", "gelu", True), (450, 2056, 7, 9, 2, 3, "bf16", "gelu", True),
               (500, 512, 20, 21, 4, 16, "bf16", "gelu", True), (1023, 520, 12, 13, 2, 8, "f32", "silu", True),
               (1024, 520, 12, 13, 2, 8, "f32", "silu", True), (100, 1024, 20, 21, 1, 16, "f32", "gelu", True),
               (600, 4088, 128, 129, 2, 82, "bf16", "gelu", True), (608, 4088, 128, 129, 2, 82, "bf16", "gelu", False)]


@pytest.mark.parametrize("case", STAGE_CASES, ids=[str(c) for c in STAGE_CASES])
def test_token_stage_layer(case):
    T, d, nr, nc, H, K, dtype, act, one = case
    say(f"[token stage] {case}")
    w = synth.Workload("stage", T=T, d=d, n_rows=nr, n_cols=nc, d_key=16, H=H, K=K, dtype=dtype, act=act)
    inp = synth.make_inputs(w)
    dev, D = upload(inp), B.make_desc(w)
    assert bool(B.omnimoe_layer_kernels(D) & B.PATH_TOKEN_STAGE) == one
    y = torch.full((T, d), float("nan"), device="cuda")
    idx = torch.empty((T, H, K), dtype=torch.int32, device="cuda")
    g = torch.empty((T, H, K), device="cuda")
    P.omnimoe_layer_forward(D, dev["x"], dev["keys_row"], dev["keys_col"], dev["u"], dev["v"], y, idx, g)
    # the stage on its own on the layer's routing: the dots and the sum in kernels of their own
    perm, act_, off, na = (torch.empty(n, dtype=torch.int32, device="cuda")
                           for n in (w.M, min(w.M, w.N), min(w.M, w.N) + 1, 1))
    P.omnimoe_schedule(D, idx, perm, act_, off, na)
    y_ef = torch.full((T, d), float("nan"), device="cuda")
    P.omnimoe_expert_forward(D, dev["x"], dev["u"], dev["v"], idx, g, perm, y_ef)
    torch.cuda.synchronize()
    f = {k: synth.as_f32(v) for k, v in inp.items()}
    gi, gg = idx.cpu().numpy(), g.cpu().numpy()
    dsc = oracle.desc(w)
    ref = oracle.expert_forward(dsc, f["x"], f["u"], f["v"], gi, gg.astype(np.float64))
    # fp32 sums of exact products: Higham's bounds through the activation (as for the routed sum above)
    got = y.cpu().numpy()
    assert np.all(np.abs(got.astype(np.float64) - ref) <= grouped_gap_bound(f, gi, gg, d, dsc.act))
    # the same dots and the same partial sums, with a workgroup per token or without
    assert np.array_equal(got.view(np.uint8), y_ef.cpu().numpy().view(np.uint8))


# (T, d, n_rows, n_cols, H, K, dtype, act, group size, swept): the expert stage in sweeps in the layer (at least 512 tokens, two
# tasks per expert, rows of 2, 4 and 8 KiB): tokens that a workgroup's share does not divide, one walk and more than one
# per lane group, four waves and sixteen in step, slots that sixteen and 64 do not divide, fewer than sixteen; the dots in
# two passes (layers that one pass would take past 64 MiB); with groups (the sum alone), and just below the line.
SWEEP_CASES = [(512, 1024, 8, 9, 2, 7, "bf16", "gelu", 1, "stage"), (515, 2048, 30, 31, 2, 21, "bf16", "silu", 1, "stage"),
               (2051, 1024, 40, 41, 3, 23, "bf16", "gelu", 1, "stage"), (1030, 2048, 7, 9, 1, 16, "f32", "gelu", 1, "stage"),
               (517, 4096, 6, 7, 2, 17, "bf16", "gelu", 1, "stage"), (4200, 512, 9, 9, 1, 1, "f32", "gelu", 1, "stage"),
               (9000, 1024, 5, 6, 2, 3, "bf16", "gelu", 1, "stage"), (2600, 1024, 40, 41, 4, 128, "bf16", "gelu", 1, "stage"),
               (3501, 512, 40, 41, 4, 128, "f32", "silu", 1, "stage"), (2400, 1024, 40, 41, 4, 128, "bf16", "gelu", 64, "sum"), (700, 1024, 20, 21, 2, 80, "bf16", "gelu", 16, "sum"),
               (2100, 1024, 50, 60, 2, 33, "bf16", "silu", 64, "sum"), (511, 1024, 8, 9, 2, 7, "bf16", "gelu", 1, ""),
               (512, 1024, 50, 60, 1, 11, "bf16", "gelu", 1, "")]


@pytest.mark.parametrize("case", SWEEP_CASES, ids=[str(c) for c in SWEEP_CASES])
def test_sweep_layer(case):
    T, d, nr, nc, H, K, dtype, act, Bg, swept = case
    say(f"[sweep] {case}")
    w = synth.Workload("sweep", T=T, d=d, n_rows=nr, n_cols=nc, d_key=16, H=H, K=K, dtype=dtype, act=act,
                       group_size=Bg)
    inp = synth.make_inputs(w)
    dev, D = upload(inp), B.make_desc(w)
    assert B.omnimoe_layer_kernels(D) & (B.PATH_SWEEP_STAGE | B.PATH_SWEEP_SUM) == {
        "stage": B.PATH_SWEEP_STAGE, "sum": B.PATH_SWEEP_SUM, "": 0}[swept]
    ws = P.workspace(D, B.STAGE_LAYER)
    ys = []
    for fill in (0, 255):  # the workspace's contents do not matter
        ws.fill_(fill)
        y = torch.full((T, d), float("nan"), device="cuda")
        idx = torch.empty((T, H, K), dtype=torch.int32, device="cuda")
        g = torch.empty((T, H, K), device="cuda")
        P.omnimoe_layer_forward(D, dev["x"], dev["keys_row"], dev["keys_col"], dev["u"], dev["v"], y, idx, g, ws=ws)
        torch.cuda.synchronize()
        ys.append(y.cpu().numpy())
    f = {k: synth.as_f32(v) for k, v in inp.items()}
    gi, gg = idx.cpu().numpy(), g.cpu().numpy()
    dsc = oracle.desc(w)
    ref = oracle.expert_forward(dsc, f["x"], f["u"], f["v"], gi, gg.astype(np.float64))
    bound = grouped_gap_bound(f, gi, gg, d, dsc.act)  # fp32 sums in any order: Higham's bounds
    ratio = np.abs(ys[0].astype(np.float64) - ref) / bound
    say(f"  max err / bound {ratio.max():.3f}")
    assert ratio.max() <= 1.0
    assert np.array_equal(ys[0].view(np.uint8), ys[1].view(np.uint8))


# (T, H, K): slots that sixteen does not divide; the loads past a token's last task repeat a row that must not be added again
SWEEP_TAIL_CASES = [(512, 2, 7), (520, 3, 13), (2048, 2, 9)]


@pytest.mark.parametrize("case", SWEEP_TAIL_CASES, ids=[str(c) for c in SWEEP_TAIL_CASES])
def test_sweep_tail_adds_nothing(case):
    T, H, K = case
    say(f"[sweep tail] {case}")
    w = synth.Workload("tail", T=T, d=1024, n_rows=7, n_cols=9, d_key=16, H=H, K=K)
    dev, D = upload(synth.make_inputs(w)), B.make_desc(w)
    assert B.omnimoe_layer_kernels(D) & B.PATH_SWEEP_STAGE
    # an overflowed value of every expert in a column of its own: the sum there is infinite where the token picked that
    # expert and finite elsewhere (zero times such a row would be NaN)
    e = torch.arange(w.N, device="cuda")
    dev["v"].view(torch.bfloat16)[e, e] = float("inf")
    y = torch.full((T, 1024), float("nan"), device="cuda")
    idx = torch.empty((T, H, K), dtype=torch.int32, device="cuda")
    g = torch.empty((T, H, K), device="cuda")
    P.omnimoe_layer_forward(D, dev["x"], dev["keys_row"], dev["keys_col"], dev["u"], dev["v"], y, idx, g)
    torch.cuda.synchronize()
    picked = torch.zeros((T, 1024), dtype=torch.bool, device="cuda").scatter_(1, idx.view(T, -1).long(), True)
    assert not torch.isnan(y).any()
    assert torch.equal(torch.isinf(y), picked)


# (T, n, d, H, K): the selection that forms the dot with a workgroup per row (up to 512 rows) and with a wave per row past it; picks
# that four waves share evenly, unevenly, and fewer picks than waves.
TEAM_CASES = [(64, 256, 512, 4, 16), (512, 256, 512, 1, 13), (513, 256, 512, 1, 13), (128, 512, 1024, 3, 64),
              (300, 256, 2048, 1, 3), (65, 1024, 512, 4, 1), (256, 256, 4096, 2, 30)]


@pytest.mark.parametrize("case", TEAM_CASES, ids=[str(c) for c in TEAM_CASES])
def test_selection_dot_team(case):
    T, n, d, H, K = case
    say(f"[selection dot] {case}")
    w = synth.Workload("team", T=T, d=d, n_rows=n, n_cols=n, d_key=64, H=H, K=K)
    inp = synth.make_inputs(w)
    dev, D = upload(inp), B.make_desc(w)
    assert B.omnimoe_layer_path(D) & B.PATH_SELECT_DOT
    y = torch.full((T, d), float("nan"), device="cuda")
    idx = torch.empty((T, H, K), dtype=torch.int32, device="cuda")
    g = torch.empty((T, H, K), device="cuda")
    P.omnimoe_layer_forward(D, dev["x"], dev["keys_row"], dev["keys_col"], dev["u"], dev["v"], y, idx, g)
    # the stage on its own (the separate dot kernel) on the layer's routing: the same bits
    perm = torch.empty(w.M, dtype=torch.int32, device="cuda")
    cap = min(w.M, w.N)
    act = torch.empty(cap, dtype=torch.int32, device="cuda")
    off = torch.empty(cap + 1, dtype=torch.int32, device="cuda")
    na = torch.empty(1, dtype=torch.int32, device="cuda")
    P.omnimoe_schedule(D, idx, perm, act, off, na)
    y2 = torch.full((T, d), float("nan"), device="cuda")
    P.omnimoe_expert_forward(D, dev["x"], dev["u"], dev["v"], idx, g, perm, y2)
    idx2, g2 = torch.empty_like(idx), torch.empty_like(g)
    P.omnimoe_route(D, dev["x"], dev["keys_row"], dev["keys_col"], idx2, g2)
    torch.cuda.synchronize()
    assert torch.equal(idx, idx2) and torch.equal(g, g2)
    assert np.array_equal(y.cpu().numpy().view(np.uint8), y2.cpu().numpy().view(np.uint8))


# (T, d, d_key, n_rows, n_cols, H): bf16 logits on 64 x 64, 128 x 64, 128 x 128 and 256 x 256 tiles: one k step, fewer than the
# ring holds and more; tokens and keys at a tile's edge and past it, an uneven pair of halves.
TILE_CASES = [(65, 128, 64, 64, 65, 1), (70, 256, 128, 3, 130, 2), (129, 1024, 512, 100, 7, 3), (200, 2048, 1024, 1024, 1000, 8),
              (257, 256, 128, 512, 512, 8), (500, 512, 256, 1024, 1024, 8), (513, 128, 64, 700, 1025, 9),
              (769, 128, 64, 2048, 2047, 4)]


@pytest.mark.parametrize("case", TILE_CASES, ids=[str(c) for c in TILE_CASES])
def test_bf16_logit_tiles(case):
    T, d, dk, nr, nc, H = case
    say(f"[bf16 logits] {case}")
    w = synth.Workload("tiles", T=T, d=d, n_rows=nr, n_cols=nc, d_key=dk, H=H, K=1)
    x, (kr, kc) = synth.make_x(w), synth.make_keys(w)
    hs = torch.full((T, H, nr + nc), float("nan"), device="cuda")
    idx = torch.empty((T, H, 1), dtype=torch.int32, device="cuda")
    g = torch.empty((T, H, 1), device="cuda")
    P.omnimoe_route(B.make_desc(w), to_dev(x), to_dev(kr), to_dev(kc), idx, g, half_scores=hs)
    torch.cuda.synchronize()
    hs = hs.cpu().numpy()
    # Higham's bound on a sample of the tokens: the first, the last and those around each tile edge
    rows = sorted({t for e in range(0, T + 256, 64) for t in (e - 1, e) if 0 <= t < T} | {T - 1})
    fx, fr, fc = synth.as_f32(x)[rows], synth.as_f32(kr), synth.as_f32(kc)
    for keys, xq, got in ((fr, fx[:, :dk], hs[rows][..., :nr]), (fc, fx[:, dk:2 * dk], hs[rows][..., nr:])):
        ref = np.matmul(xq.astype(np.float64)[None], keys.astype(np.float64).transpose(0, 2, 1)).transpose(1, 0, 2)
        bound = np.matmul(np.abs(xq).astype(np.float64)[None],
                          np.abs(keys).astype(np.float64).transpose(0, 2, 1)).transpose(1, 0, 2)
        gamma = dk * 2.0 ** -23 / (1 - dk * 2.0 ** -23)
        assert np.all(np.abs(got - ref) <= 2 * gamma * bound + 1e-30)
    assert np.isfinite(hs).all()


# (T, d, d_ff): the accumulating projection on each tile, on top of what y holds; the gate and up projections with the step
# between them in one kernel on 128 x 128 and 256 x 256 tiles, features and tokens past a tile's edge
MLP_TILE_CASES = [(66, 192, 64), (300, 704, 704), (700, 1024, 512), (1500, 512, 1024), (1501, 128, 2056),
                  (3001, 64, 2056), (3072, 192, 2048), (65, 64, 16384)]


@pytest.mark.parametrize("case", MLP_TILE_CASES, ids=[str(c) for c in MLP_TILE_CASES])
def test_shared_mlp_tiles(case):
    T, d, d_ff = case
    say(f"[shared mlp] {case}")
    w = synth.Workload("mlpt", T=T, d=d, n_rows=2, n_cols=2, d_key=8, H=1, K=1)
    x, (gu, dn) = synth.make_x(w), synth.make_mlp_weights(w, d_ff)
    y0 = np.random.default_rng(3).standard_normal((T, d)).astype(np.float32)
    y = to_dev(y0.copy())
    P.omnimoe_shared_mlp(B.make_desc(w), d_ff, to_dev(x), to_dev(gu), to_dev(dn), y)
    torch.cuda.synchronize()
    fx, fg, fd = (synth.as_f32(v).astype(np.float64) for v in (x, gu, dn))
    h = fx @ fg.T
    act = h[:, :d_ff] / (1 + np.exp(-h[:, :d_ff])) * h[:, d_ff:]
    # silu(g) u rounded to bf16 (2^-8 relative at most, with the fp32 products before it) times w_down
    bound = (2.0 ** -8) * (np.abs(act) @ np.abs(fd).T) + 1e-5 * (np.abs(fx) @ np.abs(fg).T).max() + 1e-6
    assert np.all(np.abs(y.cpu().numpy() - (y0 + act @ fd.T)) <= bound)


# (n_rows, n_cols, K, kind): more than 64 picks per row: halves of one and two sorting waves at their edges; the order by score
# buckets and, where a bucket is too full (coarse scores, one far outlier, every score alike), by merged runs or a sort.
LARGE_K_CASES = [(256, 257, 512, "normal"), (512, 512, 513, "normal"), (300, 100, 65, "normal"), (513, 40, 700, "normal"),
                 (320, 320, 2048, "normal"), (17, 16, 200, "normal"), (320, 320, 4096, "coarse"),
                 (512, 256, 400, "coarse"), (320, 320, 1024, "outlier"), (64, 80, 300, "outlier"),
                 (320, 320, 512, "alike"), (256, 256, 3000, "alike"), (512, 511, 4096, "mixed")]


@pytest.mark.parametrize("case", LARGE_K_CASES, ids=[str(c) for c in LARGE_K_CASES])
def test_select_large_orders(case):
    nr, nc, K, kind = case
    say(f"[select] {case}")
    rng = np.random.default_rng(nr + nc + K)
    T = 7
    hs = rng.standard_normal((T, 1, nr + nc)).astype(np.float32)
    if kind in ("coarse", "mixed"):
        hs[::2 if kind == "mixed" else 1] = np.round(hs[::2 if kind == "mixed" else 1] * 4) / 4
    if kind == "outlier":
        hs[:, 0, 3], hs[:, 0, nr + 5] = 64.0, 100.0  # (sums stay exact in double)
    if kind == "alike":
        hs[:] = 0.25
    w = synth.Workload("sel", T=T, d=16, n_rows=nr, n_cols=nc, d_key=8, H=1, K=K, dtype="f32")
    idx = torch.empty((T, 1, K), dtype=torch.int32, device="cuda")
    g = torch.empty((T, 1, K), dtype=torch.float32, device="cuda")
    P.omnimoe_select(B.make_desc(w), to_dev(hs), idx, g)
    torch.cuda.synchronize()
    ri, _, rg, inexact = oracle.select_f32(oracle.desc(w), hs, oracle.BRUTE)
    assert inexact == 0 and np.array_equal(idx.cpu().numpy(), ri)
    np.testing.assert_allclose(g.cpu().numpy(), rg, rtol=GATE_TOL, atol=1e-7)


# (n_rows, n_cols, K, kind, n): the order by score buckets at its edges: n equal scores around the fullest bucket that is ranked;
# as many keys as the buckets take and one more; masked columns (a large negative value, or minus infinity) among the
# picks, some of them and most; infinite and NaN logits at the top.
BUCKET_CASES = [(1, 400, 300, "ties", 47), (1, 400, 300, "ties", 48), (1, 400, 300, "ties", 49), (1, 400, 400, "ties", 200),
                (1, 3000, 2500, "ties", 49), (64, 64, 2048, "normal", 0), (64, 64, 2049, "normal", 0),
                (64, 64, 4096, "normal", 0), (20, 300, 4096, "masked", 150), (20, 300, 4096, "masked", 290),
                (20, 300, 4096, "-inf", 150), (20, 300, 300, "-inf", 290), (20, 300, 500, "+inf", 1),
                (320, 320, 4096, "+inf", 3), (40, 300, 700, "nan", 2)]


@pytest.mark.parametrize("case", BUCKET_CASES, ids=[str(c) for c in BUCKET_CASES])
def test_select_large_buckets(case):
    nr, nc, K, kind, n = case
    say(f"[select, buckets] {case}")
    rng = np.random.default_rng(nr + nc + K + n)
    T = 5
    hs = rng.standard_normal((T, 1, nr + nc)).astype(np.float32)
    if kind == "ties":  # evenly spread scores, n of them alike (in shuffled places, among the best K)
        hs[..., :nr] = 0.0
        for t in range(T):
            c = np.linspace(4.0, -4.0, nc).astype(np.float32)
            c[50:50 + n] = c[50]
            hs[t, 0, nr:] = rng.permutation(c)
    if kind == "masked":
        hs = np.round(hs * 1024) / 1024  # (sums with the mask stay exact in double)
    put = {"masked": -2.0 ** 30, "-inf": -np.inf, "+inf": np.inf, "nan": np.nan}.get(kind)
    if put is not None:
        for t in range(T):
            hs[t, 0, nr + rng.permutation(nc)[:n]] = put
    w = synth.Workload("sel", T=T, d=16, n_rows=nr, n_cols=nc, d_key=8, H=1, K=K, dtype="f32")
    idx = torch.empty((T, 1, K), dtype=torch.int32, device="cuda")
    g = torch.empty((T, 1, K), dtype=torch.float32, device="cuda")
    P.omnimoe_select(B.make_desc(w), to_dev(hs), idx, g)
    torch.cuda.synchronize()
    got, gg = idx.cpu().numpy()[:, 0], g.cpu().numpy()[:, 0]
    # scores as sums of two fp32 in double (exact here), NaN above plus infinity; ties to the lower id
    s = (hs[:, 0, :nr, None].astype(np.float64) + hs[:, 0, None, nr:].astype(np.float64)).reshape(T, -1)
    for t in range(T):
        key = np.where(np.isnan(s[t]), np.inf, s[t])
        order = np.lexsort((np.arange(nr * nc), -key, ~np.isnan(s[t])))[:K]
        # (scores of minus infinity: any of them, since the order among rows and columns is not that among their sums)
        m = int(np.isfinite(s[t][order]).sum()) if kind == "-inf" else K
        assert np.array_equal(got[t][:m], order[:m]), t
        assert len(set(got[t])) == K and np.all(s[t][got[t][m:]] == -np.inf)
        if kind not in ("+inf", "nan"):
            e = np.exp(s[t][order] - s[t][order[0]])
            np.testing.assert_allclose(gg[t], e / e.sum(), rtol=GATE_TOL, atol=1e-7)
