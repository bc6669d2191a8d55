"""The fp32 router and the fp32 grouped GEMMs at the edges of their tiles, K
slices and expert groups, through the C ABI, against fp64."""
import numpy as np
import pytest

from oracle import route as oroute

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_2607_17154_amd import ordermoe as om  # noqa: E402


@pytest.mark.parametrize("E", [1, 8, 17, 33, 65, 129, 256])
@pytest.mark.parametrize("T,d", [(1, 64), (33, 192), (16, 2048)])
def test_f32_router_logits_are_rounded_once(E, T, d):
    """Every logit is an fp64 sum rounded once, so a margin differs from the
    fp64 one by at most three roundings of 2^-24 (two logits and their
    difference), and tokens past that margin route alike."""
    rng = np.random.default_rng(E * 10 + T)
    k = min(E, 8)
    x = rng.standard_normal((T, d), dtype=np.float32)
    w = (rng.standard_normal((E, d)) * d ** -0.5).astype(np.float32)
    tabs = dict(t1_k=np.full((E, 1), -1, np.int32), t1_q=np.full((E, 1), np.inf, np.float32), t1_n=np.zeros(E, np.int32),
                srvmask=np.ones(E, np.int32), S=np.zeros((1, 1, E), np.float32))
    dev = {n: torch.from_numpy(v).cuda() for n, v in tabs.items()}
    L = om.make_layer(om.F32, d, E, k, 1, 1, torch.from_numpy(w).cuda(), dev, 0.25, 0.5)
    keep = torch.from_numpy(w).cuda()
    L.w_router = keep.data_ptr()
    out = om.alloc_route_out(T, k, 1, "cuda")
    ws = torch.empty(om.ordermoe_route_workspace_size(T, k, 1), dtype=torch.uint8, device="cuda")
    om.ordermoe_route_select(L, torch.from_numpy(x).cuda(), T, torch.zeros(T, dtype=torch.uint8, device="cuda"),
                             torch.zeros(T, dtype=torch.float32, device="cuda"), out, ws)
    torch.cuda.synchronize()
    idx, gate, margin, logits = oroute.route(x, w, k)
    tol = 3 * 2.0 ** -24 * max(np.abs(logits).max(), 1.0)
    got = out["margin"].cpu().numpy().astype(np.float64)
    if E > 1:
        assert np.max(np.abs(got - margin)) <= tol
    ok = margin > 2 * tol
    np.testing.assert_array_equal(out["idx"].cpu().numpy()[ok], idx[ok])
    # expf of a logit difference of at most ~10: a few ulp each over k terms
    np.testing.assert_allclose(out["w"].cpu().numpy()[ok], gate[ok], rtol=2e-6 + 10 * tol)


@pytest.mark.parametrize("rows,d,f,n_shared", [
    ([1], 64, 32, 0),                       # the smallest matrices, one row
    ([31, 33, 0, 64], 192, 96, 1),          # row tile edges, a K slice count that is no multiple of the slices
    ([65, 129], 320, 160, 2),               # shared K twice the routed K
    ([1100, 900], 512, 1056, 0),            # gate/up in 64-row tiles (1188), down in 32-row tiles
    ([8300, 8200], 256, 96, 0),             # both GEMMs in 64-row tiles (gate/up 777, down 1036)
])
def test_f32_forward_at_the_tile_edges(rows, d, f, n_shared):
    """Rows per expert as listed, one slot per token.  A sum of n fp32 products
    in any order is off by at most n 2^-24 of the sum of magnitudes; with random
    signs it grows as sqrt(n), and the bound below is 16 sqrt(n) 2^-24 of the
    output's scale through both projections."""
    rng = np.random.default_rng(len(rows) * 1000 + d)
    n, T = len(rows), int(sum(rows))
    ek = rng.permutation(np.repeat(np.arange(n), rows)).astype(np.int32)
    mk = lambda *s: torch.randn(*s, generator=g, device="cuda") * 0.05  # noqa: E731
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    x = torch.randn(T, d, generator=g, device="cuda")
    wt = torch.rand(T, 1, generator=g, device="cuda")
    loc = torch.from_numpy((rng.random(T) < 0.4).astype(np.uint8)).cuda()    # 0: the shared expert runs
    wg, wu, wd = mk(n, f, d), mk(n, f, d), mk(n, d, f)
    gu, dn = torch.empty((n, 2 * f, d), device="cuda"), torch.empty_like(wd)
    om.ordermoe_pack_gate_up(wg, wu, gu)
    om.ordermoe_pack_down(wd, dn)
    sgu = sdn = None
    if n_shared:
        sg, su, sd = mk(1, n_shared * f, d), mk(1, n_shared * f, d), mk(1, d, n_shared * f)
        sgu, sdn = torch.empty((1, 2 * n_shared * f, d), device="cuda"), torch.empty_like(sd)
        om.ordermoe_pack_gate_up(sg, su, sgu)
        om.ordermoe_pack_down(sd, sdn)
    ex = om.make_experts(om.F32, d, f, n, list(range(n)), gu, dn, n_shared, sgu, sdn)
    y = torch.empty((T, d), device="cuda")
    ro = torch.empty(n + 2, dtype=torch.int32, device="cuda")
    ws = torch.empty(om.ordermoe_forward_workspace_size(ex, T, 1), dtype=torch.uint8, device="cuda")
    ekd = torch.from_numpy(ek).cuda().view(T, 1)
    om.ordermoe_local_moe_forward(ex, x, T, 1, wt, ekd, torch.zeros((T, 1), dtype=torch.uint8, device="cuda"), loc, 0,
                                  y, ro, ws)
    torch.cuda.synchronize()

    def ffn(xs, a, b, c):
        h = xs @ a.double().t()
        return (h / (1 + torch.exp(-h)) * (xs @ b.double().t())) @ c.double().t()

    xd = x.double()
    want = torch.zeros_like(xd)
    for e in range(n):
        at = torch.nonzero(ekd[:, 0] == e).flatten()
        want[at] += wt[at].double() * ffn(xd[at], wg[e], wu[e], wd[e])
    if n_shared:
        at = torch.nonzero(loc == 0).flatten()
        want[at] += ffn(xd[at], sg[0], su[0], sd[0])
    err = ((y.double() - want).abs().amax() / want.abs().amax()).item()
    bound = 16 * max(d, max(n_shared, 1) * f) ** 0.5 * 2.0 ** -24
    print("rows %s d %d f %d: max err %.3g of the largest output (bound %.3g)" % (rows, d, f, err, bound), flush=True)
    assert err <= bound
    assert ro.cpu().tolist()[:n] == list(np.concatenate([[0], np.cumsum(rows)[:-1]]))


@pytest.mark.parametrize("E,T", [(1, 1), (8, 2048), (16, 129), (17, 1000), (33, 15), (64, 700), (65, 257), (128, 1041), (128, 128), (127, 129)])
def test_f32_similarity_at_the_partial_edges(E, T):
    """The fp32 similarity build at the edges of its partial sizes (16, 32, 64,
    128 experts) and chunks of 16 tokens.  A Gram entry sums at most 128 fp32
    products per partial before fp64 takes over: each addition rounds by
    2^-24 of a partial that is at most |h_i||h_j|, so a cosine is off by at most
    128 x 2^-24 and a little from the rounded logits."""
    from oracle import similarity as osim
    rng = np.random.default_rng(E * 7 + T)
    d, k = 192, min(E, 4)
    x = rng.standard_normal((T, d), dtype=np.float32)
    w = (rng.standard_normal((E, d)) * d ** -0.5).astype(np.float32)
    ws = torch.empty(om.ordermoe_similarity_workspace_size(T, d, E), dtype=torch.uint8, device="cuda")
    top1 = torch.empty(T, dtype=torch.int32, device="cuda")
    got = om.ordermoe_build_similarity(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), k, 0.7, 0.5, ws, top1=top1)
    H = osim.logit_matrix(x, w)                                   # [E][T]
    gram = H @ H.T
    n = np.sqrt(np.diag(gram))
    want = gram / np.outer(n, n)
    np.fill_diagonal(want, 1.0)
    assert np.max(np.abs(got["sim"] - want)) <= 130 * 2.0 ** -24
    # no ties within rounding in these draws except by chance: count them out
    idx, srt = oroute.topk(H.T, k)
    near = int(np.sum(oroute.margin(srt) < 1e-6)) if E > 1 else 0
    counts = np.bincount(idx.ravel(), minlength=E)
    assert np.abs(got["counts"] - counts).sum() <= 2 * near
    assert int(np.sum(top1.cpu().numpy() != idx[:, 0])) <= near
