"""The bf16 tiled forward where its work list can go wrong: row counts at the
edges of the 64-row units and of the tile heights, empty groups, shared tiles cut
into K pieces beside whole routed tiles, tiles of several heights over several
rounds of the grid.  Against fp64, through the C ABI."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_2607_17154_amd import ordermoe as om  # noqa: E402


@pytest.mark.parametrize("rows,d,f,n_shared,here", [
    ([129], 256, 128, 0, 0),                            # the smallest matrices: one column tile, 2 K tiles
    ([63, 64, 65, 1, 0, 128, 129], 256, 256, 0, 0),     # unit edges, an empty group between others
    ([192, 193, 255, 256, 257, 0], 512, 384, 1, 130),   # height edges, the last group empty, shared K = routed K
    ([0, 40, 300], 512, 256, 4, 321),                   # shared K four times the routed K, in whole tiles
    ([700, 20, 513], 2048, 1024, 2, 900),               # long K: shared down tiles in two K pieces
    ([5000, 300, 4000, 33], 512, 2048, 2, 3000),        # gate/up tiles of three heights over three rounds and a partial one, ragged ends
    ([20] * 64, 256, 128, 1, 1280),                     # as many groups as fit, all in 64-row tiles
])
def test_bf16_forward_at_the_tile_edges(rows, d, f, n_shared, here):
    """Rows per expert as listed, one slot per token; the first `here` tokens also
    run the shared expert.  Three roundings to bf16 (activation, row output, y),
    each 2^-9 relative to values of the output's scale, spread over the sums:
    8 x 2^-9 of the largest output bounds them with room; two runs are equal."""
    rng = np.random.default_rng(sum(rows) + d)
    n, T = len(rows), int(sum(rows))
    bf = torch.bfloat16
    g = torch.Generator(device="cuda")
    g.manual_seed(d + f)
    mk = lambda *s: (torch.randn(*s, generator=g, device="cuda") * s[-1] ** -0.5).to(bf)  # noqa: E731
    x = torch.randn(T, d, generator=g, device="cuda").to(bf)
    wt = torch.rand(T, 1, generator=g, device="cuda") + 0.25
    ek = torch.from_numpy(rng.permutation(np.repeat(np.arange(n), rows)).astype(np.int32)).cuda().view(T, 1)
    loc = torch.from_numpy((np.arange(T) >= here).astype(np.uint8)).cuda()      # 0: the shared expert runs
    wg, wu, wd = mk(n, f, d), mk(n, f, d), mk(n, d, f)
    gu, dn = torch.empty((n, 2 * f, d), dtype=bf, device="cuda"), torch.empty_like(wd)
    om.ordermoe_pack_gate_up(wg, wu, gu)
    om.ordermoe_pack_down(wd, dn)
    sgu = sdn = None
    if n_shared:
        sg, su, sd = mk(1, n_shared * f, d), mk(1, n_shared * f, d), mk(1, d, n_shared * f)
        sgu, sdn = torch.empty((1, 2 * n_shared * f, d), dtype=bf, device="cuda"), torch.empty_like(sd)
        om.ordermoe_pack_gate_up(sg, su, sgu)
        om.ordermoe_pack_down(sd, sdn)
    ex = om.make_experts(om.BF16, d, f, n, list(range(n)), gu, dn, n_shared, sgu, sdn)
    ro = torch.empty(n + 2, dtype=torch.int32, device="cuda")
    ws = torch.empty(om.ordermoe_forward_workspace_size(ex, T, 1), dtype=torch.uint8, device="cuda")
    m = torch.zeros((T, 1), dtype=torch.uint8, device="cuda")
    ys = []
    for _ in range(2):
        ws.fill_(255)                                   # nothing of an earlier call is relied on
        y = torch.empty((T, d), dtype=bf, device="cuda")
        om.ordermoe_local_moe_forward(ex, x, T, 1, wt, ek, m, loc, 0, y, ro, ws)
        torch.cuda.synchronize()
        ys.append(y)
    assert torch.equal(ys[0], ys[1])

    def ffn(xs, a, b, c):
        h = xs @ a.double().t().contiguous()
        return (h / (1 + torch.exp(-h)) * (xs @ b.double().t().contiguous())) @ c.double().t().contiguous()

    xd = x.double()
    want = torch.zeros_like(xd)
    for e in range(n):
        at = torch.nonzero(ek[:, 0] == e).flatten()
        if at.numel():
            want[at] += wt[at].double() * ffn(xd[at], wg[e], wu[e], wd[e])
    if n_shared:
        want[:here] += ffn(xd[:here], sg[0], su[0], sd[0])
    err = ((ys[0].double() - want).abs().amax() / want.abs().amax()).item()
    print("rows %s d %d f %d: max err %.3g of the largest output" % (rows[:8], d, f, err), flush=True)
    assert err <= 8 * 2.0 ** -9
    assert ro.cpu().tolist()[:n] == list(np.concatenate([[0], np.cumsum(rows)[:-1]]))


def test_a_workspace_without_partial_tiles_is_enough_for_a_decode_batch():
    """128 tokens of wide experts take the tiled GEMMs, and the thin ones in a
    workspace that only they fit.  The two add in another order: the bound is the
    three bf16 roundings' (above)."""
    n, E, T, k, d, f = 2, 8, 128, 2, 256, 12288
    bf = torch.bfloat16
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    mk = lambda *s: (torch.randn(*s, generator=g, device="cuda") * s[-1] ** -0.5).to(bf)  # noqa: E731
    gu, dn, x = mk(n, 2 * f, d), mk(n, d, f), torch.randn(T, d, generator=g, device="cuda").to(bf)
    w = torch.rand(T, k, generator=g, device="cuda")
    ek = torch.arange(k, dtype=torch.int32, device="cuda").repeat(T, 1)
    m = torch.zeros((T, k), dtype=torch.uint8, device="cuda")
    loc = torch.zeros(T, dtype=torch.uint8, device="cuda")
    ex = om.make_experts(om.BF16, d, f, E, list(range(n)), gu, dn, 0, None, None)
    need = om.ordermoe_forward_workspace_size(ex, T, k)
    ys = []
    for size in (need, need - (64 << 20)):
        y, ro = torch.empty((T, d), dtype=bf, device="cuda"), torch.empty(n + 2, dtype=torch.int32, device="cuda")
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        om.ordermoe_local_moe_forward(ex, x, T, k, w, ek, m, loc, 0, y, ro, ws)
        torch.cuda.synchronize()
        ys.append(y.double())
    assert (ys[0] - ys[1]).abs().amax() <= 8 * 2.0 ** -9 * ys[0].abs().amax()
    with pytest.raises(om.OrderMoEError) as ei:
        om.ordermoe_local_moe_forward(ex, x, T, k, w, ek, m, loc, 0, y, ro, ws[:-1])
    assert ei.value.code == om.EWORKSPACE


@pytest.mark.parametrize("dtype,n,d,f", [("bf16", 1, 256, 128), ("bf16", 3, 768, 640), ("f32", 2, 72, 96),
                                         ("f32", 1, 512, 32)])
def test_packed_weights_are_the_documented_layout(dtype, n, d, f):
    """Every packed element equals the source element that the layout names
    (K steps that are no multiple of a wave's, one and several experts)."""
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(d * f)
    wg, wu, wd = (torch.randn(n, *s, generator=g, device="cuda").to(dt) for s in ((f, d), (f, d), (d, f)))
    gu, dn = torch.full((n, 2 * f, d), 7.0, dtype=dt, device="cuda"), torch.full((n, d, f), 7.0, dtype=dt, device="cuda")
    om.ordermoe_pack_gate_up(wg, wu, gu)
    om.ordermoe_pack_down(wd, dn)
    want = torch.stack([wg.view(n, f // 32, 32, d), wu.view(n, f // 32, 32, d)], 2).reshape(n, 2 * f, d)
    blk = lambda t, N, K: t.reshape(n, N // 256, 256, K // 64, 64).transpose(2, 3).reshape(n, N, K)  # noqa: E731
    if dtype == "bf16":
        assert torch.equal(gu, blk(want, 2 * f, d)) and torch.equal(dn, blk(wd, d, f))
    else:
        assert torch.equal(gu, want) and torch.equal(dn, wd)
