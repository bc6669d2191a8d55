"""Which GEMMs a bf16 batch takes and how its work list cuts the tiles, read from
what the row kernels publish in the workspace, and the outputs of those paths
against fp64, through the C ABI."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_2607_17154_amd import ordermoe as om  # noqa: E402

from ._pipeline import PARTIAL_TILES, published_plans  # noqa: E402

BF = torch.bfloat16


class Layer:
    """A layer of E experts, the first n of them here, one slot of k in use: rows[e]
    tokens run expert e, the first `here` tokens also the shared expert, the
    remaining slots run on another server."""

    def __init__(self, rows, d, f, n_shared, here, T, E, k):
        g = torch.Generator(device="cuda")
        g.manual_seed(d + f)
        mk = lambda *s: (torch.randn(*s, generator=g, device="cuda") * s[-1] ** -0.5).to(BF)  # noqa: E731
        n = len(rows)
        assert sum(rows) <= T and n <= E
        self.rows, self.here, self.T, self.k, self.d, self.n = rows, here, T, k, d, n
        self.x, self.w = torch.randn(T, d, generator=g, device="cuda").to(BF), torch.rand(T, k, generator=g, device="cuda") + 0.25
        ek, m = np.full((T, k), E - 1, np.int32), np.ones((T, k), np.uint8)
        at = np.random.default_rng(T + n).permutation(T)[:sum(rows)]
        ek[at, 0], m[at, 0] = np.repeat(np.arange(n), rows), 0
        self.ek, self.m = torch.from_numpy(ek).cuda(), torch.from_numpy(m).cuda()
        self.loc = torch.from_numpy((np.arange(T) >= here).astype(np.uint8)).cuda()
        self.routed, self.shared = (mk(n, f, d), mk(n, f, d), mk(n, d, f)), None
        gu, dn = self._pack(*self.routed)
        sgu = sdn = None
        if n_shared:
            self.shared = mk(1, n_shared * f, d), mk(1, n_shared * f, d), mk(1, d, n_shared * f)
            sgu, sdn = self._pack(*self.shared)
        self.keep = gu, dn, sgu, sdn
        self.ex = om.make_experts(om.BF16, d, f, E, list(range(n)), gu, dn, n_shared, sgu, sdn)
        self.need = om.ordermoe_forward_workspace_size(self.ex, T, k)

    @staticmethod
    def _pack(wg, wu, wd):
        n, f, d = wg.shape
        gu, dn = torch.empty((n, 2 * f, d), dtype=BF, device="cuda"), torch.empty_like(wd)
        om.ordermoe_pack_gate_up(wg, wu, gu)
        om.ordermoe_pack_down(wd, dn)
        return gu, dn

    def run(self, size=None):
        """(y, workspace) of one call; nothing in the workspace is relied on."""
        ws = torch.full((self.need if size is None else size,), 255, dtype=torch.uint8, device="cuda")
        y = torch.empty((self.T, self.d), dtype=BF, device="cuda")
        ro = torch.empty(self.n + 2, dtype=torch.int32, device="cuda")
        om.ordermoe_local_moe_forward(self.ex, self.x, self.T, self.k, self.w, self.ek, self.m, self.loc, 0, y, ro, ws)
        torch.cuda.synchronize()
        assert ro.cpu().tolist()[:self.n] == list(np.concatenate([[0], np.cumsum(self.rows)[:-1]]))
        return y, ws

    def error(self, y):
        """Largest error against fp64 over the largest output.  Three roundings to
        bf16 (activation, row output, y), each 2^-9 relative to values of the
        output's scale: at most 8 x 2^-9 with room."""
        def ffn(x, wg, wu, wd):
            h = x @ wg.double().t().contiguous()
            return (h / (1 + torch.exp(-h)) * (x @ wu.double().t().contiguous())) @ wd.double().t().contiguous()
        x, want = self.x.double(), torch.zeros((self.T, self.d), dtype=torch.float64, device="cuda")
        for e in range(self.n):
            at = torch.nonzero((self.ek[:, 0] == e) & (self.m[:, 0] == 0)).flatten()
            if at.numel():
                want[at] += self.w[at, :1].double() * ffn(x[at], *(t[e] for t in self.routed))
        if self.shared and self.here:
            want[:self.here] += ffn(x[:self.here], *(t[0] for t in self.shared))
        return ((y.double() - want).abs().amax() / want.abs().amax().clamp_min(1e-30)).item()


ERROR = 8 * 2.0 ** -9


@pytest.mark.parametrize("rows,n_shared,here,tiled", [
    ([18] * 16, 0, 0, False),                       # one row tile of 32 per expert
    ([300], 0, 0, True),                            # one hot expert
    ([33, 32, 32, 32], 0, 0, False),                # five row tiles of four groups: the last count that is thin
    ([33, 1, 1], 0, 0, True),                       # four of three
    ([0, 33, 1, 0, 32], 1, 30, False),              # five of four, the shared group among them
    ([32, 32], 1, 270, True),                       # the shared group is the hot one
    ([0, 0], 1, 0, False),                          # no rows at all
])
def test_sparse_batches_choose_their_gemms_by_the_rows(rows, n_shared, here, tiled):
    """129 to 512 tokens, at most 20 rows per expert by the mean, a layer of 64 MiB."""
    l = Layer(rows + [0] * (16 - len(rows)), 2048, 512, n_shared, here, T=300, E=16, k=1)   # 64 MiB of gate/up weights
    y, ws = l.run()
    plans = published_plans(ws)
    print(rows[:5], [p["items"] for p in plans], flush=True)
    assert all((p["items"] > 0) == tiled for p in plans)
    assert l.error(y) <= ERROR
    assert torch.equal(y, l.run()[0])
    # without room for partial tiles: thin whatever the rows
    z, _ = l.run(l.need - PARTIAL_TILES)
    assert l.error(z) <= ERROR
    assert tiled or torch.equal(y, z)


@pytest.mark.parametrize("rows,d,f,n_shared,here,gate_up,down", [
    # shared tiles in K pieces and left-over routed tiles cut in the same launch: slots and counters of both
    ([15] * 32, 2048, 2048, 2, 40, {}, dict(q=2, split=3, rounds=1)),
    # a cut 256-row tile (the shared group's), gate/up and down, in two to four pieces
    ([39, 29, 45, 48, 33], 1024, 128, 4, 194, dict(H=4, split=2), {}),
    ([49, 50, 32, 49, 54], 2048, 128, 4, 223, dict(H=4, split=3), {}),
    ([31, 30, 37, 32, 36, 29, 35, 51], 4096, 128, 1, 238, dict(H=4, split=4), {}),
    ([50, 55, 40, 48, 54], 256, 1024, 1, 222, {}, dict(H=4, split=2)),
    ([12, 8, 14, 16, 15, 16, 13, 15, 8, 15, 11, 10, 12, 15, 15, 15], 256, 2048, 1, 203, {}, dict(H=4, split=3)),
    ([54, 38, 29, 47, 53], 256, 3072, 1, 199, {}, dict(H=4, split=4)),
    # cut 128- and 64-row tiles
    ([72, 75, 133, 107, 121, 97, 102, 92], 4096, 256, 4, 783, dict(H=2, split=3), {}),
    ([133], 4096, 128, 1, 22, dict(H=1, split=4), {}),
    # shared tiles in two, three and four K pieces beside whole rounds of routed ones
    ([12] * 32, 2048, 512, 4, 191, {}, dict(q=2, rounds=1)),
    ([128, 103], 4096, 512, 4, 193, {}, dict(q=3, rounds=1)),
    ([196, 197], 2048, 1024, 4, 356, {}, dict(q=4, rounds=1)),
])
def test_work_lists_that_cut_tiles(rows, d, f, n_shared, here, gate_up, down):
    l = Layer(rows, d, f, n_shared, here, T=sum(rows), E=len(rows), k=1)
    y, ws = l.run()
    for p, want in zip(published_plans(ws), (gate_up, down)):
        print({n: v for n, v in p.items() if n != "groups"}, flush=True)
        assert {n: p[n] for n in want} == want
    assert l.error(y) <= ERROR
    for _ in range(3):
        assert torch.equal(y, l.run()[0])


@pytest.mark.parametrize("T,k,E,d,f,n_shared,rows,path", [
    (33, 4, 60, 512, 256, 4, [3, 9, 1], "thin"),               # four shared experts, a small layer
    (32, 4, 60, 2048, 512, 3, [1, 2] * 8, "thin"),             # three, 64 MiB of gate/up weights
    (33, 4, 60, 2048, 512, 3, [1, 2] * 8, "tiled"),
    (33, 4, 60, 2048, 512, 2, [1, 2] * 8, "thin"),
    (33, 4, 60, 2048, 512, 3, [1, 2] * 7 + [1], "thin"),       # 60 MiB
    (128, 6, 64, 512, 256, 2, [97, 31], "thin"),               # several row tiles, a shared K twice the routed one
    (129, 6, 64, 512, 256, 2, [97, 31], "tiled"),
    (129, 1, 7, 512, 256, 1, [97, 31], "thin"),                # 18.4 rows per expert
    (160, 8, 64, 512, 256, 1, [150, 10], "thin"),              # 20 rows per expert, a small layer
    (161, 8, 64, 512, 256, 1, [150, 10], "tiled"),
    (161, 8, 65, 512, 256, 1, [150, 10], "tiled"),             # 19.8, small, above 160 tokens
    (512, 5, 128, 2048, 512, 0, [32] * 16, "thin"),            # 20, 64 MiB of gate/up weights: by the rows
    (512, 5, 128, 2048, 512, 0, [100, 412] + [0] * 14, "tiled"),
    (513, 5, 129, 2048, 512, 0, [32] * 16, "tiled"),
    (80, 2, 8, 256, 12288, 1, [70, 10], "thin"),               # wide experts: 20 rows per expert
    (81, 2, 8, 256, 12288, 1, [70, 10], "tiled"),
    (81, 2, 8, 256, 12288 - 128, 1, [70, 10], "thin"),
    (81, 2, 8, 256, 12288, 2, [70, 10], "thin"),
])
def test_batches_on_either_side_of_the_rules(T, k, E, d, f, n_shared, rows, path):
    l = Layer(rows, d, f, n_shared, T // 2 if n_shared else 0, T, E, k)
    y, ws = l.run()
    tiled = l.need > PARTIAL_TILES and published_plans(ws)[0]["items"] > 0
    assert ("tiled" if tiled else "thin") == path
    assert l.error(y) <= ERROR
    assert torch.equal(y, l.run()[0])


def test_a_captured_sparse_batch_follows_its_rows():
    """The choice of the GEMMs is made on the device, so one graph serves batches of
    either kind: each replay equals the eager call on the same rows."""
    rows = [18] * 16
    l = Layer(rows, 2048, 512, 0, 0, T=300, E=16, k=1)
    even, hot = l.ek.clone(), torch.full_like(l.ek, 3)
    hot[l.m == 1] = 15
    ws = torch.empty(l.need, dtype=torch.uint8, device="cuda")
    y, ro = torch.empty((l.T, l.d), dtype=BF, device="cuda"), torch.empty(l.n + 2, dtype=torch.int32, device="cuda")
    ek = even.clone()

    def step():
        om.ordermoe_local_moe_forward(l.ex, l.x, l.T, l.k, l.w, ek, l.m, l.loc, 0, y, ro, ws)

    want = []
    for src in (even, hot):
        ek.copy_(src)
        step()
        torch.cuda.synchronize()
        want.append((y.clone(), published_plans(ws)[0]["items"] > 0))
    assert [t for _, t in want] == [False, True]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step()
    for i in (0, 1, 1, 0, 1):
        ek.copy_((even, hot)[i])
        y.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want[i][0]) and (published_plans(ws)[0]["items"] > 0) == want[i][1]
    del g
