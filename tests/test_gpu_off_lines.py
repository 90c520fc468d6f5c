"""Calls on rows that do not begin on cache lines, whose tiles are planned wider with up to 16
splits: every entry point at sizes on both sides of that rule, against the CPU oracle, and the
fused, stack, static and one-launch calls bitwise against the calls they stand for."""
import numpy as np
import pytest

import teal_inputs as ti
from oracle import teal_oracle as orc
from test_gpu_parity import T, TIGHT, dev, rel_l2, survivors  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

EPS = 1e-5
BITS = {"bf16": 16, "w8": 8}


class Group:
    """Matrices that read one x, in a format, and the calls on them."""

    def __init__(self, T, fmt, m, ns, seed):   # noqa: F811
        self.T, self.fmt, self.m, self.ns = T, fmt, m, ns
        w = [ti.weights_bf16(n, m, seed + k) for k, n in enumerate(ns)]
        if fmt == "bf16":
            self.host, self.W, self.scale = w, [dev(ti.to_input_channel_major(a)) for a in w], []
        else:
            self.host = [ti.quantize_w8(a) for a in w]
            self.W, self.scale = [dev(q) for q, _ in self.host], [dev(s) for _, s in self.host]
        self.ws = torch.zeros(T.teal_workspace_bytes(m, sum(ns)), dtype=torch.uint8, device="cuda")

    def outputs(self):
        return [torch.full((n,), float("nan"), dtype=torch.float32, device="cuda") for n in self.ns]

    def call(self, name, *args):
        """teal_sparse_gemv_<fmt><name> on the whole group."""
        lists = [self.W] + ([self.scale] if self.scale else [])
        self.T.check(getattr(self.T, f"teal_sparse_gemv_{self.fmt}{name}")(*lists, *args))
        torch.cuda.synchronize()

    def one(self, name, *args):
        """The same on its first matrix, with the single-matrix call."""
        first = [self.W[0]] + ([self.scale[0]] if self.scale else [])
        self.T.check(getattr(self.T, f"teal_sparse_gemv_{self.fmt}{name}")(*first, *args))
        torch.cuda.synchronize()

    def oracle(self, k, x, t):
        if self.fmt == "bf16":
            return orc.sparse_gemv_bf16(self.host[k], x, t)
        return orc.sparse_gemv_w8(*self.host[k], x, t)

    def planned_bytes(self):
        st, p = self.T.teal_gemv_plan_multi(BITS[self.fmt], self.m, self.ns)
        assert st == 0
        return p["tile_cols"] * BITS[self.fmt] // 8


# (format, input channels, widths, whether the rule widens)
CASES = [("bf16", 2560, [2824], True), ("bf16", 2552, [2824], False), ("bf16", 2560, [2808], False),
         ("bf16", 5000, [3416], True), ("bf16", 2568, [1032, 1032, 264, 1032], True),
         ("bf16", 4664, [4664, 1160, 1168], True), ("bf16", 8200, [4096, 1000, 1000], True),
         ("bf16", 3000, [12344, 12344], True), ("w8", 2560, [6160], True), ("w8", 2544, [6160], False),
         ("w8", 4656, [4656, 1152, 1168], True), ("w8", 8192, [8208, 1040], True)]


@pytest.mark.parametrize("fmt,m,ns,widens", CASES)
def test_calls_on_rows_off_cache_lines(T, fmt, m, ns, widens):   # noqa: F811
    G = Group(T, fmt, m, ns, seed=7000 + m)
    assert (G.planned_bytes() >= 512) == widens
    tight = TIGHT if fmt == "bf16" else 1e-4
    x = ti.make_x(m, 7100 + m, "laplace")
    xd = dev(x)
    for p in (0.25, 0.8):
        ts = [ti.quantile_threshold(x, min(0.95, p + 0.05 * k)) for k in range(len(ns))]
        got, again = G.outputs(), G.outputs()
        G.call("_multi", ts, got, ns, xd, m, G.ws)
        assert survivors(T, G.ws, len(ns)) == [orc.sparsify(x, t)[3] for t in ts]
        for k in range(len(ns)):
            assert rel_l2(got[k].cpu().numpy(), G.oracle(k, x, ts[k])) <= tight, k
        # the group in a stack of one, and a single matrix in its own call and in the library's scratch
        ws = torch.zeros(T.teal_workspace_bytes_stack([len(ns)], ns, [m]), dtype=torch.uint8, device="cuda")
        lists = [G.W] + ([G.scale] if G.scale else [])
        T.check(getattr(T, f"teal_sparse_gemv_{fmt}_stack")([len(ns)], *lists, ts, again, ns, [xd], [m], ws))
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, again))
        G.one("", xd, ts[0], again[0], m, ns[0], G.ws)
        assert rel_l2(again[0].cpu().numpy(), G.oracle(0, x, ts[0])) <= tight
        if len(ns) == 1:
            assert torch.equal(again[0], got[0])
        if fmt == "bf16":
            static = torch.full((ns[0],), float("nan"), dtype=torch.float32, device="cuda")
            T.check(T.teal_sparse_gemv_bf16_static(G.W[0], xd, ts[0], static, m, ns[0]))
            torch.cuda.synchronize()
            assert torch.equal(static, again[0])


@pytest.mark.parametrize("fmt,m,ns,widens", CASES)
def test_fused_calls_on_rows_off_cache_lines(T, fmt, m, ns, widens):   # noqa: F811
    """The input formed in the kernel, bitwise the producer kernel and the plain call."""
    G = Group(T, fmt, m, ns, seed=7200 + m)
    rng = np.random.default_rng(m)
    h, gamma = dev((2.5 * rng.standard_normal(m)).astype(np.float32)), dev((0.5 + 0.1 * rng.standard_normal(m)).astype(np.float32))
    gate, up = dev(rng.standard_normal(m).astype(np.float32)), dev(rng.standard_normal(m).astype(np.float32))
    xd = torch.empty(m, dtype=torch.int16, device="cuda")
    plain, fused = G.outputs(), G.outputs()
    T.check(T.teal_rmsnorm_f16(h, gamma, EPS, xd, m))
    ts = [0.3125] * len(ns)
    G.call("_multi", ts, plain, ns, xd, m, G.ws)
    G.call("_rmsnorm_multi", ts, fused, ns, h, gamma, EPS, m, G.ws)
    assert all(torch.equal(a, b) for a, b in zip(plain, fused))
    T.check(T.teal_swiglu_f16(gate, up, xd, m))
    G.one("", xd, 0.125, plain[0], m, ns[0], G.ws)
    G.one("_swiglu", gate, up, 0.125, fused[0], m, ns[0], G.ws)
    assert torch.equal(plain[0], fused[0])
    x = xd.cpu().numpy().view(np.float16)
    assert rel_l2(plain[0].cpu().numpy(), G.oracle(0, x, 0.125)) <= (TIGHT if fmt == "bf16" else 1e-4)


@pytest.mark.parametrize("fmt,m,f,d", [("bf16", 2560, 3080, 2824), ("bf16", 5128, 3592, 3336), ("w8", 2576, 6160, 6160)])
def test_one_launch_mlp_on_rows_off_cache_lines(T, fmt, m, f, d):   # noqa: F811
    """With the grouped call's own shape for gate and up, bitwise the grouped and the fused call."""
    gu, dn = Group(T, fmt, m, [f, f], 7300 + m), Group(T, fmt, f, [d], 7400 + m)
    st, sh = T.teal_mlp_plan(BITS[fmt], m, f, d)
    T.check(st)
    st, p = T.teal_gemv_plan_multi(BITS[fmt], m, [f, f])
    sh.gu_lanes_per_row, sh.gu_tile_cols, sh.gu_splits = p["lanes_per_row"], p["tile_cols"], p["splits"]
    assert gu.planned_bytes() >= 512 and sh.down_tile_cols * BITS[fmt] // 8 >= 512
    x = ti.gaussian_x(m, 7500 + m)
    t = ti.quantile_threshold(x, 0.5)
    xd = dev(x)
    ref, y_ref = gu.outputs(), dn.outputs()
    gu.call("_multi", [t, t], ref, [f, f], xd, m, gu.ws)
    dn.one("_swiglu", *ref, 0.0625, y_ref[0], f, d, dn.ws)
    got, y = gu.outputs(), dn.outputs()
    ws = torch.zeros(T.teal_workspace_bytes_mlp(m, f, d), dtype=torch.uint8, device="cuda")
    scales = [*gu.scale, *dn.scale]
    T.check(getattr(T, f"teal_sparse_mlp_{fmt}")(*gu.W, *dn.W, *scales, xd, t, t, 0.0625, *got, y[0], m, f, d,
                                                 ws, shape=sh))
    torch.cuda.synchronize()
    assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1]) and torch.equal(y[0], y_ref[0])
    want = gu.oracle(0, x, t)
    assert rel_l2(got[0].cpu().numpy(), want) <= (TIGHT if fmt == "bf16" else 1e-4)
