"""Calls whose sizes are any whole numbers or whose operands sit at any element alignment, against the fp64 oracle.

The bf16 calls keep the rank-space and hidden rows in fp32 between the stages (as three bf16 parts inside the matrix cores, which
hold all 24 bits), so the only coarse rounding is the result's: half a unit in the last place of each value.  Beyond that there are
the roundings of the fp32 sums: about 2^-24 of the sum of magnitudes for each of n terms, in either direction, sqrt(n) * 2^-24
together and 2^-18 for the longest sum here; with random factors the sum of magnitudes is below ten times the largest result, and no
call has more than four stages: 40 * 2^-18 of the largest result, and twice that as the bound (rounding the rank-space rows to
bf16 once, as the kernels for regular sizes do, is off by several times as much).  The fp32 calls sum in fp64 and round the rank-space and
hidden rows to fp32: the same with 2^-24."""
import numpy as np
import pytest

from paper_2605_08314_amd import synth
pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOL = {"bf16": 40 * 2.0 ** -17, "f32": 40 * 2.0 ** -24}
MANTISSA = {"bf16": 7, "f32": 23}


def beyond_rounding(got, want, dtype="bf16"):
    """Largest distance from the half-unit interval around the exact value, over the largest value."""
    unit = np.exp2(np.floor(np.log2(np.maximum(np.abs(want), 1e-30))) - MANTISSA[dtype])
    return float(np.max(np.abs(got - want) - 0.5 * unit) / np.max(np.abs(want)))


# around the 32-row blocks of K, the 64- and 128-column tiles of N, the 16-row blocks and 128-row tiles of M (33: the first
# row count of the tile kernels; 4096 x 371 at 130 rows: K cut into chunks)
ROWS = [1, 16, 17, 32, 33, 128, 130, 389]
SIZES = [  # (d_in, r, d_out)
    (31, 5, 19), (33, 63, 65), (257, 65, 127), (130, 33, 257), (1000, 301, 701), (64, 1, 4), (4096, 371, 1031), (2050, 512, 130),
]


@pytest.fixture(scope="module")
def G():
    import gpu_util
    assert torch.cuda.is_available()
    return gpu_util


def rand_t(rng, shape, scale=1.0, dtype="bf16"):
    return synth.to_dtype(rng.standard_normal(shape) * scale, dtype)


def offset_dev(G, t, by):
    """The tensor's copy on the device, `by` elements behind an aligned address."""
    d = G.dev(t)
    buf = torch.empty(d.numel() + by, dtype=d.dtype, device=d.device)
    v = buf[by:].view(d.shape)
    v.copy_(d)
    return v


@pytest.mark.parametrize("shared", [0, 1])       # 1: one launch per stage
@pytest.mark.parametrize("size", SIZES)
@pytest.mark.parametrize("M", ROWS)
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_linear(G, oracle, dtype, M, size, shared):
    B = G.B
    d_in, r, d_out = size
    rng = np.random.default_rng(M * 1000 + d_in)
    x, U, V = rand_t(rng, (M, d_in), 1.0, dtype), rand_t(rng, (d_in, r), d_in ** -0.5, dtype), rand_t(rng, (r, d_out), r ** -0.5, dtype)
    bias = rand_t(rng, (d_out,), 1.0, dtype)
    want = oracle.linear(x.f64, U.f64, V.f64, bias.f64)
    B.lowrank_configure(B.LR_CFG_DEVICE_SHARED, shared)
    try:
        y = G.run_linear(x, U, V, bias, "auto", dtype)
    finally:
        B.lowrank_configure(B.LR_CFG_DEVICE_SHARED, 0)
    assert beyond_rounding(G.host64(y), want, dtype) <= TOL[dtype]
    if not shared and M * r <= 131072:
        z = torch.full((M, d_out), float("nan"), dtype=G.tdtype(dtype), device="cuda")
        B.lowrank_linear_noalloc(G.dev(x), G.dev(U), G.dev(V), G.dev(bias), z)
        assert beyond_rounding(G.host64(z), want, dtype) <= TOL[dtype]


@pytest.mark.parametrize("M", [3, 20, 70])
@pytest.mark.parametrize("off", [1, 2, 7])
def test_regular_sizes_at_any_alignment(G, oracle, M, off):
    B = G.B
    rng = np.random.default_rng(off)
    x, U, V = rand_t(rng, (M, 512)), rand_t(rng, (512, 128), 512 ** -0.5), rand_t(rng, (128, 256), 128 ** -0.5)
    y = torch.full((M * 256 + off,), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = B.new_workspace(B.LR_OP_LINEAR, M, 512, 128, 256, B.LR_BF16)
    B.lowrank_linear(offset_dev(G, x, off), offset_dev(G, U, off), offset_dev(G, V, off), None, y[off:].view(M, 256), "auto", ws)
    assert torch.isnan(y[:off]).all()
    assert beyond_rounding(G.host64(y[off:].view(M, 256)), oracle.linear(x.f64, U.f64, V.f64)) <= TOL["bf16"]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("M", [1, 13, 32, 33, 260])
def test_small_integers_are_exact(G, oracle, M, dtype):
    """-1 / 0 / +1 operands whose partial sums are small whole numbers: bit for bit, so that an element taken from the wrong
    place (the end of a factor, the border of a column tile) cannot hide under a tolerance."""
    B = G.B
    rng = np.random.default_rng(M)
    for d_in, r, d_out in [(97, 67, 131), (321, 129, 63), (45, 31, 1)]:
        f = lambda *s: synth.to_dtype(rng.choice([-1.0, 0.0, 1.0], size=s) * (rng.random(s) < 0.15), dtype)  # noqa: E731
        x, U, V = f(M, d_in), f(d_in, r), f(r, d_out)
        y = G.run_linear(x, U, V, None, "auto", dtype)
        want = oracle.linear(x.f64, U.f64, V.f64)
        assert np.abs(want).max() <= 256                 # every whole number up to 256 is a bf16 value
        assert np.array_equal(G.host64(y), want), (d_in, r, d_out)


@pytest.mark.parametrize("shared", [0, 1])
@pytest.mark.parametrize("M,ranks", [(1, (101, 67, 93)), (5, (64, 1, 65)), (16, (33, 129, 31)), (17, (96, 95, 97)), (32, (131, 66, 250)),
                                     (33, (101, 67, 93)), (129, (1, 129, 31)), (300, (127, 64, 257))])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_packed_mlp(G, oracle, dtype, M, ranks, shared):
    B = G.B
    # fp32: SiLU itself is fp32 (hardware exponential and division, a few units in the last place of h)
    tol = TOL[dtype] * (1 if dtype == "bf16" else 8)
    w = synth.mlp_layer(M, d=389, ffn=1027, r_g=ranks[0], r_u=ranks[1], r_d=ranks[2], seed=700 + M, dtype=dtype, with_bias=True)
    t = w.t
    want = oracle.packed_mlp(t["x"].f64, t["U_gu"].f64, t["V_g"].f64, t["V_u"].f64, t["U_d"].f64, t["V_d"].f64,
                             t["b_g"].f64, t["b_u"].f64, t["b_d"].f64)
    B.lowrank_configure(B.LR_CFG_DEVICE_SHARED, shared)
    try:
        assert beyond_rounding(G.host64(G.run_mlp(w, "auto")), want, dtype) <= tol
    finally:
        B.lowrank_configure(B.LR_CFG_DEVICE_SHARED, 0)


@pytest.mark.parametrize("Bn,T", [(1, 1), (5, 3), (11, 2), (60, 3), (3, 50), (1, 200)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_qkv_with_cache_and_shared_basis(G, oracle, dtype, Bn, T):
    """Projections of different whole-number ranks, two of them on one basis, K and V rows into the cache (head_dim 33)."""
    B = G.B
    rng = np.random.default_rng(Bn)
    d_in, H, E, S_max, M = 203, 3, 33, T + 6, Bn * T
    N = H * E
    ranks = (37, 70, 70, 1)
    td = G.tdtype(dtype)
    Us = [rand_t(rng, (d_in, r), d_in ** -0.5, dtype) for r in ranks]
    Vs = [rand_t(rng, (r, n), r ** -0.5, dtype) for r, n in zip(ranks, (257, N, N, 66))]
    x = rand_t(rng, (M, d_in), 1.0, dtype)
    pos = np.asarray(rng.integers(0, S_max - T + 1, size=Bn), dtype=np.int32)
    U = [G.dev(u) for u in Us]
    U[2] = U[1]
    outs = [torch.full((M, v.f64.shape[1]), float("nan"), dtype=td, device="cuda") for v in Vs]
    kc = torch.full((Bn, S_max, H, E), 7.0, dtype=td, device="cuda")
    vc = torch.full_like(kc, 7.0)
    ws = B.new_workspace(B.LR_OP_QKV, M, d_in, sum(ranks), 257 + 2 * N + 66, G.code(dtype))
    B.lowrank_qkv(G.dev(x), U, [G.dev(v) for v in Vs], None, outs,
                  dict(k_cache=kc, v_cache=vc, pos=G.dev(pos), tokens_per_seq=T, k_index=1, v_index=2), "auto", ws)
    B.lowrank_workspace_status(ws)
    for i, u in enumerate((Us[0], Us[1], Us[1], Us[3])):
        assert beyond_rounding(G.host64(outs[i]), oracle.linear(x.f64, u.f64, Vs[i].f64), dtype) <= TOL[dtype], i
    for c, o in ((kc, outs[1]), (vc, outs[2])):
        want = np.full((Bn, S_max, N), G.bits(torch.tensor([7.0], dtype=td))[0])
        for b in range(Bn):
            want[b, pos[b]:pos[b] + T] = G.bits(o)[b * T:(b + 1) * T]
        assert np.array_equal(G.bits(c).reshape(want.shape), want)


def test_rank_project(G, oracle):
    B = G.B
    rng = np.random.default_rng(17)
    for M, d_in, r, dtype in [(5, 300, 67, "bf16"), (200, 777, 131, "bf16"), (70, 300, 67, "f32")]:
        x, U = rand_t(rng, (M, d_in), 1.0, dtype), rand_t(rng, (d_in, r), d_in ** -0.5, dtype)
        t = torch.full((M, r), float("nan"), dtype=G.tdtype(dtype), device="cuda")
        B.lowrank_rank_project(G.dev(x), G.dev(U), t, B.new_workspace(B.LR_OP_LINEAR, M, d_in, r, 0, G.code(dtype)))
        assert beyond_rounding(G.host64(t), x.f64 @ U.f64, dtype) <= TOL[dtype]


def same_pattern(got, want, dtype="bf16"):
    """Infinities of the same sign and NaN in the same places, everything else within the tolerance."""
    assert np.array_equal(np.isnan(got), np.isnan(want))
    inf = np.isinf(want)
    assert np.array_equal(np.isinf(got), inf) and np.array_equal(np.sign(got[inf]), np.sign(want[inf]))
    ok = np.isfinite(want)
    assert ok.any() and inf.any()
    assert beyond_rounding(got[ok], want[ok], dtype) <= TOL[dtype]


@pytest.mark.parametrize("whole", [False, True])       # True: rank-space values that are bf16 numbers, so that the lower half of their pair is zero
@pytest.mark.parametrize("M", [1, 16, 31, 33, 200])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_infinite_weights(G, oracle, dtype, M, whole):
    """An infinite weight makes its product infinite with the sign of the rank-space or hidden value, whatever the bits of that value."""
    rng = np.random.default_rng(M)
    d_in, r, d_out = 203, 67, 131
    f = lambda *s: rng.integers(1, 4, size=s) * rng.choice([-1.0, 1.0], size=s) * (rng.random(s) < 0.1) if whole else rng.standard_normal(s)  # noqa: E731
    x, U, V = f(M, d_in), f(d_in, r) if whole else f(d_in, r) * d_in ** -0.5, f(r, d_out) if whole else f(r, d_out) * r ** -0.5
    x[:, :r] += (2.0 if whole else 0.0) * (np.arange(r) % 2 * 2 - 1)
    V[5, 7], V[66, 64], V[0, 130], V[10, 20], V[11, 20] = np.inf, -np.inf, np.inf, np.inf, -np.inf
    x, U, V = (synth.to_dtype(a, dtype) for a in (x, U, V))
    t = x.f64 @ U.f64
    assert not whole or np.array_equal(synth.to_dtype(t, "bf16").f64, t)
    with np.errstate(invalid="ignore"):
        want = t @ V.f64
    same_pattern(G.host64(G.run_linear(x, U, V, None, "auto", dtype)), want, dtype)


@pytest.mark.parametrize("shared", [0, 1])
@pytest.mark.parametrize("where", ["V_g", "V_u", "U_d", "V_d"])
@pytest.mark.parametrize("M", [3, 32, 33, 140])
def test_infinite_weights_of_an_mlp(G, oracle, M, where, shared):
    """Every stage of the packed MLP: what an infinite weight reaches is infinite or NaN as in the formula, the rest as ever.  An infinite
    hidden value goes through positive weights into every rank; two columns of the result take the ranks up with one sign each."""
    B = G.B
    w = synth.mlp_layer(M, d=101, ffn=187, r_g=33, r_u=65, r_d=35, seed=40 + M, dtype="bf16", with_bias=True)
    t = dict(w.t)
    a = {k: t[k].f64.copy() for k in ("V_g", "V_u", "U_d", "V_d")}
    at = {"V_g": (4, 100), "V_u": (64, 130), "U_d": (186, 34), "V_d": (0, 100)}[where]
    if where in ("V_g", "V_u"):
        a["U_d"][at[1]] = np.abs(a["U_d"][at[1]]) + 0.125
        a["V_d"][:, 0], a["V_d"][:, 1] = np.abs(a["V_d"][:, 0]) + 0.125, -np.abs(a["V_d"][:, 1]) - 0.125
    a[where][at] = np.inf
    for k in a:
        t[k] = synth.to_dtype(a[k], "bf16")
        a[k] = t[k].f64
    w.t = t
    with np.errstate(all="ignore"):
        tt = t["x"].f64 @ t["U_gu"].f64
        g = tt[:, :33] @ a["V_g"] + t["b_g"].f64
        h = g / (1 + np.exp(-g)) * (tt[:, 33:] @ a["V_u"] + t["b_u"].f64)
        want = (h @ a["U_d"]) @ a["V_d"] + t["b_d"].f64
    B.lowrank_configure(B.LR_CFG_DEVICE_SHARED, shared)
    try:
        got = G.host64(G.run_mlp(w, "auto"))
    finally:
        B.lowrank_configure(B.LR_CFG_DEVICE_SHARED, 0)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    inf, ok = np.isinf(want), np.isfinite(want)
    assert np.array_equal(np.isinf(got), inf) and np.array_equal(np.sign(got[inf]), np.sign(want[inf]))
    assert inf.any()
    if ok.any():
        assert beyond_rounding(got[ok], want[ok]) <= TOL["bf16"]


@pytest.mark.parametrize("shared", [0, 1])
@pytest.mark.parametrize("M", [1, 16, 32, 33, 150])
def test_rank_space_and_hidden_rows_keep_all_bits(G, M, shared):
    """Rank-space and hidden values of 21 bits whose difference is one unit in their last place: it comes out exactly wherever the next
    factor subtracts them, so no bit of an fp32 value may be lost on the way into the matrix cores (two bf16 parts hold 16)."""
    B = G.B
    B.lowrank_configure(B.LR_CFG_DEVICE_SHARED, shared)
    try:
        # t[5], t[66] = 2^20 + 2^10 + 1 and 2^20 + 2^10
        d, r, n = 75, 67, 131
        x, U, V = np.zeros((M, d)), np.zeros((d, r)), np.zeros((r, n))
        s = 2.0 ** (np.arange(M) % 5)[:, None]
        x[:, [3, 40, 74]] = s
        U[[3, 40, 74], 5] = 2.0 ** 20, 2.0 ** 10, 1.0
        U[[3, 40], 66] = 2.0 ** 20, 2.0 ** 10
        V[5, 64:], V[66, 64:] = 1.0, -1.0
        V[5, :64], V[66, :64] = -1.0, 1.0
        y = G.host64(G.run_linear(synth.to_dtype(x, "bf16"), synth.to_dtype(U, "bf16"), synth.to_dtype(V, "bf16"), None, "auto", "bf16"))
        assert np.array_equal(y, s * np.where(np.arange(n) < 64, -1.0, 1.0))
        # the same in the packed MLP: g = 64 everywhere (SiLU(64) = 64 in fp32), u = the two values in hidden columns 1 and 99, their
        # difference in column 50; ranks 0, 20, 34 of the down factor take up each, column 0 of the result subtracts hidden rows,
        # column 1 takes the difference that gate/up made, column 2 subtracts down-factor ranks
        f, r_g, r_u, r_d = 101, 33, 37, 35
        U_gu, V_g, V_u, U_d, V_d = np.zeros((d, r_g + r_u)), np.zeros((r_g, f)), np.zeros((r_u, f)), np.zeros((f, r_d)), np.zeros((r_d, d))
        x[:, [3, 40, 74]] = 1.0
        x[:, 10] = 1.0
        U_gu[10, 32] = 64.0
        V_g[32] = 1.0
        U_gu[[3, 40, 74], r_g + 2] = 2.0 ** 20, 2.0 ** 10, 1.0
        U_gu[[3, 40], r_g + 36] = 2.0 ** 20, 2.0 ** 10
        V_u[2, 1] = V_u[36, 99] = V_u[2, 50] = 1.0
        V_u[36, 50] = -1.0
        U_d[1, 0], U_d[99, 0] = 1.0, -1.0
        U_d[50, 10] = 1.0
        U_d[1, 20], U_d[99, 34] = 1.0, 1.0
        V_d[0, 0] = V_d[10, 1] = V_d[20, 74] = 1.0
        V_d[34, 74] = -1.0
        w = [G.dev(synth.to_dtype(a, "bf16")) for a in (x, U_gu, V_g, V_u, U_d, V_d)]
        out = torch.full((M, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        ws = B.new_workspace(B.LR_OP_PACKED_MLP, M, d, r_g + r_u + r_d, f, B.LR_BF16)
        B.lowrank_packed_mlp(*w, None, None, None, out, "auto", ws)
        B.lowrank_workspace_status(ws)
        want = np.zeros((M, d))
        want[:, [0, 1, 74]] = 64.0
        assert np.array_equal(G.host64(out), want)
    finally:
        B.lowrank_configure(B.LR_CFG_DEVICE_SHARED, 0)


@pytest.mark.parametrize("kind", ["linear_f32", "mlp_f32", "qkv_bf16"])
def test_more_tiles_than_one_launch_has(G, kind):
    """Hundreds of millions of rows of one column: more workgroups than a grid may have (2^32 threads)."""
    B = G.B
    M = (1 << (27 if kind == "mlp_f32" else 28)) + 40
    g = torch.Generator(device="cuda"); g.manual_seed(3)
    x = torch.randn((M, 1), device="cuda", dtype=torch.bfloat16 if kind == "qkv_bf16" else torch.float32, generator=g)
    w = lambda *s: torch.randn(s, device="cuda", dtype=x.dtype, generator=g)     # noqa: E731
    if kind == "linear_f32":
        U, V, y = w(1, 1), w(1, 1), torch.full_like(x, float("nan"))
        B.lowrank_linear(x, U, V, None, y, "auto", B.new_workspace(B.LR_OP_LINEAR, M, 1, 1, 1, B.LR_F32))
        assert torch.equal(y, x * U * V)                                          # products of one term: two fp32 roundings on either side
    elif kind == "mlp_f32":
        U_gu, V_g, V_u, U_d, V_d = w(1, 2), w(1, 1), w(1, 1), w(1, 1), w(1, 1)
        y = torch.full_like(x, float("nan"))
        B.lowrank_packed_mlp(x, U_gu, V_g, V_u, U_d, V_d, None, None, None, y, "auto", B.new_workspace(B.LR_OP_PACKED_MLP, M, 1, 3, 1, B.LR_F32))
        h = torch.nn.functional.silu(x * U_gu[0, 0] * V_g) * (x * U_gu[0, 1] * V_u)
        torch.testing.assert_close(y, h * U_d * V_d, rtol=40 * 8 * 2.0 ** -24, atol=1e-30)      # (as for the packed MLP above)
    else:
        U, V = [w(1, 1) for _ in range(8)], [w(1, 1) for _ in range(8)]
        y = [torch.full_like(x, float("nan")) for _ in range(8)]
        B.lowrank_qkv(x, U, V, None, y, None, "auto", B.new_workspace(B.LR_OP_QKV, M, 1, 8, 8, B.LR_BF16))
        for i in range(8):                                                        # 24-bit products: exact before the one rounding
            assert torch.equal(y[i], (x.float() * U[i].float() * V[i].float()).to(torch.bfloat16)), i


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_sizes_beyond_24_bits(G, oracle, dtype):
    """Widths of 2^24 and more run the plain kernels, one thread per output element: layers, a cache, the hidden rows of an MLP."""
    B = G.B
    td, n = G.tdtype(dtype), (1 << 24) + 5
    g = torch.Generator(device="cuda"); g.manual_seed(5)
    w = lambda *s: torch.randn(s, device="cuda", dtype=td, generator=g)     # noqa: E731
    x, U, V, b = w(2, 3), [w(3, 2), w(3, 2)], [w(2, n), w(2, n)], w(n)
    want = [(x.double() @ U[i].double()).float().double() @ V[i].double() for i in range(2)]
    y = torch.full((2, n), float("nan"), device="cuda", dtype=td)
    B.lowrank_linear(x, U[0], V[0], b, y, "auto", B.new_workspace(B.LR_OP_LINEAR, 2, 3, 2, n, G.code(dtype)))
    eps = 2.0 ** -8 if dtype == "bf16" else 2.0 ** -23              # one rounding of the result (and of two terms in fp32)
    close = lambda got, ref: torch.all((got.double() - ref).abs() <= eps * ref.abs() + 4 * eps * 2.0 ** -10)     # noqa: E731
    assert close(y, want[0] + b.double())
    kc, vc = (torch.full((2, 3, 1, n), 7.0, device="cuda", dtype=td) for _ in range(2))
    pos = torch.tensor([0, 2], device="cuda", dtype=torch.int32)
    B.lowrank_qkv(x, U, V, None, [y, None], dict(k_cache=kc, v_cache=vc, pos=pos, tokens_per_seq=1, k_index=0, v_index=1), "auto",
                  B.new_workspace(B.LR_OP_QKV, 2, 3, 4, 2 * n, G.code(dtype)))
    assert close(y, want[0])
    for c, ref in ((kc, want[0]), (vc, want[1])):
        assert close(c[0, 0, 0], ref[0]) and close(c[1, 2, 0], ref[1])
        assert (c[0, 1:] == 7.0).all() and (c[1, :2] == 7.0).all()
    del kc, vc, y, want
    # the hidden rows are read back through a down factor that takes up three of them, the last one included
    U_gu, V_g, V_u, U_d, V_d = w(3, 4), w(2, n), w(2, n), torch.zeros((n, 3), device="cuda", dtype=td), torch.eye(3, device="cuda", dtype=td)
    at = [0, 12345678, n - 1]
    for i, k in enumerate(at):
        U_d[k, i] = 1.0
    out = torch.full((2, 3), float("nan"), device="cuda", dtype=td)
    B.lowrank_packed_mlp(x, U_gu, V_g, V_u, U_d, V_d, None, None, None, out, "auto", B.new_workspace(B.LR_OP_PACKED_MLP, 2, 3, 7, n, G.code(dtype)))
    t = x.double() @ U_gu.double()
    h = torch.nn.functional.silu(t[:, :2] @ V_g[:, at].double()) * (t[:, 2:] @ V_u[:, at].double())
    assert torch.all((out.double() - h).abs() <= 16 * eps * h.abs().max())
