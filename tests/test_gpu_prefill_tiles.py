"""Products on the 256-row tiles, whose two halves of a workgroup take turns: the shortest and longest K, row and column
remainders, one and several tiles per workgroup, cache rows."""
import pytest
import torch

from util import TOL, max_rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import gpu_util
    assert torch.cuda.is_available()
    return gpu_util


def normal(g, *s):
    return torch.randn(*s, device="cuda", dtype=torch.bfloat16, generator=g)


def check(got, want, n_out=1):
    assert max_rel_err(got.double().cpu().numpy(), want.double().cpu().numpy()) <= TOL["bf16"]


@pytest.mark.parametrize("M,K,N", [(1281, 64, 8192), (2048, 128, 8192), (1300, 192, 8320), (3000, 384, 4096), (4096, 64, 12416), (2305, 4096, 6272),
                                   (8192, 4096, 1536), (7937, 128, 1536)])
def test_product(G, M, K, N):
    assert G.B.lowrank_prefill_tile(M, K, N, 1) in {(256, 256, 0), (256, 192, 0)}
    g = torch.Generator(device="cuda"); g.manual_seed(M + K)
    x, U = normal(g, M, K), normal(g, K, N)
    t = torch.full((M + 1, N), float("nan"), device="cuda", dtype=torch.bfloat16)      # one row more: must stay as it is
    ws = G.B.new_workspace(G.B.LR_OP_QKV, M, K, N, N, G.B.LR_BF16)
    want = x.float() @ U.float()
    for _ in range(2):
        G.B.lowrank_rank_project(x, U, t[:M], ws)
        torch.cuda.synchronize()
        check(t[:M], want)
    assert torch.isnan(t[M]).all()


@pytest.mark.parametrize("M,K,N", [(33, 128, 128), (128, 128, 4096), (129, 192, 640), (500, 768, 4096), (1000, 384, 4096), (40, 4096, 384), (100, 11008, 768),
                                   (512, 4096, 1536), (300, 64, 4096)])
def test_product_of_few_tiles(G, M, K, N):
    """At most one 128 x 128 tile per compute unit: the two halves of a workgroup share K (not below K = 128)."""
    g = torch.Generator(device="cuda"); g.manual_seed(M + K)
    x, U = normal(g, M, K), normal(g, K, N)
    t = torch.full((M + 1, N), float("nan"), device="cuda", dtype=torch.bfloat16)
    ws = G.B.new_workspace(G.B.LR_OP_QKV, M, K, N, N, G.B.LR_BF16)
    for _ in range(2):
        G.B.lowrank_rank_project(x, U, t[:M], ws)
        torch.cuda.synchronize()
        check(t[:M], x.float() @ U.float())
    assert torch.isnan(t[M]).all()


def runs_prefill_kernels(M, d, f, r_g, r_u, r_d):
    """The rule of the tuned prefill products: K in 64-row steps, N in 128-column tiles, for all five factors."""
    return all(k >= 64 and k % 64 == 0 and n >= 128 and n % 128 == 0 for k, n in ((d, r_g + r_u), (r_g, f), (r_u, f), (f, r_d), (r_d, d)))


# K of gate/up at its shortest for two halves (128: two steps each), in odd steps per half (192, 320), unequal on the two sides, below
# 128 on one side or both (one workgroup of four waves per tile then); row remainders.  The last three have ranks outside the rule
# of the tuned kernels and run the any-size tile kernels.
MLP_OF_FEW_TILES = [(40, 128, 128, 128), (129, 192, 192, 128), (200, 192, 320, 128), (128, 128, 256, 384), (100, 64, 64, 128), (77, 64, 192, 128), (256, 768, 512, 256),
                    (40, 128, 192, 128), (128, 256, 128, 192), (200, 64, 128, 64)]


@pytest.mark.parametrize("M,r_g,r_u,r_d", MLP_OF_FEW_TILES)
def test_mlp_of_few_tiles(G, M, r_g, r_u, r_d):
    assert runs_prefill_kernels(M, 512, 1408, r_g, r_u, r_d) == ((M, r_g, r_u, r_d) not in MLP_OF_FEW_TILES[-3:])
    assert ((M + 127) // 128) * (1408 // 128) <= 256                 # gate/up: at most one tile per compute unit
    g = torch.Generator(device="cuda"); g.manual_seed(M)
    d, f = 512, 1408
    x = normal(g, M, d)
    w = [normal(g, a, b) * a ** -0.5 for a, b in ((d, r_g + r_u), (r_g, f), (r_u, f), (f, r_d), (r_d, d))]
    b = [normal(g, n) for n in (f, f, d)]
    y = torch.empty_like(x)
    ws = G.B.new_workspace(G.B.LR_OP_PACKED_MLP, M, d, r_g + r_u + r_d, f, G.B.LR_BF16)
    G.B.lowrank_packed_mlp(x, *w, *b, y, "prefill", ws)
    torch.cuda.synchronize()
    W, c = [t.float() for t in w], [t.float() for t in b]
    t = x.float() @ W[0]
    h = torch.nn.functional.silu(t[:, :r_g] @ W[1] + c[0]) * (t[:, r_g:] @ W[2] + c[1])
    check(y, h @ W[3] @ W[4] + c[2])


@pytest.mark.parametrize("n,T,past", [(7, 300, 7), (2, 1025, 0), (30, 70, 3)])
def test_cache_rows_and_bias(G, n, T, past):
    g = torch.Generator(device="cuda"); g.manual_seed(T)
    M, d, r, H, S = n * T, 4096, 128, 32, past + T + 2
    assert G.B.lowrank_prefill_tile(M, r, d, 3)[:2] == (256, 256)
    x = normal(g, M, d)
    U, V = [normal(g, d, r) * d ** -0.5 for _ in range(3)], [normal(g, r, d) * r ** -0.5 for _ in range(3)]
    b = [normal(g, d), None, normal(g, d)]
    q = torch.empty((M, d), device="cuda", dtype=torch.bfloat16)
    kc, vc = (normal(g, n, S, H, 128) for _ in range(2))
    k0, v0 = kc.clone(), vc.clone()
    pos = torch.tensor([past + i % 3 for i in range(n)], device="cuda", dtype=torch.int32)
    ws = G.B.new_workspace(G.B.LR_OP_QKV, M, d, 3 * r, 3 * d, G.B.LR_BF16)
    G.B.lowrank_qkv(x, U, V, b, [q, None, None], dict(k_cache=kc, v_cache=vc, pos=pos, tokens_per_seq=T, k_index=1, v_index=2), "prefill", ws)
    torch.cuda.synchronize()
    want = [(x.float() @ u.float()) @ v.float() + (0 if c is None else c.float()) for u, v, c in zip(U, V, b)]
    check(q, want[0])
    for cache, old, w in ((kc, k0, want[1]), (vc, v0, want[2])):
        for i in range(n):
            p = int(pos[i])
            assert torch.equal(cache[i, :p], old[i, :p]) and torch.equal(cache[i, p + T:], old[i, p + T:])
            check(cache[i, p:p + T].reshape(T, d), w[i * T:(i + 1) * T])


@pytest.mark.parametrize("M,K,N,tile", [(4096, 8192, 1536, (256, 192, 1)), (8192, 4096, 1536, (256, 192, 0)), (3000, 384, 4096, (256, 256, 0)), (512, 768, 4096, (128, 128, 0)),
                                        (512, 4096, 1536, (128, 128, 5))])
def test_infinite_weights(G, M, K, N, tile):
    """An infinite weight makes its column infinite, with the sign of the row's value, in every form of the product: also where K is shared
    between workgroups or cut into chunks, whichever part it falls into."""
    assert G.B.lowrank_prefill_tile(M, K, N, 1) == tile
    g = torch.Generator(device="cuda"); g.manual_seed(M + K)
    x, U = normal(g, M, K), normal(g, K, N)
    at = {3: 0, 130: K // 2 + 5, 700: K - 1, N - 1: 77}
    for n, k in at.items():
        U[k, n] = float("inf")
    t = torch.empty((M, N), device="cuda", dtype=torch.bfloat16)
    G.B.lowrank_rank_project(x, U, t, G.B.new_workspace(G.B.LR_OP_LINEAR, M, K, N, 0, G.B.LR_BF16))
    torch.cuda.synchronize()
    for n, k in at.items():
        assert torch.equal(t[:, n].float(), x[:, k].float() * float("inf"))        # (NaN for a zero in x: equal() refuses NaN, and randn has none)
    rest = [n for n in range(N) if n not in at]
    check(t[:, rest], (x.float() @ U[:, rest].float()))
