"""Matrix-triple product on the GPU (VALU and int8-MFMA engines) against the oracle.

Small and ragged shapes are compared in full; the 1024-wide workload in full;
the 4096-wide workload on 4096 sampled entries computed one by one by the
oracle, on Freivalds' check of the reconstructed product and of its MAC, and on
the MAC-check sigma (which only depends on the opened E and F).
"""
import math

import numpy as np
import pytest
import torch

import oracle.fast as F
from oracle.pipelines import deal_matrices, matrix_triple_entries, matrix_triple_open, matrix_triple_run
from tests._util import dev, host, ints_of_sigma, share_to_dev
from workloads import ARR_MA, ARR_MX, P61

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def run_device(D, variant, check_seed):
    from paper_2512_11112_amd.spdz import Context, ShareTensor, TripleTensor
    ctx = Context(D.n, D.f.p, ints_of_sigma(D.alpha), check_seed)
    T = TripleTensor(share_to_dev(D.T.a), share_to_dev(D.T.b), share_to_dev(D.T.c))
    Z = ShareTensor.empty(D.n, 1, D.M * D.N)
    E = torch.empty((1, D.M * D.K), dtype=torch.int64, device="cuda")
    Fo = torch.empty((1, D.K * D.N), dtype=torch.int64, device="cuda")
    ctx.spdz_matmul_triple(D.M, D.K, D.N, share_to_dev(D.X), share_to_dev(D.Y), T, Z, E, Fo, variant)
    assert ctx.opened_count() == D.M * D.K + D.K * D.N
    ok, sigma = ctx.spdz_mac_check()
    return Z, E, Fo, ok, sigma


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("n,M,K,N", [(2, 70, 45, 33), (3, 64, 64, 64), (2, 1, 1, 1), (4, 130, 97, 65)])
def test_matmul_small_shapes(variant, n, M, K, N):
    D = deal_matrices(P61, n, M, K, N, 3)
    ref = matrix_triple_run(D, check_seed=3)
    Z, E, Fo, ok, sigma = run_device(D, variant, 3)
    assert np.array_equal(host(E), ref["E"]) and np.array_equal(host(Fo), ref["F"])
    assert np.array_equal(host(Z.val), ref["Z"].val)
    assert np.array_equal(host(Z.mac), ref["Z"].mac)
    assert ok and ref["ok"] and sigma == ints_of_sigma(ref["sigma"])


@pytest.mark.parametrize("variant", [0, 1])
def test_matmul_1024_full(variant):
    print(f"case N=1024 variant={variant}", flush=True)
    D = deal_matrices(P61, 2, 1024, 1024, 1024, 0)
    ref = matrix_triple_run(D, check_seed=0)
    Z, E, Fo, ok, sigma = run_device(D, variant, 0)
    assert np.array_equal(host(Z.val), ref["Z"].val)
    assert np.array_equal(host(Z.mac), ref["Z"].mac)
    assert ok and sigma == ints_of_sigma(ref["sigma"])


def test_matmul_extreme_digits_long_k():
    """Inputs whose balanced base-256 digits are near -128/127, inner dimension 8191 (the MFMA limit)."""
    from oracle.pipelines import DealtMat
    p, n, M, K, N = P61, 2, 64, 8191, 48
    rng = np.random.default_rng(5)
    pool = np.array([p - 1, 0x80, 0x7F7F7F7F7F7F7F & p, 0x8080808080808080 & p, 0x1F80808080808080 & p,
                     p - 0x80, 1, 0], dtype=np.uint64)
    f = F.Field(p)

    def sh(rows, cols):
        return F.Shares(pool[rng.integers(0, len(pool), (n, 1, rows * cols))],
                        pool[rng.integers(0, len(pool), (n, 1, rows * cols))])
    al = np.array([[p - 1], [0x8080808080808080 & p]], dtype=np.uint64)
    D = DealtMat(f, n, 0, M, K, N, al, None, sh(M, K), None, sh(K, N), F.TripleArr(sh(M, K), sh(K, N), sh(M, N)))
    ref = matrix_triple_run(D, check_seed=2)
    for variant in (0, 1):
        Z, E, Fo, ok, sigma = run_device(D, variant, 2)
        assert np.array_equal(host(Z.val), ref["Z"].val), variant
        assert np.array_equal(host(Z.mac), ref["Z"].mac), variant
        assert ok == ref["ok"] and sigma == ints_of_sigma(ref["sigma"])


def test_device_matrix_dealer_matches_oracle():
    from paper_2512_11112_amd.spdz import Context, TripleTensor
    D = deal_matrices(P61, 2, 100, 67, 40, 9)
    ctx = Context(2, P61, ints_of_sigma(D.alpha), 9)
    T = TripleTensor.empty_matrix(2, 100, 67, 40)
    ctx.spdz_deal_matrix_triple(9, ARR_MA, 100, 67, 40, T)
    for got, want in ((T.a, D.T.a), (T.b, D.T.b), (T.c, D.T.c)):
        assert np.array_equal(host(got.val), want.val) and np.array_equal(host(got.mac), want.mac)


@pytest.mark.timeout(900)
def test_matmul_4096_sampled_and_freivalds():
    """The 4096-wide workload as the benchmark runs it (device-dealt, MFMA engine)."""
    from paper_2512_11112_amd.spdz import Context, ShareTensor, TripleTensor
    print("case N=4096 MFMA sampled + Freivalds", flush=True)
    n, Nn, seed = 2, 4096, 0
    D = deal_matrices(P61, n, Nn, Nn, Nn, seed)
    f = D.f
    ctx = Context(n, P61, ints_of_sigma(D.alpha), seed)
    X, Y = share_to_dev(D.X), share_to_dev(D.Y)
    T = TripleTensor(share_to_dev(D.T.a), share_to_dev(D.T.b), share_to_dev(D.T.c))
    Z = ShareTensor.empty(n, 1, Nn * Nn)
    E = torch.empty((1, Nn * Nn), dtype=torch.int64, device="cuda")
    Fo = torch.empty((1, Nn * Nn), dtype=torch.int64, device="cuda")
    ctx.spdz_matmul_triple(Nn, Nn, Nn, X, Y, T, Z, E, Fo, 1)
    ok, sigma = ctx.spdz_mac_check()
    log = F.MacLog(f, n, seed, 0)
    E_ref, F_ref = matrix_triple_open(D, log)
    ok_ref, sig_ref = log.check(D.alpha)
    assert np.array_equal(host(E), E_ref) and np.array_equal(host(Fo), F_ref)
    assert ok and ok_ref and sigma == ints_of_sigma(sig_ref)
    rng = np.random.default_rng(1)
    rows = rng.integers(0, Nn, 4096)
    cols = rng.integers(0, Nn, 4096)
    rows[:2], cols[:2] = [0, Nn - 1], [0, Nn - 1]
    zv, zm = matrix_triple_entries(D, E_ref, F_ref, rows, cols)
    Zv, Zm = host(Z.val), host(Z.mac)
    flat = rows * Nn + cols
    for i in range(n):
        assert np.array_equal(Zv[i, 0, flat], zv[i]) and np.array_equal(Zm[i, 0, flat], zm[i])
    # Freivalds: (sum_i Z_i) v = X (Y v) and (sum_i M(Z)_i) v = alpha X (Y v) for random v
    Zs = f.open(Zv.reshape(n, 1, -1)).reshape(Nn, Nn)
    MZs = f.open(Zm.reshape(n, 1, -1)).reshape(Nn, Nn)
    Xs, Ys = D.Xs.reshape(Nn, Nn), D.Ys.reshape(Nn, Nn)
    v = f.uniform(77, 5, 20 * Nn).reshape(Nn, 20)
    lhs = f.matmul(Zs, v)
    rhs = f.matmul(Xs, f.matmul(Ys, v))
    assert np.array_equal(lhs, rhs)
    a = sum(int(D.alpha[i, 0]) for i in range(n)) % P61
    assert np.array_equal(f.matmul(MZs, v), f.scale_public(a, rhs.reshape(1, -1)).reshape(Nn, 20))


@pytest.mark.parametrize("n,M,K,N", [
    (2, 40, 2143, 30), (2, 40, 2144, 30),    # 17 moduli up to 2 K = 4287, then 18
    (2, 129, 63, 257), (3, 64, 65, 129),     # one past a tile, inner dimension around a plane block
    (2, 1281, 70, 1030),                     # several rounds of 256-wide tiles, ragged in both directions
    (8, 33, 5, 31), (5, 257, 1, 255),
])
def test_matmul_matrix_engine_shapes(n, M, K, N):
    """Sizes at the edges of the matrix engine's moduli, tiles and plane blocks, all entries."""
    D = deal_matrices(P61, n, M, K, N, 4)
    ref = matrix_triple_run(D, check_seed=4)
    Z, E, Fo, ok, sigma = run_device(D, 1, 4)
    assert np.array_equal(host(E), ref["E"]) and np.array_equal(host(Fo), ref["F"])
    assert np.array_equal(host(Z.val), ref["Z"].val) and np.array_equal(host(Z.mac), ref["Z"].mac)
    assert ok and sigma == ints_of_sigma(ref["sigma"])


@pytest.mark.parametrize("K,word", [(2143, (1 << 60) - 1), (2143, 1 << 60), (8191, (1 << 60) - 1), (8191, 1 << 60)])
def test_matmul_largest_sums(K, word):
    """Every opened and shared word at the largest balanced magnitude: sums next to the bound of the
    moduli (X - A = Y - B = word, so that no product cancels)."""
    from oracle.pipelines import DealtMat
    n, M, N = 2, 3, 5
    f = F.Field(P61)

    def sh(first, rows, cols):
        a = np.full((n, 1, rows * cols), 0, dtype=np.uint64)
        a[0] = first
        return F.Shares(a, a.copy())
    al = np.array([[1], [0]], dtype=np.uint64)
    X, A = sh((2 * word) % P61, M, K), F.Shares(*(np.full((n, 1, M * K), word, dtype=np.uint64) for _ in range(2)))
    Y, B = sh((2 * word) % P61, K, N), F.Shares(*(np.full((n, 1, K * N), word, dtype=np.uint64) for _ in range(2)))
    A.val[1] = A.mac[1] = B.val[1] = B.mac[1] = 0
    C = F.Shares(np.zeros((n, 1, M * N), dtype=np.uint64), np.zeros((n, 1, M * N), dtype=np.uint64))
    D = DealtMat(f, n, 0, M, K, N, al, None, X, None, Y, F.TripleArr(A, B, C))
    ref = matrix_triple_run(D, check_seed=6)
    Z, E, Fo, ok, sigma = run_device(D, 1, 6)
    assert np.array_equal(host(Z.val), ref["Z"].val) and np.array_equal(host(Z.mac), ref["Z"].mac)
    assert ok == ref["ok"] and sigma == ints_of_sigma(ref["sigma"])


def test_matmul_panels_match_valu_engine():
    """A product whose planes exceed the workspace bound runs in panels; the VALU engine gives the same shares."""
    from paper_2512_11112_amd import spdz as S
    n, M, K, N, seed = 2, 8200, 4100, 8190, 3
    ctx = S.Context(n, P61, S.deal_alpha(P61, n, seed), seed)
    X = ctx.spdz_deal_secret(seed, ARR_MX, S.ShareTensor.empty(n, 1, M * K))
    Y = ctx.spdz_deal_secret(seed, ARR_MX + 1, S.ShareTensor.empty(n, 1, K * N))
    T = ctx.spdz_deal_matrix_triple(seed, ARR_MX + 2, M, K, N, S.TripleTensor.empty_matrix(n, M, K, N))
    out = []
    for variant in (1, 0):
        print(f"case panels variant={variant}", flush=True)
        Z = S.ShareTensor.empty(n, 1, M * N)
        ctx.spdz_matmul_triple(M, K, N, X, Y, T, Z, variant=variant)
        assert ctx.spdz_mac_check()[0]
        out.append(Z)
    assert torch.equal(out[0].val, out[1].val) and torch.equal(out[0].mac, out[1].mac)
    ctx.close()


@pytest.mark.parametrize("n,M,K,N,limit", [
    (2, 300, 1362, 160, 40 << 20),    # tiles of 128 x 128: whole 79 MB, one tile 30 MB
    (4, 900, 64, 900, 9 << 20),       # 256 x 128: whole 155 MB, 256 x 256 13 MB, one tile 8 MB
    (2, 1000, 2200, 1000, 120 << 20), # 256 x 256, 18 moduli: whole 466 MB, one tile 103 MB
])
def test_matmul_short_workspace(monkeypatch, n, M, K, N, limit):
    """A context whose workspace is refused beyond a limit (by the runtime itself: the library asks for what no
    device has) runs a product in smaller panels, down to one tile; below that the call does nothing but say so."""
    from paper_2512_11112_amd import spdz as S
    seed = 6

    def context(bytes_):
        if bytes_:
            monkeypatch.setenv("SPDZ_WORKSPACE_LIMIT", str(bytes_))
        else:
            monkeypatch.delenv("SPDZ_WORKSPACE_LIMIT", raising=False)
        return S.Context(n, P61, S.deal_alpha(P61, n, seed), seed)
    whole = context(0)
    X = whole.spdz_deal_secret(seed, ARR_MX, S.ShareTensor.empty(n, 1, M * K))
    Y = whole.spdz_deal_secret(seed, ARR_MX + 1, S.ShareTensor.empty(n, 1, K * N))
    T = whole.spdz_deal_matrix_triple(seed, ARR_MX + 2, M, K, N, S.TripleTensor.empty_matrix(n, M, K, N))

    def product(ctx, variant):
        Z = S.ShareTensor.empty(n, 1, M * N)
        E, Fo = (torch.empty((1, w), dtype=torch.int64, device="cuda") for w in (M * K, K * N))
        ctx.spdz_matmul_triple(M, K, N, X, Y, T, Z, E, Fo, variant)
        assert ctx.spdz_mac_check()[0]
        return Z.val, Z.mac, E, Fo
    ref = product(whole, 0)
    bounded, short = context(limit), context(1 << 20)
    for ctx in (bounded, bounded, whole):  # the second finds the first one's workspace
        assert all(torch.equal(a, b) for a, b in zip(product(ctx, 1), ref))
    with pytest.raises(S.SpdzError) as e:
        product(short, 1)
    assert e.value.status == -4 and short.opened_count() == 0  # SPDZ_E_NOMEM
    assert torch.equal(short.spdz_open(X), whole.spdz_open(X))  # the failure is not the next call's
    assert short.spdz_mac_check()[0] and whole.spdz_mac_check()[0]
    for ctx in (bounded, short, whole):
        ctx.close()


def test_dealing_makes_room_for_the_product():
    """A product whose triple was dealt in its context allocates nothing, with the opened matrices kept or not."""
    from paper_2512_11112_amd import spdz as S
    n, M, K, N, seed = 3, 64, 4000, 64, 6
    ctx = S.Context(n, P61, S.deal_alpha(P61, n, seed), seed)
    X = ctx.spdz_deal_secret(seed, ARR_MX, S.ShareTensor.empty(n, 1, M * K))
    Y = ctx.spdz_deal_secret(seed, ARR_MX + 1, S.ShareTensor.empty(n, 1, K * N))
    Z = S.ShareTensor.empty(n, 1, M * N)
    E, Fo = (torch.empty((1, w), dtype=torch.int64, device="cuda") for w in (M * K, K * N))
    T = S.TripleTensor.empty_matrix(n, M, K, N)
    before = torch.cuda.mem_get_info()[0]
    ctx.spdz_deal_matrix_triple(seed, ARR_MX + 2, M, K, N, T)
    dealt = torch.cuda.mem_get_info()[0]
    assert before - dealt >= 18 * (2 * n + 1) * (M + N) * K  # the planes' bytes, without their padding
    for out in ((E, Fo), (None, None)):
        ctx.spdz_matmul_triple(M, K, N, X, Y, T, Z, *out)
        assert ctx.spdz_mac_check()[0] and torch.cuda.mem_get_info()[0] == dealt
    ctx.close()


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("over", ["val", "mac"])
def test_matmul_opened_right_matrix_over_the_left_operand(variant, over):
    """F_pub may take the place of X, which nothing reads once E is open (each operand at the far end of its own
    buffer, so that a launch of both opens would write F long before it reads X there)."""
    from paper_2512_11112_amd import spdz as S
    n, M, K, N, seed = 2, 1200, 600, 1100, 9
    got = []
    for place in (False, True):
        ctx = S.Context(n, P61, S.deal_alpha(P61, n, seed), seed)
        X = ctx.spdz_deal_secret(seed, ARR_MX, S.ShareTensor.empty(n, 1, M * K))
        Y = ctx.spdz_deal_secret(seed, ARR_MX + 1, S.ShareTensor.empty(n, 1, K * N))
        T = ctx.spdz_deal_matrix_triple(seed, ARR_MX + 2, M, K, N, S.TripleTensor.empty_matrix(n, M, K, N))
        Z, E = S.ShareTensor.empty(n, 1, M * N), torch.empty((1, M * K), dtype=torch.int64, device="cuda")
        Fo = torch.empty((1, K * N), dtype=torch.int64, device="cuda")
        if place:
            Fo = getattr(X, over).view(-1)[-K * N:].view(1, K * N)
        ctx.spdz_matmul_triple(M, K, N, X, Y, T, Z, E, Fo, variant)
        ok, sigma = ctx.spdz_mac_check()
        got.append((Z.val, Z.mac, E, Fo.clone()))
        assert ok and (not place or sigma == first)
        first = sigma
        ctx.close()
    assert all(torch.equal(a, b) for a, b in zip(*got))


LARGEST, SMALLEST = (1 << 60) - 1, 1 << 60  # balanced: 2^60 - 1 and -(2^60 - 1)


@pytest.mark.parametrize("K,left,right", [
    (2143, LARGEST, LARGEST), (2143, LARGEST, SMALLEST),  # 0.4499 M of 17 moduli, both signs
    (2144, LARGEST, LARGEST), (8191, LARGEST, LARGEST), (8191, LARGEST, SMALLEST),  # 18 moduli
    (8191, 128, 128), (8191, 128, 127),  # bytes mod 256: all -128 (sums 0.02 % below 2^28), -128 by 127
])
def test_matmul_sums_at_the_bounds(K, left, right):
    """Party 1's MAC output is a sum of 2 K equal products of the largest magnitude: its product is
    [E | M(A)_1] [M(B)_1 + alpha_1 F; F] with E = M(A)_1 = left, M(B)_1 = F = right and alpha_1 = 0."""
    from oracle.pipelines import DealtMat
    n, M, N = 2, 3, 5
    f = F.Field(P61)

    def sh(rows, cols, v0, m1):  # party 0's value shares, party 1's MAC shares
        val, mac = (np.zeros((n, 1, rows * cols), dtype=np.uint64) for _ in range(2))
        val[0], mac[1] = v0, m1
        return F.Shares(val, mac)
    if max(left, right) >= LARGEST:
        moduli = [256, 253, 251, 249, 247, 241, 239, 235, 233, 229, 227, 223, 217, 211, 199, 197, 193]
        assert (2 * K * LARGEST ** 2 / math.prod(moduli) > 0.4498) and (K > 2143 or 2 * K * LARGEST ** 2 < 0.45 * math.prod(moduli))
    X, Y, A, B = sh(M, K, left, 0), sh(K, N, right, 0), sh(M, K, 0, left), sh(K, N, 0, right)
    C = sh(M, N, 0, 0)
    al = np.array([[1], [0]], dtype=np.uint64)
    D = DealtMat(f, n, 0, M, K, N, al, None, X, None, Y, F.TripleArr(A, B, C))
    ref = matrix_triple_run(D, check_seed=6)
    balanced = [w if w < SMALLEST else w - P61 for w in (left, right)]
    assert (ref["Z"].mac[1] == 2 * K * balanced[0] * balanced[1] % P61).all()
    Z, E, Fo, ok, sigma = run_device(D, 1, 6)
    assert np.array_equal(host(Z.val), ref["Z"].val) and np.array_equal(host(Z.mac), ref["Z"].mac)
    assert ok == ref["ok"] and sigma == ints_of_sigma(ref["sigma"])
