"""Kernels at the sizes where their tiles, remainders and dispatch lines lie, against fp64 results."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2605_16184_amd as ast
from paper_2605_16184_amd import binding as B
from paper_2605_16184_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _with_spectrum(n, lam, *key):
    U = W.haar(n, DEV, *key, dtype=torch.float64)
    A = (U * lam) @ U.T.contiguous()
    return (0.5 * (A + A.T)).float().contiguous()


def _spectrum(kind, n):
    if kind == "flat":
        return torch.linspace(1.0, 0.9, n, device=DEV, dtype=torch.float64)
    if kind == "power":
        return 0.05 * W.powerlaw_sigma(n, DEV).double() ** 2
    return 0.05 * W.logspaced_sigma(n, 8.0, DEV).double() ** 2


# packed tiles whose padding, the rows and columns beyond n, is not data
def _packed_with_nan_padding(A):
    n, T = A.shape[0], 128
    P = torch.empty(ast.packed_elems(n), device=DEV)
    ast.sym_pack([(A, P)])
    if n % T:
        last = P.view(-1, T, T)[-((n + T - 1) // T):]           # the tiles of the last block row
        last[:, n % T:] = float("nan")
        last[-1, :, n % T:] = float("nan")
    return P


def _root_error(A, X, eps):
    w, V = torch.linalg.eigh(A.double())
    e = eps * float(w[-1])
    ref = (V * (w + e).clamp_min(1e-3 * e).pow(-0.25)) @ V.T.contiguous()
    return float(torch.linalg.norm(X.double() - ref) / torch.linalg.norm(ref)), float(w[-1])


@pytest.mark.parametrize("kind", ["flat", "power", "log"])
@pytest.mark.parametrize("eps", [1e-3, 1e-6, 1e-8])
@pytest.mark.parametrize("sizes", [
    [1, 2, 31, 33, 64, 65, 127, 128, 129, 255, 256, 257],       # 64-wide tiles; recurrence of all in the registers of one or two workgroups
    [513, 640],                                                 # ... of six and seven
    [130] * 190 + [97, 128, 256],                               # 128-wide tiles
    [514] * 192,                                                # more workgroups that share a factor than find room at once
    [761] * 118 + [33, 520, 768, 770],                          # 256-wide tiles: remainders of 249, 8 and 2, transposed panels
    [76, 80, 520] * 60, [900] * 70 + [1040] * 4,                # 128- and 256-wide tiles: a block row beyond the last row
    [64, 33] * 150, [200, 333] * 32, [200, 333] * 40,           # many small tiles: as many as large ones; below four per CU; beyond
    [64, 65, 96, 97, 192, 193] * 40,                            # digit tiles with 64 rows left, one more, 32 more and less
])
def test_roots_at_the_edges(kind, eps, sizes):
    made = {}
    for n in sizes:
        if n not in made:
            made[n] = _with_spectrum(n, _spectrum(kind, n), 7, n)
    As = [made[n] for n in sizes]
    Xs = [torch.full_like(A, float("nan")) for A in As]
    lam = torch.zeros(len(As), device=DEV)
    info = torch.full((len(As),), -1, dtype=torch.int32, device=DEV)
    ast.inverse_root(list(zip(As, Xs)), eps, info=info, lambda_max=lam)
    torch.cuda.synchronize()
    assert bool((info == 0).all())
    last = {n: i for i, n in enumerate(sizes)}
    for n, i in last.items():
        err, top = _root_error(As[i], Xs[i], eps)
        assert err <= 2e-3, (n, err)
        assert abs(float(lam[i]) - top) <= 1e-4 * top, (n, float(lam[i]), top)
        assert bool((Xs[i] == Xs[i].T).all())
        first = sizes.index(n)
        assert torch.equal(Xs[first], Xs[i])                    # the same factor anywhere in the batch


# Largest eigenvalue with the matrix in the registers of several workgroups: rows and columns of a member's last wavefront and last
# chunk, one member and 43, rows of every alignment, packed tiles whose padding is not a number.  The estimate is fp32 arithmetic on a
# spectrum whose top is a factor of 4 apart: a few units of 2^-24 of a sum of n products, far below the 1e-5 asked here.
@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("sizes", [[257, 1, 2, 3, 4, 5], [512, 192, 193, 191], [513, 608, 577], [1024, 300], [1025, 97], [2048, 2047], [333] * 300,
                                   [2049, 1500, 700, 300, 100]])      # beside a factor that does not fit: all by the other ways
def test_largest_eigenvalue_from_registers(sizes, packed):
    made = {n: _with_spectrum(n, _spectrum("power", n), 7, n) for n in set(sizes)}
    top = {n: float(torch.linalg.eigvalsh(A.double())[-1]) for n, A in made.items()}
    items = []
    for n in sizes:
        X = torch.full((n, n), float("nan"), device=DEV)
        if packed:
            items.append((_packed_with_nan_padding(made[n]), X, 1))
        else:
            wide = torch.full((n, n + n % 3), float("nan"), device=DEV)      # what lies beyond a row's end is not data
            wide[:, :n] = made[n]
            items.append((wide[:, :n], X, 0))
    info = torch.full((len(sizes),), -1, dtype=torch.int32, device=DEV)
    lam = torch.zeros(len(sizes), device=DEV)
    ast.inverse_root(items, 1e-6, info=info, lambda_max=lam)
    torch.cuda.synchronize()
    assert bool((info == 0).all())
    for n, x in zip(sizes, lam.tolist()):
        assert abs(x - top[n]) <= 1e-5 * top[n], (n, x, top[n])
    n = max(sizes)
    made[n][n - 1, n - 1] = float("nan")                        # reported, by every member alike
    A = _packed_with_nan_padding(made[n]) if packed else made[n]
    ast.inverse_root([(A, torch.zeros(n, n, device=DEV), int(packed))], 1e-6, info=info[:1])
    torch.cuda.synchronize()
    assert int(info[0]) == 2


# Roots with bounds on the waits of the estimate that several workgroups share: how often a member looks for the others' sums and for y.
def _roots_with_waits(items, eps, looks_sums, looks_y, info, lam):
    f = ast.Factors(items)
    ws = torch.empty(ast.inverse_root_workspace_bytes(f)[0], dtype=torch.uint8, device=DEV)
    st = ast.lib().asteria_inverse_root_waits(f.array, f.count, 4, B.EPS_RELATIVE, (ctypes.c_float * 1)(eps), 1, None, info.data_ptr(), None, None,
                                              lam.data_ptr(), ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream, looks_sums, looks_y)
    assert st == B.OK
    torch.cuda.synchronize()


# Sums of squares that did not arrive must not pass for small ones: with a trace of half of n lambda_max (and the matrix itself far from a
# multiple of the identity) they would make the iteration end after one update, with a root that is none.
@pytest.mark.parametrize("n", [320, 1000])
def test_sums_that_a_wait_gave_up_are_not_used(n):
    trace = 0.5 * 1.01 * (n - 0.05)                             # n - 2 tr / (1.01 lambda_max) = 0.05, the squares left out
    lam = torch.full((n,), 1e-5, device=DEV, dtype=torch.float64)
    lam[:int(trace)] = 1.0
    lam[int(trace)] = 0.0
    lam[int(trace)] = trace - float(lam.sum())
    A = _with_spectrum(n, lam, 7, n)
    X, top = torch.full_like(A, float("nan")), torch.zeros(1, device=DEV)
    info = torch.full((1,), -1, dtype=torch.int32, device=DEV)
    _roots_with_waits([(A, X)], 1e-6, 1 << 21, 1 << 21, info, top)
    assert int(info[0]) == 0 and _root_error(A, X, 1e-6)[0] <= 2e-3
    X.fill_(float("nan"))
    _roots_with_waits([(A, X)], 1e-6, 0, 1 << 21, info, top)
    assert int(info[0]) != 0 or _root_error(A, X, 1e-6)[0] <= 2e-3, (info, top)


# Workgroups that give up a wait leave their factor to one that waits for nobody: the same outcome.  At once, after a few looks (some give
# up, some do not), by the first one alone; every width of a row's share, one member and 43, packed, a factor that is not finite.
@pytest.mark.parametrize("looks", [(0, 1 << 21), (1 << 21, 0), (1 << 21, 1), (1 << 21, 4), (2, 2)])
@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("sizes", [[257, 1, 2, 3, 129], [513, 100, 641], [333] * 300, [2048, 2047, 1025]])
def test_roots_where_workgroups_give_up_waiting(sizes, packed, looks):
    made = {n: _with_spectrum(n, _spectrum("power", n), 7, n) for n in set(sizes)}
    items = [(_packed_with_nan_padding(made[n]) if packed else made[n], torch.full((n, n), float("nan"), device=DEV), int(packed)) for n in sizes]
    info = torch.full((len(sizes),), -1, dtype=torch.int32, device=DEV)
    lam = torch.zeros(len(sizes), device=DEV)
    _roots_with_waits(items, 1e-6, *looks, info, lam)
    assert bool((info == 0).all())
    for n in made:
        i = max(k for k, m in enumerate(sizes) if m == n)
        err, top = _root_error(made[n], items[i][1], 1e-6)
        assert err <= 2e-3, (n, err)
        assert abs(float(lam[i]) - top) <= 1e-5 * top, (n, float(lam[i]), top)
    items[0][0].view(-1)[0] = float("inf")
    _roots_with_waits(items[:1], 1e-6, *looks, info[:1], lam)
    assert int(info[0]) == 2


# Refreshes on several streams at once, each with factors whose workgroups wait for each other, beside other work: as one after the other
def test_roots_on_several_streams_at_once():
    batches = [[2048, 1100, 700, 300] * 4, [1500, 2047] * 6, [600, 1024] * 20]
    made = {n: _with_spectrum(n, _spectrum("power", n), 7, n) for n in {n for b in batches for n in b}}
    streams = [torch.cuda.Stream() for _ in batches]
    busy = torch.randn(4096, 4096, device=DEV)
    want, got, infos, ws = [], [], [], []
    for b in batches:
        want.append([torch.full_like(made[n], float("nan")) for n in b])
        got.append([torch.full_like(made[n], float("nan")) for n in b])
        infos.append(torch.full((len(b),), -1, dtype=torch.int32, device=DEV))
        f = ast.Factors([(made[n], X) for n, X in zip(b, want[-1])])
        ws.append(torch.empty(ast.inverse_root_workspace_bytes(f)[0], dtype=torch.uint8, device=DEV))
        ast.inverse_root(f, 1e-6, info=infos[-1], ws=ws[-1])
    torch.cuda.synchronize()
    assert all(bool((i == 0).all()) for i in infos)
    for _ in range(4):
        for s, b, X, i, w in zip(streams, batches, got, infos, ws):
            i.fill_(-1)
            s.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(s):
                ast.inverse_root([(made[n], x) for n, x in zip(b, X)], 1e-6, info=i, ws=w)
        for _ in range(4):
            busy = busy @ busy * 1e-3
        torch.cuda.synchronize()
        assert all(bool((i == 0).all()) for i in infos)
        for X, Y in zip(want, got):
            assert all(torch.equal(x, y) for x, y in zip(X, Y))
            for y in Y:
                y.fill_(float("nan"))


# Captured into a graph, the stream asked for its compute units while it captures: every replay on new statistics as the eager call
@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("sizes", [[300, 700], [64, 100]])
def test_roots_in_a_captured_graph(sizes, static):
    made = [[_with_spectrum(n, _spectrum("power", n), seed, n) for n in sizes] for seed in (7, 8, 9)]
    As = [A.clone() for A in made[0]]
    Xs, eager = ([torch.full_like(A, float("nan")) for A in As] for _ in range(2))
    info = torch.full((len(sizes),), -1, dtype=torch.int32, device=DEV)
    f = ast.Factors(list(zip(As, Xs)))
    ws = torch.empty(ast.inverse_root_workspace_bytes(f)[0], dtype=torch.uint8, device=DEV)

    def call(factors):
        if static:
            ast.inverse_root_static(factors, 1e-6, info=info)
        else:
            ast.inverse_root(factors, 1e-6, info=info, ws=ws)
    call(f)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(f)
    for statistics in made + made[:1]:
        for A, new, X in zip(As, statistics, Xs):
            A.copy_(new)
            X.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert bool((info == 0).all())
        call(ast.Factors(list(zip(As, eager))))
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(Xs, eager))


# Few digit tiles are computed in quarters, many in halves: the same integers.  (The sums of the residual have another order; it enters the
# interval of a factor off the schedule only, a few units of 2^-24.)  Remainders in either half of a tile, and none.
@pytest.mark.parametrize("eps", [1e-6, 1e-8])
@pytest.mark.parametrize("n", [65, 128, 130, 192, 200, 300])
def test_digit_products_in_quarters_are_those_of_halves(n, eps):
    A = _with_spectrum(n, _spectrum("power", n), 7, n)
    count = 129 // (((n + 127) // 128) * ((n + 127) // 128 + 1) // 2) + 1
    alone, Xs = torch.full_like(A, float("nan")), [torch.full_like(A, float("nan")) for _ in range(count)]
    info = torch.full((count,), -1, dtype=torch.int32, device=DEV)
    ast.inverse_root([(A, alone)], eps, info=info[:1])
    ast.inverse_root([(A, X) for X in Xs], eps, info=info)
    torch.cuda.synchronize()
    assert bool((info == 0).all())
    for X in Xs:
        assert float(torch.linalg.norm(X - alone) / torch.linalg.norm(alone)) <= 1e-5
    assert _root_error(A, alone, eps)[0] <= 2e-3


# mostly small factors, for which small tiles pay, beside one that is too large for them
def test_roots_of_small_factors_beside_a_large_one():
    sizes = [2700] + [64] * 1100
    made = {n: _with_spectrum(n, _spectrum("power", n), 7, n) for n in set(sizes)}
    Xs = [torch.full_like(made[n], float("nan")) for n in sizes]
    alone = {n: torch.full_like(made[n], float("nan")) for n in made}
    info = torch.full((len(sizes),), -1, dtype=torch.int32, device=DEV)
    ast.inverse_root([(made[n], X) for n, X in zip(sizes, Xs)], 1e-6, info=info)
    for n in made:
        ast.inverse_root([(made[n], alone[n])], 1e-6)
    torch.cuda.synchronize()
    assert bool((info == 0).all())
    assert all(torch.equal(X, alone[n]) for n, X in zip(sizes, Xs))


def _dense(n, kind):
    i = torch.arange(1, n + 1, device=DEV, dtype=torch.float64)
    if kind == "graded":                                        # rows scaled over 4 decades
        A = W.haar(n, DEV, 13, n, dtype=torch.float64) * i.pow(-0.5)
        s = 10 ** (-4 * (i - 1) / (n - 1))
        A = (A @ A.T.contiguous()) * s[:, None] * s[None, :]
        return (0.5 * (A + A.T)).float().contiguous()
    if kind == "axis":                                          # a power law close to the axes: largest diagonal entry 0.8 lambda_max
        v = torch.ones_like(i) + 2.0 * (i == 1)
        v = v / v.norm()
        A = torch.diag(i ** -2.0)
        A = A - 2.0 * torch.outer(v, v @ A)
        A = A - 2.0 * torch.outer(A @ v, v)
        return (0.5 * (A + A.T)).float().contiguous()
    lam = {"power": i ** -2.0, "log": 10 ** (-16 * (i - 1) / (n - 1)),
           "lowrank": torch.where(i <= 32, 1.0 / i, torch.full_like(i, 1e-5))}[kind]
    return _with_spectrum(n, 0.03 * lam, 13, n)


@pytest.mark.parametrize("eps", [1e-6, 1e-8])
@pytest.mark.parametrize("n", [130, 333, 1024])
@pytest.mark.parametrize("kind", ["power", "lowrank", "graded", "log", "axis"])
def test_round_off_of_the_roots(kind, n, eps):
    A = _dense(n, kind)
    X = torch.empty_like(A)
    ast.inverse_root([(A, X)], eps)
    w, V = torch.linalg.eigh(A.double())
    d = (w + eps * w[-1]).clamp_min(1e-3 * eps * float(w[-1]))
    Y = V.T.contiguous() @ X.double() @ V
    D = torch.diag(torch.diagonal(Y))
    # The schedule's own truncation commutes with A; what does not is round-off.  Bounds: the most that the iteration on
    # fp32 matrices, which hands over to the 16-bit cores one step later, gives for these spectra at n up to 1024 (3.6e-5;
    # log-spaced 3.5e-4 and 6.5e-4).  32 directions out of 130: a larger diagonal at that step, 6e-5
    r = d.pow(0.125)
    noise = float(torch.linalg.norm((Y - D) * r[:, None] * r[None, :])) / n ** 0.5
    assert noise <= {"log": 3.5e-4 if eps == 1e-6 else 6.5e-4}.get(kind, 3.6e-5 if kind != "lowrank" or n > 130 else 1e-4), noise
    ref = torch.diag(d.pow(-0.25))
    assert float(torch.linalg.norm(Y - ref) / torch.linalg.norm(ref)) <= 5e-4


@pytest.mark.parametrize("eps", [0.1, 1e-2, 1e-4, 1e-6, 1e-8])
@pytest.mark.parametrize("n", [16, 64, 600])
@pytest.mark.parametrize("below, count", [(0.45, 1), (0.9, 1), (0.9, 16), (1.3, 1), (1.3, 16), (5.0, 1)])
def test_roots_of_statistics_with_negative_eigenvalues(n, eps, below, count):
    # eigenvalues -below * eps * lambda_max: with A + eps I positive definite the root is found, otherwise refused
    lam = torch.linspace(1.0, 0.5, n, device=DEV, dtype=torch.float64)
    lam[n - min(count, n // 2):] = -below * eps
    A = torch.diag(lam).float()                                 # exact: the fp32 rounding of a dense one is of the size of eps = 1e-8
    X = torch.empty_like(A)
    info = torch.full((1,), -1, dtype=torch.int32, device=DEV)
    ast.inverse_root([(A, X)], eps, info=info)
    torch.cuda.synchronize()
    if below > 1.0:
        assert int(info[0]) == ast.binding.INFO_NOT_PD
    else:
        assert int(info[0]) == 0
        ref = torch.diag((torch.diagonal(A).double() + eps).pow(-0.25))
        assert float(torch.linalg.norm(X.double() - ref) / torch.linalg.norm(ref)) <= 2e-3


def test_roots_of_a_batch_with_an_eps_per_factor():
    items, eps = [], []
    for n in (130, 333, 520):
        for kind in ("power", "graded", "log"):
            for e in (0.3, 1e-3, 1e-4, 1e-6, 1e-8):
                items.append((_dense(n, kind), torch.empty(n, n, device=DEV)))
                eps.append(e)
    info = torch.full((len(items),), -1, dtype=torch.int32, device=DEV)
    ast.inverse_root(items, eps, info=info)
    torch.cuda.synchronize()
    assert bool((info == 0).all())
    for (A, X), e in zip(items, eps):
        assert _root_error(A, X, e)[0] <= 2e-3, (A.shape[0], e)


@pytest.mark.parametrize("opts", [None, dict(lowp_from=40)])
@pytest.mark.parametrize("sizes", [[128] * 200 + [1500], [700] * 191 + [513], [700] * 192, [700] * 191 + [1000]])
def test_roots_of_uneven_batches(sizes, opts):
    # the general path: either side of the line between a workgroup per factor and a launch per step for the largest eigenvalue
    made = {n: _with_spectrum(n, _spectrum("power", n), 7, n) for n in set(sizes)}
    Xs = [torch.empty_like(made[n]) for n in sizes]
    lam = torch.zeros(len(sizes), device=DEV)
    ast.inverse_root([(made[n], X) for n, X in zip(sizes, Xs)], 1e-6, opts=None if opts is None else ast.RootOpts(**opts), lambda_max=lam)
    torch.cuda.synchronize()
    last = {n: i for i, n in enumerate(sizes)}
    for n, i in last.items():
        err, top = _root_error(made[n], Xs[i], 1e-6)
        assert err <= 2e-3 and abs(float(lam[i]) - top) <= 1e-4 * top, (n, err)
        assert torch.equal(Xs[sizes.index(n)], Xs[i])


@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("m, n", [(8, 8), (8, 136), (120, 64), (128, 128), (136, 120), (264, 8), (7, 9), (129, 63), (256, 392), (384, 200)])
def test_statistics_at_the_edges(m, n, packed):
    g = torch.Generator(device=DEV).manual_seed(m * 1000 + n)
    G = torch.randn(m, n, generator=g, device=DEV).bfloat16()
    full, made = [], []
    for k in (m, n):
        a = torch.randn(k, k, generator=g, device=DEV)
        full.append((a + a.T).contiguous())
        made.append(full[-1].clone())
    if packed:
        made = [torch.empty(ast.packed_elems(k), device=DEV) for k in (m, n)]
        ast.sym_pack(list(zip(full, made)))
    for beta in (0.75, 0.0):
        ast.stats_update([(G, made[0], made[1], 0, 1 if packed else 0)], beta)
        got = made
        if packed:
            got = [torch.empty(k, k, device=DEV) for k in (m, n)]
            ast.sym_unpack(list(zip(got, made)))
        torch.cuda.synchronize()
        H = G.double()
        for side, a in enumerate(got):
            P = H @ H.T.contiguous() if side == 0 else H.T.contiguous() @ H
            ref = beta * full[side].double() + (1.0 - beta) * P
            k = H.shape[1 - side]
            # exact products, fp32 sums of k of them, one rounding each of the two terms and their sum
            tol = (k + 3) * 2.0 ** -24 * (beta * full[side].double().abs() + (1.0 - beta) * (H.abs() @ H.abs().T if side == 0 else H.abs().T @ H.abs()))
            assert bool(((a.double() - ref).abs() <= tol).all()), (m, n, side, beta)
            assert torch.equal(a, a.T), (m, n, side, beta)
            full[side] = a.clone()


@pytest.mark.parametrize("sizes", [[1, 2, 15, 16, 17, 33, 48], [127, 128, 129, 191, 192, 193], [385, 1153],
                                   [256] * 49 + [250], [256] * 129 + [384]])    # products on whole tiles of 128 with a ragged factor beside them, of both
def test_refresh_at_the_edges(sizes):
    As = [_with_spectrum(n, _spectrum("power", n) + 1e-4, 9, n) for n in sizes]
    Q0 = [W.haar(n, DEV, 11, n) for n in sizes]
    Qs, Qt = [q.clone() for q in Q0], [torch.zeros(n, n, device=DEV) for n in sizes]
    info = torch.full((len(sizes),), -1, dtype=torch.int32, device=DEV)
    ast.soap_refresh(list(zip(As, Qs)), info=info, qt=Qt)
    torch.cuda.synchronize()
    assert bool((info == 0).all())
    for n, A, q0, q, qt in zip(sizes, As, Q0, Qs, Qt):
        assert torch.equal(qt, q.T)
        Q, Z = q.double().cpu().numpy(), (A.double() @ q0.double()).cpu().numpy()
        R = Q.T @ Z
        assert np.linalg.norm(Q.T @ Q - np.eye(n)) / np.sqrt(n) <= 1e-5, n
        assert np.linalg.norm(np.tril(R, -1)) <= 1e-5 * np.linalg.norm(Z), n
        assert np.all(np.diag(R) >= 0), n


# whole panels of 128 rows: one, an odd number, pairs and one over; the last fills the 256-wide tiles of the panel products
@pytest.mark.parametrize("n,count", [(128, 2), (384, 2), (640, 3), (640, 513)])
def test_refresh_on_whole_panels(n, count):
    A = _with_spectrum(n, _spectrum("power", n) + 1e-4, 9, n)
    q0 = W.haar(n, DEV, 11, n)
    Qs, Qt = [q0.clone() for _ in range(count)], [torch.zeros(n, n, device=DEV) for _ in range(count)]
    other = torch.empty(n, n + 1, device=DEV)[:, :n]             # a row pitch that the general products take
    other.copy_(q0)
    info = torch.full((count,), -1, dtype=torch.int32, device=DEV)
    ast.soap_refresh([(A, q) for q in Qs], info=info, qt=Qt)
    one = torch.full((1,), -1, dtype=torch.int32, device=DEV)
    ast.soap_refresh([(A, other)], info=one)
    torch.cuda.synchronize()
    assert bool((info == 0).all()) and int(one[0]) == 0
    for q, qt in zip(Qs, Qt):
        assert torch.equal(q, Qs[0]) and torch.equal(qt, q.T)
    Z = (A.double() @ q0.double()).cpu().numpy()
    for q in (Qs[0], other):
        Q = q.double().cpu().numpy()
        R = Q.T @ Z
        assert np.linalg.norm(Q.T @ Q - np.eye(n)) / np.sqrt(n) <= 1e-5
        assert np.linalg.norm(np.tril(R, -1)) <= 1e-5 * np.linalg.norm(Z)
        assert np.all(np.diag(R) >= 0)


# workspaces from the smallest one to that of the whole batch: panels share passes over the finished rows where their coefficients fit
@pytest.mark.parametrize("sizes", [(512, 640, 1024, 300, 768), (1024,), (1000, 100)])
def test_refresh_does_not_depend_on_the_size_of_the_workspace(sizes):
    As = [_with_spectrum(n, _spectrum("power", n) + 1e-4, 9, n) for n in sizes]
    q0 = [W.haar(n, DEV, 11, n) for n in sizes]
    full, least = ast.soap_refresh_workspace_bytes([(A, q) for A, q in zip(As, q0)])
    got = []
    for size in sorted({least, min(full, least + 600_000), max(least, full - 256), full}):
        buf = torch.full((size + 4096,), 255, dtype=torch.uint8, device=DEV)      # NaN in whatever is read before it is written
        Qs, info = [q.clone() for q in q0], torch.full((len(sizes),), -1, dtype=torch.int32, device=DEV)
        ast.soap_refresh(list(zip(As, Qs)), info=info, ws=buf[:size])
        torch.cuda.synchronize()
        assert bool((info == 0).all()) and bool((buf[size:] == 255).all()), size
        got.append(Qs)
    for Qs in got[1:]:
        assert all(torch.equal(q, r) for q, r in zip(Qs, got[0]))
    for A, q, Q in zip(As, q0, got[0]):
        Z = (A.double() @ q.double()).cpu().numpy()
        Q = Q.double().cpu().numpy()
        assert np.linalg.norm(Q.T @ Q - np.eye(len(Q))) / np.sqrt(len(Q)) <= 1e-5
        assert np.linalg.norm(np.tril(Q.T @ Z, -1)) <= 1e-5 * np.linalg.norm(Z)


# a workspace for half of the batch without the coefficients that shared passes over the finished rows take: two passes, not more;
# the product A Q is one launch a pass
@pytest.mark.parametrize("extra,passes", [(0, 2), (-256, 4)])    # two factors a pass; just not two: one each
def test_refresh_takes_no_more_passes_for_shared_ones(extra, passes):
    n, count = 512, 4
    A = _with_spectrum(n, _spectrum("power", n) + 1e-4, 9, n)
    Qs = [W.haar(n, DEV, 11, n) for _ in range(count)]
    f = [(A, q) for q in Qs]
    (full1, least), (full4, _) = ast.soap_refresh_workspace_bytes(f[:1]), ast.soap_refresh_workspace_bytes(f)
    fixed = full1 - (full4 - full1) // (count - 1)
    ws = torch.empty(fixed + 2 * (least - fixed) + extra, dtype=torch.uint8, device=DEV)
    ast.profile_enable(4096)
    ast.soap_refresh(f, ws=ws)
    torch.cuda.synchronize()
    kinds = [k for _, k in ast.profile_collect()]
    assert kinds.count(513) == passes
    assert all(torch.equal(q, Qs[0]) for q in Qs)


# a batch on the large tiles of the product A Q, its parts on the small ones; factors of either kernel
# (the last takes 256-wide tiles for whole panels too)
@pytest.mark.parametrize("sizes", [[256] * 110 + [512, 768, 300, 640, 1024], [256] * 260 + [250, 130], [256] * 341 + [130], [384] * 260 + [130] * 9])
def test_refresh_does_not_depend_on_the_batch(sizes):
    made = {n: (_with_spectrum(n, _spectrum("power", n) + 1e-4, 9, n), W.haar(n, DEV, 11, n)) for n in set(sizes)}
    As, q0 = zip(*[made[n] for n in sizes])
    full, least = ast.soap_refresh_workspace_bytes(list(zip(As, q0)))
    streams = [torch.cuda.Stream() for _ in range(2)]

    def run(which, size=None, aux=None):
        Qs = [q0[i].clone() for i in which]
        ws = torch.full((size,), 255, dtype=torch.uint8, device=DEV) if size else None
        ast.soap_refresh([(As[i], q) for i, q in zip(which, Qs)], ws=ws, aux_streams=aux)
        torch.cuda.synchronize()
        return Qs

    every = list(range(len(sizes)))
    want = run(every)
    for size, aux in ((least, None), (least + (full - least) // 3, None), (full, streams)):
        assert all(torch.equal(a, b) for a, b in zip(run(every, size, aux), want)), size
    for i in {n: k for k, n in enumerate(sizes)}.values():
        assert torch.equal(run([i])[0], want[i]), sizes[i]


@pytest.mark.parametrize("out", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("blocks", [
    [(256, 256)] * 3 + [(250, 256)],                            # too few whole tiles: 128-wide tiles
    [(256, 512)] * 48 + [(512, 256)] * 48 + [(257, 260)],       # whole tiles, and a ragged block beside them
    [(256, 256)] * 48, [(256, 256)] * 49,                       # either side of the dispatch line, short K
    [(512, 512)] * 32, [(512, 512)] * 33, [(512, 512)] * 65,    # K = 512: either side of it, a round and a remainder
])
def test_two_sided_products_at_the_edges(blocks, out):
    g = torch.Generator(device=DEV).manual_seed(5)

    def mk(m, n, dt=torch.float32):
        return torch.randn(m, n, generator=g, device=DEV).to(dt)

    def sym(n):                                                 # roots are symmetric
        a = mk(n, n)
        return (a + a.T).contiguous()

    items = []
    for i, (m, n) in enumerate(blocks):
        # every third output is a view with a row pitch that is no multiple of 8
        P = torch.full((m, n + (3 if i % 3 == 0 else 0)), float("nan"), device=DEV, dtype=out)[:, :n]
        items.append((sym(m), mk(m, n, torch.bfloat16), sym(n), P))
    ast.precondition(items)
    steps = [(G, mk(*XL.shape) / XL.shape[0] ** 0.5, mk(*XR.shape) / XR.shape[0] ** 0.5, torch.zeros(P.shape, device=DEV), torch.ones(P.shape, device=DEV),
              torch.empty(P.shape, device=DEV)) for XL, G, XR, P in items]
    ast.soap_step(steps, 0.0, 0.5, 1e-8, 100)
    torch.cuda.synchronize()
    for (XL, G, XR, P), (_, QL, QR, M, _, _) in zip(items, steps):
        ref = XL.double() @ G.double() @ XR.double()
        # two bf16 terms of every fp32 operand keep 16 bits, in three operands; a bf16 result adds 2^-9
        tol = 3 * 2.0 ** -16 + (2.0 ** -9 if out == torch.bfloat16 else 0.0)
        assert float(torch.linalg.norm(P.double() - ref) / torch.linalg.norm(ref)) <= tol, P.shape
        rot = QL.double().T.contiguous() @ G.double() @ QR.double()      # beta1 = 0: the first moment is G'
        assert float(torch.linalg.norm(M.double() - rot) / torch.linalg.norm(rot)) <= 3 * 2.0 ** -16, P.shape


# Few tiles stage two slabs, many one: the same sums in the same order
@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("m, n", [(8, 8), (136, 264), (264, 56), (128, 1024)])
def test_statistics_of_few_tiles_are_those_of_many(m, n, packed):
    g = torch.Generator(device=DEV).manual_seed(m + n)
    G = torch.randn(m, n, device=DEV, generator=g).bfloat16()

    def fresh():
        return [torch.zeros(ast.packed_elems(k) if packed else (k, k), device=DEV) for k in (m, n)]
    one, layout = fresh(), 1 if packed else 0
    tiles = sum(((k + 127) // 128) * ((k + 127) // 128 + 1) // 2 for k in (m, n))
    many = [fresh() for _ in range(512 // tiles + 1)]
    ast.stats_update([(G, one[0], one[1], 0, layout)], 0.95)
    ast.stats_update([(G, L, R, 0, layout) for L, R in many], 0.95)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for s in many for a, b in zip(s, one))


# Few tiles are computed in quarters, many whole: the same sums in the same order, so the same bits.  Sizes with remainders in the
# first, the second and no quarter of a tile, rows of every alignment, k within one slab and over several.
@pytest.mark.parametrize("grad", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("m, n", [(1, 1), (63, 65), (64, 64), (65, 127), (129, 31), (191, 193), (300, 517)])
def test_products_in_quarters_are_those_of_whole_tiles(m, n, grad):
    g = torch.Generator(device=DEV).manual_seed(m * 1000 + n)
    XL, XR = (X + X.T for X in (torch.randn(k, k, device=DEV, generator=g) for k in (m, n)))
    G = torch.randn(m, n, device=DEV, generator=g).to(grad)
    alone = torch.empty(m, n, device=DEV)
    ast.precondition([(XL, G, XR, alone)])
    count = 257 // (((m + 127) // 128) * ((n + 127) // 128)) + 1
    Ps = [torch.empty(m, n, device=DEV) for _ in range(count)]
    ast.precondition([(XL, G, XR, P) for P in Ps])
    torch.cuda.synchronize()
    assert all(torch.equal(P, alone) for P in Ps)
    ref = XL.double() @ G.double() @ XR.double()
    # both terms kept to 2^-16 of every fp32 operand, products of random sign
    assert float(torch.linalg.norm(alone.double() - ref) / torch.linalg.norm(ref)) <= 4 * 2.0 ** -16


def _pitched(A, extra):
    wide = torch.full((A.shape[0], A.shape[1] + extra), float("nan"), dtype=A.dtype, device=DEV)
    wide[:, :A.shape[1]] = A
    return wide[:, :A.shape[1]]


# ... and the statistics on the fp32 and fp64 cores, and on the bf16 cores where the rows of the gradient are no whole 16-byte pieces: dense and
# packed, with aligned rows and without.  The error is that of sums of k products of random sign, rounded to fp32 (fp64 sums: once).
@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("grad, double", [(torch.float32, 0), (torch.float32, 1), (torch.bfloat16, 1), (torch.bfloat16, 0)])
@pytest.mark.parametrize("m, n, extra", [(1, 1, 1), (63, 65, 0), (64, 128, 0), (65, 127, 3), (129, 31, 1), (191, 193, 0), (256, 128, 0), (300, 517, 2)])
def test_statistics_in_quarters_are_those_of_whole_tiles(m, n, extra, grad, double, packed):
    g = torch.Generator(device=DEV).manual_seed(m * 1000 + n)
    G = _pitched(torch.randn(m, n, device=DEV, generator=g).to(grad), extra + (1 if grad == torch.bfloat16 and not double and (n + extra) % 8 == 0 else 0))
    old = [X + X.T for X in (torch.randn(k, k, device=DEV, generator=g) for k in (m, n))]

    def fresh():
        if not packed:
            return [_pitched(X, extra) for X in old]
        Ps = [torch.empty(ast.packed_elems(k), device=DEV) for k in (m, n)]
        ast.sym_pack(list(zip(old, Ps)))
        return Ps
    one = fresh()
    ast.stats_update([(G, one[0], one[1], double, int(packed))], 0.75)
    count = 257 // min(((k + 127) // 128) * ((k + 127) // 128 + 1) // 2 for k in (m, n)) + 1
    many = [fresh() for _ in range(count)]
    ast.stats_update([(G, L, R, double, int(packed)) for L, R in many], 0.75)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for s in many for a, b in zip(s, one))
    for new, before, H in zip(one, old, (G.double(), G.double().T)):
        if packed:
            full = torch.empty_like(before)
            ast.sym_unpack([(full, new)])
            new = full
        ref = 0.75 * before.double() + 0.25 * (H.contiguous() @ H.T.contiguous())
        assert float(torch.linalg.norm(new.double() - ref) / torch.linalg.norm(ref)) <= (2.0 ** -24 if double else 2.0 ** -24 * (2 + H.shape[1] ** 0.5))


# ... and the rotations of the SOAP step, with a basis on both sides and on one
@pytest.mark.parametrize("grad", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("sides", ["L", "R", "LR"])
@pytest.mark.parametrize("m, n, extra", [(1, 1, 0), (63, 65, 0), (64, 128, 0), (65, 127, 3), (129, 31, 1), (191, 193, 0), (256, 128, 0), (300, 517, 2)])
def test_soap_steps_in_quarters_are_those_of_whole_tiles(m, n, extra, sides, grad):
    g = torch.Generator(device=DEV).manual_seed(m * 1000 + n)
    QL, QR = (_pitched(W.haar(k, DEV, 3, k), extra) if side in sides else None for side, k in (("L", m), ("R", n)))
    G = _pitched(torch.randn(m, n, device=DEV, generator=g).to(grad), extra)
    M, V = torch.randn(m, n, device=DEV, generator=g), torch.rand(m, n, device=DEV, generator=g) + 0.5

    def fresh():
        return [_pitched(M, extra), _pitched(V, extra), _pitched(torch.zeros_like(M), extra)]
    one = fresh()
    ast.soap_step([(G, QL, QR, *one)], 0.5, 0.75, 1e-8, 3)
    many = [fresh() for _ in range(257 // (((m + 127) // 128) * ((n + 127) // 128)) + 1)]
    ast.soap_step([(G, QL, QR, *s) for s in many], 0.5, 0.75, 1e-8, 3)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for s in many for a, b in zip(s, one))
    ql, qr = (torch.eye(k, device=DEV, dtype=torch.float64) if Q is None else Q.double() for Q, k in ((QL, m), (QR, n)))
    rot = ql.T.contiguous() @ G.double() @ qr
    mom, var = 0.5 * M.double() + 0.5 * rot, 0.75 * V.double() + 0.25 * rot ** 2
    step = (mom / (1 - 0.5 ** 3)) / ((var / (1 - 0.75 ** 3)).sqrt() + 1e-8)
    ref = ql @ step @ qr.T.contiguous()
    for got, want in zip(one, (mom, var, ref)):
        # both terms kept to 2^-16 of every operand of the four rotations
        assert float(torch.linalg.norm(got.double() - want) / torch.linalg.norm(want)) <= 8 * 2.0 ** -16


# ... and of the moments under new bases
@pytest.mark.parametrize("m, n, extra", [(1, 1, 0), (65, 127, 3), (191, 193, 0), (256, 128, 0), (300, 517, 2)])
def test_moments_under_new_bases_in_quarters_are_those_of_whole_tiles(m, n, extra):
    Q = [_pitched(W.haar(k, DEV, key, k), extra) for k in (m, n) for key in (3, 4)]      # L old, L new, R old, R new
    M = torch.randn(m, n, device=DEV, generator=torch.Generator(device=DEV).manual_seed(m * 1000 + n))
    one = _pitched(M, extra)
    ast.soap_reproject([(Q[0], Q[1], Q[2], Q[3], one, None, None, None)])
    many = [_pitched(M, extra) for _ in range(257 // (((m + 127) // 128) * ((n + 127) // 128)) + 1)]
    ast.soap_reproject([(Q[0], Q[1], Q[2], Q[3], X, None, None, None) for X in many])
    torch.cuda.synchronize()
    assert all(torch.equal(X, one) for X in many)
    d = [q.double() for q in Q]
    ref = d[1].T.contiguous() @ d[0] @ M.double() @ d[2].T.contiguous() @ d[3]
    assert float(torch.linalg.norm(one.double() - ref) / torch.linalg.norm(ref)) <= 8 * 2.0 ** -16


@pytest.mark.parametrize("opts", [None, dict(int8_slices=0), dict(lowp_from=40)])
@pytest.mark.parametrize("power", [-100, -80, -64, 48])
@pytest.mark.parametrize("sizes", [
    [33, 128, 257],                                             # recurrences in registers of workgroups (general path: one, streamed)
    [513, 640],                                                 # ... of several (general path: a launch per step)
    [96] * 192,                                                 # a full batch
])
def test_roots_do_not_depend_on_the_magnitude_of_the_statistics(sizes, power, opts):
    # squares of entries below 1e-19 and above 1e19 lie outside fp32; powers of 16 scale the root by a power of two
    o = None if opts is None else ast.RootOpts(**opts)
    for packed in (False, True):
        As = [_with_spectrum(n, _spectrum("power", n), 7, n) for n in sizes]
        if packed and len(As) > 3:
            continue
        got = []
        for s in (1.0, 2.0 ** power):
            Bs = [A * s for A in As]
            Xs = [torch.full_like(A, float("nan")) for A in As]
            lam = torch.zeros(len(As), device=DEV)
            info = torch.full((len(As),), -1, dtype=torch.int32, device=DEV)
            if packed:
                Ps = [torch.empty(ast.packed_elems(n), device=DEV) for n in sizes]
                ast.sym_pack(list(zip(Bs, Ps)))
            ast.inverse_root([(b, x, 1 if packed else 0) for b, x in zip(Ps if packed else Bs, Xs)], 1e-6, opts=o, info=info, lambda_max=lam)
            torch.cuda.synchronize()
            assert bool((info == 0).all()), (s, info)
            got.append((Xs, lam.double() / s))
        assert float(((got[1][1] - got[0][1]) / got[0][1]).abs().max()) <= 1e-6
        for x0, x1 in zip(got[0][0], got[1][0]):
            x1 = x1.double() * 2.0 ** (power // 4)
            # the same operations on scaled numbers: what the scale itself rounds (pow, the power of two for fp16) remains
            assert float(torch.linalg.norm(x1 - x0.double()) / torch.linalg.norm(x0.double())) <= 1e-6


def _largest_ritz_value(A, steps):
    """After `steps` Lanczos steps in fp64 from the library's start vector."""
    n = A.shape[0]
    x = (np.arange(n, dtype=np.uint64) * 0x9E3779B1 + 0x165667B1) & 0xFFFFFFFF
    x ^= x >> np.uint64(15); x = x * 0x2C1B3C6D & 0xFFFFFFFF; x ^= x >> np.uint64(12); x = x * 0x297A2D39 & 0xFFFFFFFF; x ^= x >> np.uint64(15)
    v = torch.from_numpy((x >> np.uint64(8)).astype(np.float64) / 8388608.0 - 1.0).to(DEV)
    v, prev, beta, a, b = v / v.norm(), torch.zeros_like(v), 0.0, [], []
    for _ in range(steps):
        w = A.double() @ v
        a.append(float(w @ v))
        w = w - a[-1] * v - beta * prev
        beta = float(w.norm())
        b.append(beta)
        prev, v = v, w / beta
    return float(np.linalg.eigvalsh(np.diag(a) + np.diag(b[:-1], 1) + np.diag(b[:-1], -1))[-1])


@pytest.mark.parametrize("opts", [dict(), dict(lowp_from=40)])
@pytest.mark.parametrize("steps", [1, 2, 32, 33])
@pytest.mark.parametrize("n", [256, 257, 512, 513, 2047, 2048, 8193])
def test_roots_with_a_bound_on_the_steps_of_the_largest_eigenvalue(n, steps, opts):
    if n > 4096 and (opts or steps == 33):
        pytest.skip("one size of this path is enough")
    # spectrum in about [0.9, 1]: an estimate from one step is 5 % low at most, which the interval covers
    g = torch.Generator(device=DEV).manual_seed(n)
    A = torch.randn(n, n, generator=g, device=DEV)
    A = 0.95 * torch.eye(n, device=DEV) + (0.05 / (2.0 * (2.0 * n) ** 0.5)) * (A + A.T)
    X = torch.full_like(A, float("nan"))
    lam = torch.zeros(1, device=DEV)
    info = torch.full((1,), -1, dtype=torch.int32, device=DEV)
    o = ast.RootOpts(power_iters=steps, power_tol=1e-30, **opts)
    ws = torch.full((ast.inverse_root_workspace_bytes([(A, X)], o)[0],), 255, dtype=torch.uint8, device=DEV)   # NaN in every format
    ast.inverse_root([(A, X)], 1e-6, opts=o, info=info, lambda_max=lam, ws=ws)
    torch.cuda.synchronize()
    assert int(info[0]) == 0
    want = _largest_ritz_value(A, steps)
    # fp32 sums of n terms in A v and v^T A v
    assert abs(float(lam[0]) - want) <= 1e-5 * want, (float(lam[0]), want)
    Y = X.double()
    Y = Y @ Y
    E = Y @ Y @ (A.double() + 1e-6 * float(lam[0]) * torch.eye(n, device=DEV, dtype=torch.float64)) - torch.eye(n, device=DEV, dtype=torch.float64)
    assert float(torch.linalg.norm(E)) / n ** 0.5 <= 4 * 2e-3       # four factors of the accuracy of the root


@pytest.mark.parametrize("eps", [1e-3, 1e-6, 1e-8])
@pytest.mark.parametrize("opts", [None, dict(int8_slices=0), dict(int8_slices=4), dict(fp64_iters=0), dict(lowp_from=40)])
@pytest.mark.parametrize("n", [1, 2, 33, 129, 513, 1025])
def test_roots_stay_inside_the_smallest_workspace_and_do_not_depend_on_its_size(n, opts, eps):
    o = None if opts is None else ast.RootOpts(**opts)
    A = _with_spectrum(n, _spectrum("power", n), 7, n)
    got = []
    for copies in (1, 3):                                       # three factors in one pass, and one after the other
        Xs = [torch.full_like(A, float("nan")) for _ in range(3)]
        items = [(A, X) for X in Xs]
        full, least = ast.inverse_root_workspace_bytes(items, o)
        size = least if copies == 1 else full
        assert full > least
        buf = torch.full((size + (1 << 20),), 255, dtype=torch.uint8, device=DEV)
        info = torch.full((3,), -1, dtype=torch.int32, device=DEV)
        ast.inverse_root(items, eps, opts=o, info=info, ws=buf[:size])
        torch.cuda.synchronize()
        assert bool((info == 0).all()) and bool((buf[size:] == 255).all())
        got += Xs
    assert all(torch.equal(got[0], X) for X in got[1:])


@pytest.mark.parametrize("count", [1, 5, 28, 60])      # the tables of a call share the pieces they are uploaded in
def test_batches_of_mixed_blocks_agree_with_single_calls(count):
    g = torch.Generator(device=DEV).manual_seed(count)
    items, single = [], []
    for i in range(count):
        m, n = 8 + i, 40 - i % 9
        XL, XR, G = (torch.randn(a, b, generator=g, device=DEV) for a, b in ((m, m), (n, n), (m, n)))
        G = G.bfloat16() if i % 3 else G
        items.append((XL, G, XR, torch.empty(m, n, device=DEV)))
        single.append(torch.empty(m, n, device=DEV))
    ast.precondition(items)
    for it, P in zip(items, single):
        ast.precondition([(*it[:3], P)])
    torch.cuda.synchronize()
    for it, P in zip(items, single):
        assert torch.equal(it[3], P)


# sorted refresh: the columns' order where the ranks of one group of lanes end and the next begin
@pytest.mark.parametrize("n", [1, 15, 16, 17, 130, 257])
def test_order_of_the_sorted_refresh(n):
    lam = torch.arange(1, n + 1, device=DEV, dtype=torch.float32)
    lam[: n // 2] = lam[n // 2]                        # ties: by index
    shuffle = torch.randperm(n, generator=torch.Generator().manual_seed(n)).to(DEV)
    A, Q = torch.diag(lam[shuffle]), torch.eye(n, device=DEV)
    perm = [torch.full((n,), -1, dtype=torch.int32, device=DEV)]
    ast.soap_refresh([(A, Q)], sort=True, perm=perm[0])
    torch.cuda.synchronize()
    assert torch.equal(perm[0].long(), torch.sort(-lam[shuffle], stable=True).indices)


# sorted refresh of statistics that are not finite: reported, in an order that still is one, beside factors that are
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_order_of_the_sorted_refresh_with_estimates_that_are_no_numbers(bad):
    sizes = [257, 130, 256, 16, 130, 1]
    As = [_with_spectrum(n, _spectrum("power", n) + 1e-4, 9, n) if n > 1 else torch.ones(1, 1, device=DEV) for n in sizes]
    As[1][5, 5] = bad                                  # one element: every column of A Q
    As[2][:] = bad
    As[3][2, 2] = bad
    Q = [W.haar(n, DEV, 11, n) if n != 16 else torch.eye(16, device=DEV) for n in sizes]     # identity: one column of A Q only
    alone = [q.clone() for q in Q]
    info = torch.full((len(sizes),), -1, dtype=torch.int32, device=DEV)
    perm = torch.full((sum(sizes),), -1, dtype=torch.int32, device=DEV)
    ast.soap_refresh(list(zip(As, Q)), info=info, sort=True, perm=perm)
    ast.soap_refresh([(As[0], alone[0])], sort=True)
    torch.cuda.synchronize()
    assert [int(i != 0) for i in info] == [0, 1, 1, 1, 0, 0]
    for n, p in zip(sizes, perm.split(sizes)):
        assert torch.equal(p.long().sort().values, torch.arange(n, device=DEV)), n
    assert torch.equal(Q[0], alone[0])
