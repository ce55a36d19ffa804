"""Sizes at the borders of the kernels' splits: tile edges, remainders, and both
sides of the rules that pick a variant by size, against float64."""
import math
import os

import numpy as np
import pytest
import torch

import oracle
from tests import test_gpu_edges as edges
from tests.gpu_common import certify_flips, gpu_assignment, np64

pytestmark = pytest.mark.gpu

S128 = 1.0 / math.sqrt(128)
DT = {"f32": torch.float32, "bf16": torch.bfloat16}


def A():
    from paper_2609_36835_amd import arckv
    return arckv


def randn(seed, *shape, dtype=torch.float32):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(*shape, generator=g, device="cuda").to(dtype)


# (pairs, queries, compact keys, shift of z).  256-wide Cholesky panels with 64-wide
# blocks and 16-wide tile columns; 48 pairs of t = 1024 are past the rules for few
# strips (256 of 64 rows), few block inverses (64), and few rows of the
# 128-column solves (512 chunks); 100 pairs of t = 1025 update three chunks of 64
# per workgroup in the one-rhs solves.  A shift of 40 puts every pivot below 2^-96.
FITS = [(1, 16, 1, 0), (2, 63, 15, 0), (2, 200, 64, 0), (2, 300, 65, 0), (1, 600, 255, 0), (1, 600, 256, 0),
        (2, 700, 257, 0), (1, 1100, 513, 0), (1, 300, 100, 40), (48, 1300, 1024, 0), (100, 1300, 1025, 0)]
# pairs whose 128-column solves are left-looking, and one short of them
MANY_PAIRS = [(256, 40, 1), (122, 300, 65), (254, 700, 257), (162, 2200, 2049), (64, 700, 513), (66, 700, 513)]


@pytest.mark.parametrize("B,n,t,shift", FITS)
def test_mass_fit_sizes(B, n, t, shift):
    """The masses are those of known weights.  The fp32 evaluation of Phi_C (logits up to
    about 5 in size, one exponential) is off by at most 3e-6 relative, which moves a
    least-squares solution by at most twice cond(Phi_C) times that; the ridge is in the
    reference."""
    P = min(B, 2)
    print(f"mass fit B={B} n={n} t={t} shift={shift}", flush=True)
    Q, Ck = randn(1, P, n, 128), randn(2, P, t, 128)
    w = 0.5 + 1.5 * torch.rand(P, t, device="cuda", dtype=torch.float64)
    Phi = [torch.exp(q.double() @ c.double().T * S128 - shift) for q, c in zip(Q, Ck)]
    m = torch.stack([p @ x for p, x in zip(Phi, w)]).float()
    z = torch.full((P, n), float(shift), device="cuda")
    rep = lambda x: x.repeat(B // P, *[1] * (x.dim() - 1)).contiguous()
    beta, info, dused = A().fit_bias(rep(Q), rep(Ck), rep(z), rep(m), A().default_params(b_min=-30.0), scale=S128, T=4 * t)
    assert torch.all(info == 0) and torch.all(torch.isfinite(beta))
    sv = [torch.linalg.svdvals(p) for p in Phi]
    for b in range(B):
        p = Phi[b % P]
        G = p.T @ p
        G.diagonal().add_(float(dused[b]) * float(G.diagonal().mean()))
        ref = torch.linalg.solve(G, p.T @ m[b % P].double())
        tol = 6e-6 * float(sv[b % P][0] / sv[b % P][-1])
        err = float((torch.exp(beta[b].double()) - ref).norm() / ref.norm())
        assert err <= tol, (b, err, tol)


def test_mass_fit_nearly_square():
    """The biases of a nearly square system depend on the form of the solves beneath the
    refinement; these are those of solves by 64 x 64 diagonal inverses, to two units in the last
    place of the largest (256 x 256 inverses: five)."""
    print("mass fit nearly square", flush=True)
    n, t = 520, 500
    rng = np.random.default_rng(n * 1000 + t)
    f = lambda x: torch.from_numpy(x.astype(np.float32)).cuda()
    Q, C = f(rng.standard_normal((1, n, 128))), f(rng.standard_normal((1, t, 128)))
    m, z = f(rng.random((1, n)) * t), f(rng.random((1, n)))
    beta, info, _ = A().fit_bias(Q, C, 2.0 * z, m, A().default_params(b_min=-6.0), T=4 * t)
    ref = np.loadtxt(os.path.join(os.path.dirname(__file__), "golden", "mass_fit_520_500.txt"))
    assert int(info[0]) == 0
    assert np.abs(np64(beta)[0] - ref).max() <= 2.0 ** -20


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,n,t", [f[:3] for f in FITS if f[3] == 0] + MANY_PAIRS)
def test_value_fit_sizes(B, n, t, dtype):
    """The fitted block's outputs on the queries against the float64 fit at the same ridge, at
    the fp32 bar of the parity tests (compact keys and operands enter as split planes)."""
    P = min(B, 2)
    print(f"value fit {dtype} B={B} n={n} t={t}", flush=True)
    Q, Ck, Y = randn(3, P, n, 128, dtype=DT[dtype]), randn(4, P, t, 128), randn(5, P, n, 128)
    beta = 0.5 * randn(6, P, t)
    rep = lambda x: x.repeat(B // P, 1, 1).contiguous() if x.dim() == 3 else x.repeat(B // P, 1).contiguous()
    Cv, info, dused = A().fit_values(rep(Q), rep(Ck), rep(beta), rep(Y), scale=S128, T=4 * t)
    assert torch.all(info == 0)
    for b in range(B):
        p = torch.softmax(Q[b % P].double() @ Ck[b % P].double().T * S128 + beta[b % P].double(), dim=1)
        M = p.T @ p
        M.diagonal().add_(float(dused[b]) * float(M.diagonal().mean()))
        ref = p @ torch.linalg.solve(M, p.T @ Y[b % P].double())
        err = float(((p @ Cv[b].double() - ref).norm(dim=1) / ref.norm(dim=1)).max())
        assert err <= 1e-4, (b, err)


def chunked(call, B, chunks):
    """call(params) once whole and in chunks of pairs: the same bits."""
    whole = [x.clone() for x in call(pair_chunk=0)]
    for c in chunks:
        assert c < B
        for x, y in zip(whole, call(pair_chunk=c)):
            assert torch.equal(x, y), c


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,n,t", [(130, 200, 65), (70, 900, 600), (66, 1100, 1025)])
def test_value_fit_chunks(B, n, t, dtype):
    """Chunks on both sides of the rules for many pairs: the 128-column solves, the small
    tiles of the contractions and of the factorisation."""
    print(f"value fit chunks {dtype} B={B} n={n} t={t}", flush=True)
    Q, Ck, Y = randn(31, B, n, 128, dtype=DT[dtype]), randn(32, B, t, 128), randn(33, B, n, 128)
    beta = 0.5 * randn(34, B, t)
    chunked(lambda **kw: A().fit_values(Q, Ck, beta, Y, A().default_params(**kw), scale=S128, T=4 * t), B, (1, 33, 65))


def test_value_fit_bad_pairs_among_many():
    """Pairs with non-finite inputs in a left-looking call: NaN values, and the others' bits stay."""
    print("value fit bad pairs", flush=True)
    B, n, t = 70, 700, 513
    Q, Ck, Y, beta = randn(57, B, n, 128), randn(58, B, t, 128), randn(59, B, n, 128), 0.5 * randn(60, B, t)
    good = A().fit_values(Q, Ck, beta, Y, scale=S128, T=4 * t)[0]
    bad = [0, 33, B - 1]
    for b in bad:
        Y[b, 7, 5] = math.nan
    Cv, info, _ = A().fit_values(Q, Ck, beta, Y, scale=S128, T=4 * t)
    rest = [b for b in range(B) if b not in bad]
    assert torch.all(info[bad] == -1) and torch.all(torch.isnan(Cv[bad]))
    assert torch.all(info[rest] == 0) and torch.equal(Cv[rest], good[rest])


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("B,n,t", [(130, 520, 500), (66, 300, 250)])
def test_mass_fit_chunks(B, n, t, mode):
    """Unrefined weights of nearly square systems show a rounding of h = Phi_C^T m, whose
    sum over the queries is cut into ranges."""
    print(f"mass fit chunks B={B} n={n} t={t} mode={mode}", flush=True)
    Q, Ck = randn(35, B, n, 128), randn(36, B, t, 128)
    z, m = torch.full((B, n), 2.0, device="cuda"), t * torch.rand(B, n, device="cuda")
    chunked(lambda **kw: A().fit_bias(Q, Ck, z, m, A().default_params(refine_steps=0, bias_mode=mode, **kw), scale=S128,
                                      T=4 * t), B, (1, 10, 60))


def test_dsa_chunks():
    """The value head's row statistics go by the pairs of the call, not of the chunk."""
    print("dsa chunks", flush=True)
    B, T, n, dx = 136, 200, 64, 256
    bf = lambda i, *sh: randn(i, B, *sh, dtype=torch.bfloat16)
    K, V, Q = bf(44, T, 128), bf(45, T, 128), bf(46, n, 128)
    p = {k: bf(47 + i, 1024, 128) / 11 for i, k in enumerate(("L_q", "L_k", "L_c", "L_v"))}
    p.update({k: bf(51 + i, 128, 128) / 11 for i, k in enumerate(("U_q", "U_k", "U_v"))})
    p.update(L_x=bf(54, 8, dx) / 16, b_x=0.1 * randn(55, B, 8))
    X = bf(56, n, dx)
    chunked(lambda pair_chunk: [A().score_dsa(K, V, Q, X, p, n, pair_chunk=pair_chunk)], B, (8, 64))


def test_merge_chunks():
    """The anchors' norms are cut into query ranges by the pairs of the call, not of the chunk."""
    print("merge chunks", flush=True)
    B, T, n, t = 70, 1500, 700, 200
    K, V, Q = randn(37, B, T, 128, dtype=torch.bfloat16), randn(38, B, T, 128, dtype=torch.bfloat16), \
        randn(39, B, n, 128, dtype=torch.bfloat16)
    W1, b1, w2, b2 = randn(40, B, 64, 256, dtype=torch.bfloat16) / 16, randn(41, B, 64), randn(42, B, 64) / 8, randn(43, B)
    chunked(lambda **kw: A().compact(K, V, Q, W1, b1, w2, b2, t / T, scale=S128, params=A().default_params(**kw)), B,
            (1, 12, 64))


@pytest.mark.parametrize("B,n", [(2, 130), (33, 130), (129, 130)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T", [1, 63, 64, 65, 129, 1000])
def test_rowstats_sizes(T, dtype, B, n):
    """Up to 128 tiles of 256 queries (fp32: 64 of 128): key halves inside a workgroup (a wave per
    key range); more: whole tiles of keys per wave.  z and m to fp32 sums; bf16 inputs round the
    probabilities of Y's product to 2^-8."""
    print(f"rowstats {dtype} T={T} B={B} n={n}", flush=True)
    K, V, Q = (randn(i, B, k, 128, dtype=DT[dtype]) for i, k in ((7, T), (8, T), (9, n)))
    z, m, Y = A().rowstats(K, V, Q, scale=S128)
    for b in (0, B - 1):
        L = Q[b].double() @ K[b].double().T * S128
        zr = L.amax(dim=1)
        E = torch.exp(L - zr[:, None])
        Yr = (E @ V[b].double()) / E.sum(dim=1, keepdim=True)
        assert float((z[b] - zr).abs().max()) <= 1e-5
        assert float((m[b] / E.sum(dim=1) - 1).abs().max()) <= 2e-5
        assert float((Y[b] - Yr).abs().max()) <= (2e-5 if dtype == "f32" else 2.0 ** -8) * float(V[b].float().abs().max())


@pytest.mark.parametrize("T", [40, 64, 130, 200])
def test_rowstats_alone_and_in_a_batch(T):
    """A pair alone takes the form that splits the keys, in a batch of 65 the other; both round the
    same probabilities to bf16, so they differ by the order of fp32 sums of T terms."""
    print(f"rowstats alone and in a batch T={T}", flush=True)
    K, V, Q = (randn(i, 65, k, 128, dtype=torch.bfloat16) for i, k in ((22, T), (23, T), (24, 300)))
    z, m, Y = A().rowstats(K, V, Q, scale=S128)
    for b in (0, 64):
        z1, m1, Y1 = A().rowstats(*(x[b:b + 1].contiguous() for x in (K, V, Q)), scale=S128)
        assert torch.equal(z1[0], z[b])
        assert float((m1[0] / m[b] - 1).abs().max()) <= 2 * T * 2.0 ** -24
        assert float((Y1[0] - Y[b]).abs().max()) <= 2 * T * 2.0 ** -24 * float(V[b].float().abs().max())


@pytest.mark.parametrize("B,T", [(1, 1), (1, 15), (2, 17), (3, 1000), (9, 4099), (9, 8001)])
def test_score_f32_sizes(B, T):
    """16 or 64 tokens per step, one step or four.  The bound is that of sums of 256 and 64 fp32 terms in any order."""
    print(f"score f32 B={B} T={T}", flush=True)
    K, V = randn(10, B, T, 128), randn(11, B, T, 128)
    W1, b1, w2, b2 = randn(12, B, 64, 256) / 16, randn(13, B, 64), randn(14, B, 64) / 8, randn(15, B)
    out = A().score(K, V, W1, b1, w2, b2)
    for b in range(B):
        X = torch.cat([K[b], V[b]], dim=1).double()
        x = X @ W1[b].double().T + b1[b].double()
        h = 0.5 * x * (1.0 + torch.erf(x / math.sqrt(2.0)))
        ref = h @ w2[b].double() + b2[b].double()
        e = 2.0 ** -24
        eh = 260 * e * (X.abs() @ W1[b].double().abs().T + b1[b].double().abs()) * 1.13 + 8 * e * h.abs() + 1e-7
        bound = (eh + 66 * e * h.abs()) @ w2[b].double().abs() + 66 * e * b2[b].double().abs()
        assert torch.all((out[b].double() - ref).abs() <= bound)


@pytest.mark.parametrize("t", [1, 2048, 2049, 4097, 8193])
def test_group_sort_segments(t):
    """16, 8, 4 and 2 segments of the positions (their counters fill 32,768 words of LDS)."""
    print(f"merge t={t}", flush=True)
    edges.test_merge_many_groups(t)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", [1, 127, 128, 129, 257, 520, 1921, 2600])
def test_assignment_query_ranges(n, dtype):
    """Anchors in close pairs, so that keys are refined and decided in float64, over query
    counts on both sides of the ranges' tiles; kappa is the float64 argmax."""
    print(f"assignment {dtype} n={n}", flush=True)
    rng = np.random.default_rng(n)
    T, t = 600, 40
    K = rng.standard_normal((T, 128)).astype(np.float32)
    S = np.sort(rng.choice(T, t, replace=False))
    K[S[1::2]] = K[S[::2]] * (1.0 + 2.0 ** -6)
    Kd, Qd = (torch.from_numpy(x).to(DT[dtype]) for x in (K, rng.standard_normal((n, 128)).astype(np.float32)))
    kap, st = gpu_assignment(Kd[None].cuda(), Kd[None].cuda(), Qd[None].cuda(), torch.from_numpy(S.astype(np.int32))[None].cuda(),
                             S128)
    K64, Q64 = np64(Kd), np64(Qd)
    ref, _, _ = oracle.profiles_assign_phi(Q64, K64, S, S128)
    certify_flips(kap, ref, Q64, K64, S, S128)


@pytest.mark.parametrize("G,t,F", [(1, 1, 0), (2, 31, 0), (4, 33, 37), (8, 256, 1), (4, 0, 70)])
def test_attend_infinite_values(G, t, F):
    """An infinite value stays in its dimension, also in the last row, whose repeats stand in for
    the rows past the end."""
    print(f"attend G={G} t={t} F={F}", flush=True)
    Q, C, X = randn(16, 2, G, 128, dtype=torch.bfloat16), randn(17, 2, t, 128, dtype=torch.bfloat16), \
        randn(18, 2, F, 128, dtype=torch.bfloat16)
    Cv, Xv = randn(19, 2, t, 128, dtype=torch.bfloat16), randn(20, 2, F, 128, dtype=torch.bfloat16)
    beta = randn(21, 2, t)
    none = lambda x: x if x.shape[1] else None
    call = lambda: A().attend(Q, none(C), beta if t else None, none(Cv), none(X), none(Xv), scale=S128)
    plain = call()
    (Xv if F else Cv)[:, -1, 5] = math.inf
    (Cv if t else Xv)[:, 0, 77] = -math.inf
    out = call()
    assert torch.all(out[:, :, 5] == math.inf) and torch.all(out[:, :, 77] == -math.inf)
    keep = [i for i in range(128) if i not in (5, 77)]
    assert torch.equal(out[:, :, keep], plain[:, :, keep])


def test_attend_streamed_values():
    """A call whose keys and values exceed the last-level cache reads the values as a stream; each
    pair's output is that of the pair alone."""
    print("attend streamed", flush=True)
    P, t, F = 130, 4000, 99
    Q, C, Cv = randn(25, P, 4, 128, dtype=torch.bfloat16), randn(26, P, t, 128, dtype=torch.bfloat16), \
        randn(27, P, t, 128, dtype=torch.bfloat16)
    X, Xv, beta = randn(28, P, F, 128, dtype=torch.bfloat16), randn(29, P, F, 128, dtype=torch.bfloat16), randn(30, P, t)
    out = A().attend(Q, C, beta, Cv, X, Xv, scale=S128)
    for b in (0, 77, P - 1):
        one = A().attend(*(x[b:b + 1].contiguous() for x in (Q, C, beta, Cv, X, Xv)), scale=S128)
        assert torch.equal(one[0], out[b])
