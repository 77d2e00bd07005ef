"""GPU parity of the selection front end against the float64 oracle.

project: b and c to the same sum-scaled bar as the logits (S = sum_d |u_d W_d|
of each projected value); the diagonal generator D = sigmoid(a) exp(i theta)
inherits the bars of a and theta through |d sigmoid| <= 1/4 and
|exp(i x) - 1| <= |x|: |gpu - ref| <= tol_a / 4 + tol_theta + 1e-6 per
component (the last term for the fp32 exponential and sine/cosine).

dict_argmax: bit for bit (no arithmetic; ties to the first maximal index).
route: logits within |gpu - ref| <= 1e-5 + 1e-4*S, S = sum_d |u_d S_d| (an
fp32 sum of Dm bf16 products, see helpers.assert_close_sum); idx is exactly
the first argmax of the GPU's own logits, and equals the oracle's choice
wherever the oracle's two best scores are further apart than that bar (where
they are not, the GPU's choice must score within the bar of the best).
"""
import numpy as np
import pytest

from helpers import assert_close_sum, project_rule
from oracle import oracle_dict_argmax, oracle_project, oracle_route

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU machines, never run there
    pytest.skip("no GPU", allow_module_level=True)

from paper_2605_19150_amd import pdssm  # noqa: E402

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("N", [8, 16, 32, 64, 128, 256])
def test_dict_argmax(N):
    rng = np.random.default_rng(N)
    H, K = 3, 5
    M = rng.standard_normal((H, K, N, N)).astype(np.float32)
    M[0, 0] = np.round(M[0, 0])          # many exact ties
    M[1, 2, :, :] = 1.0                  # every column ties everywhere
    pi = pdssm.dict_argmax(torch.from_numpy(M).to(DEV)).cpu().numpy()
    np.testing.assert_array_equal(pi, oracle_dict_argmax(M))


def _bf16(a):
    t = torch.from_numpy(np.ascontiguousarray(a, np.float32)).to(torch.bfloat16)
    return t, t.to(torch.float64).numpy()


def check_route(B, L, H, K, Dm, seed):
    rng = np.random.default_rng(seed)
    ut, u = _bf16(rng.standard_normal((B, L, Dm)))
    St, S = _bf16(rng.standard_normal((H, K, Dm)) / np.sqrt(Dm))
    logits, idx = pdssm.route(ut.to(DEV), St.to(DEV))
    lg, ix = logits.cpu().numpy(), idx.cpu().numpy()
    rl, ri = oracle_route(u, S)
    scale = np.einsum("bld,hkd->blhk", np.abs(u), np.abs(S))
    assert_close_sum("logits", lg, rl, scale)
    np.testing.assert_array_equal(ix, np.argmax(lg, axis=3))          # first argmax of its own logits
    tol = 1e-5 + 1e-4 * scale.max(axis=3)
    top2 = np.sort(rl, axis=3)[..., -2:] if K > 1 else np.concatenate([rl, rl - 1], axis=3)
    clear = (top2[..., 1] - top2[..., 0]) > 2 * tol
    np.testing.assert_array_equal(ix[clear], ri[clear])
    chosen = np.take_along_axis(rl, ix[..., None].astype(np.int64), axis=3)[..., 0]
    assert (rl.max(axis=3) - chosen <= 2 * tol).all()
    _, idx2 = pdssm.route(ut.to(DEV), St.to(DEV), logits=False)
    np.testing.assert_array_equal(idx2.cpu().numpy(), ix)
    return clear.mean()


@pytest.mark.parametrize("B,L,H,K,Dm", [
    (2, 100, 16, 16, 1024),   # a fsa-perm-like layer: 16 heads x 16 maps, d = 1024
    (1, 70, 7, 5, 72),        # ragged: tokens, heads per tile, contraction tail
    (1, 65, 32, 64, 256),     # 4 heads per tile
    (2, 33, 2, 256, 64),      # one head per tile
    (1, 1, 1, 1, 8),          # smallest
    (3, 50, 300, 3, 16),      # many head groups
    (8, 2048, 32, 64, 64),    # 256-token tiles, 512 of them, two slices of the contraction
    (1, 18693, 28, 64, 32),   # 256-token tiles, a ragged last one, a tile count not a multiple of 8
])
def test_route(B, L, H, K, Dm):
    print("route B=%d L=%d H=%d K=%d Dm=%d" % (B, L, H, K, Dm), flush=True)
    frac = check_route(B, L, H, K, Dm, seed=B + L + H + K + Dm)
    assert frac > 0.9 or K == 1


def test_route_full_size():
    """fsa-perm routing: B16 L2048, 16 heads x 16 maps, d = 1024."""
    frac = check_route(16, 2048, 16, 16, 1024, seed=0)
    assert frac > 0.99


def test_route_hybrid_full_size_sampled():
    """hybrid-lm routing: B8 L4096 (32768 tokens), 32 heads x 64 maps, d = 4096;
    logits and choices of sampled tokens against the oracle."""
    rng = np.random.default_rng(3)
    B, L, H, K, Dm = 8, 4096, 32, 64, 4096
    ut = torch.from_numpy(rng.standard_normal((B, L, Dm), dtype=np.float32)).to(torch.bfloat16)
    St = torch.from_numpy(rng.standard_normal((H, K, Dm), dtype=np.float32) / np.float32(np.sqrt(Dm))).to(
        torch.bfloat16)
    logits, idx = pdssm.route(ut.to(DEV), St.to(DEV))
    rows = np.sort(rng.choice(B * L, size=96, replace=False))
    u = ut.reshape(B * L, Dm)[rows].to(torch.float64).numpy()[None]
    S = St.to(torch.float64).numpy()
    lg = logits.reshape(B * L, H, K)[rows].cpu().numpy()[None]
    ix = idx.reshape(B * L, H)[rows].cpu().numpy()[None]
    rl, ri = oracle_route(u, S)
    scale = np.einsum("bld,hkd->blhk", np.abs(u), np.abs(S))
    assert_close_sum("logits", lg, rl, scale)
    np.testing.assert_array_equal(ix, np.argmax(lg, axis=3))
    tol = 1e-5 + 1e-4 * scale.max(axis=3)
    top2 = np.sort(rl, axis=3)[..., -2:]
    clear = (top2[..., 1] - top2[..., 0]) > 2 * tol
    np.testing.assert_array_equal(ix[clear], ri[clear])
    assert clear.mean() > 0.9


def _check_project(u, S, W, got, rows=None):
    """got: pdssm.project's outputs (rows: the token rows of u they cover)."""
    Wb, Wc, Wd = W
    ref = oracle_project(u, S, Wb, Wc, Wd)
    au = np.abs(u)
    for name, w in (("b", Wb), ("c", Wc)):
        if w is None:
            continue
        sc = np.einsum("bld,hrd->blhr", au, np.abs(w))
        g = got[name]
        assert_close_sum(name + ".re", g.real, ref[name].real, sc[..., 0::2])
        assert_close_sum(name + ".im", g.imag, ref[name].imag, sc[..., 1::2])
    if Wd is not None:
        sc = np.einsum("bld,hrd->blhr", au, np.abs(Wd))
        tol = (1e-5 + 1e-4 * sc[..., 0::2]) / 4 + (1e-5 + 1e-4 * sc[..., 1::2]) + 1e-6
        g, r = got["D"], ref["D"]
        for part, gp, rp in (("re", g.real, r.real), ("im", g.imag, r.imag)):
            err = np.abs(gp.astype(np.float64) - rp)
            bad = err > tol
            assert not bad.any(), "D.%s: %d out of tolerance, worst %g (tol %g)" % (
                part, bad.sum(), err.max(), tol[np.unravel_index(np.argmax(err - tol), err.shape)])
        assert (np.abs(g) < 1 + 1e-6).all()
    if S is not None:
        lg, ix = got["logits"], got["idx"]
        scale = np.einsum("bld,hkd->blhk", au, np.abs(S))
        assert_close_sum("logits", lg, ref["logits"], scale)
        np.testing.assert_array_equal(ix, np.argmax(lg, axis=3))


def _proj_case(B, L, H, K, N, Dm, seed, kinds="Sbcd"):
    rng = np.random.default_rng(seed)
    ut, u = _bf16(rng.standard_normal((B, L, Dm)))
    S = W = None
    St, S = _bf16(rng.standard_normal((H, K, Dm)) / np.sqrt(Dm)) if "S" in kinds else (None, None)
    Ws, Wt = [], []
    for kch, scale in (("b", 1.0), ("c", 1.0), ("d", 2.0)):
        if kch in kinds:
            t, w = _bf16(rng.standard_normal((H, 2 * N, Dm)) * scale / np.sqrt(Dm))
            Wt.append(t.to(DEV))
            Ws.append(w)
        else:
            Wt.append(None)
            Ws.append(None)
    out = pdssm.project(ut.to(DEV), St.to(DEV) if St is not None else None, *Wt, N=N)
    got = {k: v.cpu().numpy() for k, v in out.items() if v is not None}
    _check_project(u, S, Ws, got)


@pytest.mark.parametrize("B,L,H,K,N,Dm,kinds", [
    (2, 100, 16, 16, 64, 1024, "Sbcd"),   # a fsa-perm-like layer
    (1, 70, 3, 5, 8, 64, "Sbcd"),         # ragged tokens, a partial column tile (H*2N = 48), K % 4 != 0
    (1, 300, 2, 7, 256, 96, "Sbcd"),      # N = 256: four column tiles per projection, three slices
    (3, 50, 5, 1, 32, 32, "bcd"),         # no routing; H*2N = 320: one whole and one partial tile
    (8, 2048, 4, 16, 128, 64, "Sbcd"),    # 256-token tiles
    (2, 77, 6, 9, 16, 128, "b"),          # one projection alone
    (2, 77, 6, 9, 16, 128, "d"),
    (2, 77, 6, 9, 16, 128, "Sc"),
])
def test_project(B, L, H, K, N, Dm, kinds):
    print("project B=%d L=%d H=%d K=%d N=%d Dm=%d %s" % (B, L, H, K, N, Dm, kinds), flush=True)
    _proj_case(B, L, H, K, N, Dm, seed=B * L + H + K + N + Dm, kinds=kinds)


@pytest.mark.parametrize("B,L,H,K,N,Dm", [(16, 2048, 16, 16, 64, 1024), (8, 4096, 32, 64, 128, 4096)])
def test_project_layer_full_size_sampled(B, L, H, K, N, Dm):
    """The layers of fsa-perm (d = 1024, 16 heads of 64) and hybrid-lm (d =
    4096, 32 heads of 128) at full size; routing, b, c and D of sampled
    tokens against the oracle."""
    print("project layer B=%d L=%d H=%d K=%d N=%d Dm=%d" % (B, L, H, K, N, Dm), flush=True)
    g = torch.Generator(device="cpu").manual_seed(B + Dm)
    ut = torch.randn((B, L, Dm), generator=g).to(torch.bfloat16)
    St = (torch.randn((H, K, Dm), generator=g) / Dm ** 0.5).to(torch.bfloat16)
    Wt = [(torch.randn((H, 2 * N, Dm), generator=g) * s / Dm ** 0.5).to(torch.bfloat16) for s in (1.0, 1.0, 2.0)]
    out = pdssm.project(ut.to(DEV), St.to(DEV), *[w.to(DEV) for w in Wt])
    rows = np.sort(np.random.default_rng(1).choice(B * L, size=64, replace=False))
    u = ut.reshape(B * L, Dm)[rows].to(torch.float64).numpy()[None]
    got = {k: v.reshape((B * L,) + v.shape[2:])[rows].cpu().numpy()[None] for k, v in out.items()}
    _check_project(u, St.to(torch.float64).numpy(), [w.to(torch.float64).numpy() for w in Wt], got)


@pytest.mark.parametrize("B,L,H,K,N,Dm,kinds,kernel", [
    (9, 3333, 31, 5, 8, 32, "Sbcd", "dma256"),      # two partial routing halves, H*2N = 496
    (9, 3333, 31, 5, 8, 64, "Sbcd", "dma256"),
    (9, 3333, 31, 5, 32, 32, "Sbcd", "wide"),       # one half slice, two partial routing halves, H*2N = 1984
    (9, 3333, 31, 5, 32, 64, "Sbcd", "wide"),       # one whole slice
    (2, 7001, 33, 2, 32, 96, "Sbcd", "wide"),       # a half tail slice, a ragged last token tile
    (1, 16385, 13, 37, 16, 160, "Sbcd", "dma256"),  # K % 4 != 0, one token in the last tile
    (1, 18817, 13, 7, 16, 160, "Sbcd", "wide"),     # K % 4 != 0, one token in the last block
    (4, 4100, 3, 200, 256, 64, "Sbcd", "dma256"),
    (4, 4100, 3, 200, 256, 192, "Sbcd", "wide"),    # a head over both halves of its tile
    (4, 4100, 3, 130, 256, 192, "Sbcd", "wide"),    # the same, K % 4 != 0
    (3, 11000, 9, 1, 64, 288, "bd", "wide"),        # no routing, two projections
    (2, 16390, 5, 128, 128, 1056, "Sbcd", "wide"),
])
def test_project_large_tiles(B, L, H, K, N, Dm, kinds, kernel):
    """256-token tiles (512 of them and more): sampled rows, the first and last
    among them, and every row of the last token tile."""
    print("project B=%d L=%d H=%d K=%d N=%d Dm=%d %s" % (B, L, H, K, N, Dm, kinds), flush=True)
    assert project_rule().kernel(B * L, Dm, H, K, N, "S" in kinds, len(kinds.replace("S", ""))) == kernel
    T = B * L
    g = torch.Generator().manual_seed(T + Dm)
    ut = torch.randn((B, L, Dm), generator=g).bfloat16()
    St = (torch.randn((H, K, Dm), generator=g) / Dm ** 0.5).bfloat16() if "S" in kinds else None
    Wt = [(torch.randn((H, 2 * N, Dm), generator=g) * s / Dm ** 0.5).bfloat16() if k in kinds else None
          for k, s in (("b", 1.0), ("c", 1.0), ("d", 2.0))]
    out = pdssm.project(ut.to(DEV), St.to(DEV) if St is not None else None,
                        *[w.to(DEV) if w is not None else None for w in Wt], N=N)
    rng = np.random.default_rng(2)
    rows = np.unique(np.concatenate([[0, 127, 128, 255, T - 1], np.arange(T - T % 256, T),
                                     rng.choice(T, size=128, replace=False)]))
    u = ut.reshape(T, Dm)[rows].double().numpy()[None]
    got = {k: v.reshape((T,) + v.shape[2:])[rows].cpu().numpy()[None] for k, v in out.items()}
    _check_project(u, St.double().numpy() if St is not None else None,
                   [w.double().numpy() if w is not None else None for w in Wt], got)


@pytest.mark.parametrize("T,H,K,N,Dm", [
    (18817, 5, 7, 32, 64),     # one token in the last block; H*2N = 320: the last tile's second half is empty
    (32513, 1, 16, 32, 128),   # the same with H*2N = 64
    (18817, 17, 3, 8, 192),    # H*2N = 272
    (32899, 5, 3, 8, 128),     # three tokens; H*2N = 80: rows shorter than a block is wide
])
def test_project_empty_half_tile(T, H, K, N, Dm):
    """256 x 256 tiles whose second column half lies past the last column, with
    few tokens in the last block: every row of it, and the outputs' last rows
    whole."""
    print("project T=%d H=%d K=%d N=%d Dm=%d" % (T, H, K, N, Dm), flush=True)
    assert project_rule().kernel(T, Dm, H, K, N) == "wide"
    assert 0 < T % 128 < 8 and 0 < 2 * H * N % 256 < 128
    g = torch.Generator().manual_seed(T)
    ut = torch.randn((1, T, Dm), generator=g).bfloat16()
    St = (torch.randn((H, K, Dm), generator=g) / Dm ** 0.5).bfloat16()
    Wt = [(torch.randn((H, 2 * N, Dm), generator=g) / Dm ** 0.5).bfloat16() for _ in range(3)]
    out = pdssm.project(ut.to(DEV), St.to(DEV), *[w.to(DEV) for w in Wt])
    rows = np.concatenate([[0, 127, 128], np.arange(T - T % 128 - 2, T)])
    got = {k: v[:, rows].cpu().numpy() for k, v in out.items()}
    _check_project(ut[:, rows].double().numpy(), St.double().numpy(), [w.double().numpy() for w in Wt], got)


@pytest.mark.parametrize("T", [300, 33000])
def test_project_generator_range(T):
    """D where magnitude logits and phases leave the fast generator's range
    (|m| >= 80, |p| >= 8192), in both tile sizes: the diagonal computed in 64
    bits from the logits and phases that b's weights give for the same rows."""
    H, N, Dm = 4, 128, 32
    g = torch.Generator().manual_seed(T)
    u = torch.randn((1, T, Dm), generator=g).bfloat16().to(DEV)
    W = torch.randn((H, 2 * N, Dm), generator=g)
    W[1, 1::8] *= 5000.0
    W[2, 0::16] *= 60.0
    W[3, 5] *= 1e6
    W = W.bfloat16().to(DEV)
    out = pdssm.project(u, None, W, W, W)
    m, p = out["b"].real.double(), out["b"].imag.double()
    assert (p.abs() > 1e4).any() and (m.abs() > 100).any() and (m < -100).any()
    ref = torch.polar(torch.sigmoid(m), p)
    # fp32: r and the sine and cosine to a few roundings, exp's relative error growing with |m|
    tol = 4e-7 + torch.sigmoid(m) * 2.0 ** -23 * m.abs()
    assert ((out["D"].real.double() - ref.real).abs() <= tol).all()
    assert ((out["D"].imag.double() - ref.imag).abs() <= tol).all()


def test_project_generator_neighbours():
    """D of a token has the same bits whatever the tokens and columns beside it
    hold (an entry beyond the fast generator's range among them) and in either
    tile size; and it is within 2e-7 |D| of 64 bits on its logits and phases: the
    largest over eight ranges of 2^24 samples each is 1.84e-7, of the IEEE divide
    with expf and sincosf 2.06e-7, of a form that rounds twice more 2.4e-7."""
    H, N, Dm, T = 4, 128, 32, 33000
    rule = project_rule().kernel
    assert rule(T, Dm, H, 1, N, route=False) == "wide" and rule(300, Dm, H, 1, N, route=False) == "dma128"
    g = torch.Generator().manual_seed(5)
    u = torch.randn((1, T, Dm), generator=g).bfloat16().to(DEV)
    W = (torch.randn((H, 2 * N, Dm), generator=g) * 0.4).bfloat16().to(DEV)
    out = pdssm.project(u, None, W, W, W)
    m, p = out["b"].real.double(), out["b"].imag.double()
    assert m.abs().max() < 80 and p.abs().max() < 8192
    ref = torch.polar(torch.sigmoid(m), p)
    assert ((out["D"].to(torch.complex128) - ref).abs() <= 2e-7 * ref.abs()).all()
    loud = u.clone()
    loud[0, 5::128] *= 1e6  # one token of every block
    keep = torch.ones(T, dtype=torch.bool, device=DEV)
    keep[5::128] = False
    other = pdssm.project(loud, None, W, W, W)
    assert (other["b"][0, 5].imag.abs() > 8192).any()
    for k in "bcD":
        assert torch.equal(other[k][:, keep], out[k][:, keep]), k
    loud = W.clone()
    loud[1, 6:8] *= 1e6     # one entry of head 1
    ent = torch.ones((H, N), dtype=torch.bool, device=DEV)
    ent[1, 3] = False
    assert torch.equal(pdssm.project(u, None, None, None, loud)["D"][:, :, ent], out["D"][:, :, ent])
    few = pdssm.project(u[:, :300].contiguous(), None, W, W, W)
    for k in "bcD":
        assert torch.equal(few[k], out[k][:, :300]), k


@pytest.mark.parametrize("B,L,H,K,N,Dm,kinds", [
    (1, 1, 16, 16, 64, 1024, "Sbcd"),   # one token
    (1, 32, 7, 37, 32, 608, "Sbcd"),    # a head over two row tiles, a half tail slice
    (33, 1, 24, 128, 8, 2048, "Sbcd"),  # 64-token kernel; a head over all four row tiles
    (1, 64, 3, 97, 8, 32, "Sbcd"),      # four row tiles, the last partial; one half slice
    (5, 3, 9, 1, 16, 96, "Sbcd"),       # 32 heads a workgroup, K = 1
    (1, 40, 4, 128, 256, 64, "Scd"),
    (1, 17, 2, 129, 8, 64, "Sb"),       # K > 128: the 128-token tiles
    (2, 31, 5, 3, 8, 320, "d"),
])
def test_project_few_tokens(B, L, H, K, N, Dm, kinds):
    """At most 64 tokens, and one case just outside the few-token kernel's range."""
    print("project B=%d L=%d H=%d K=%d N=%d Dm=%d %s" % (B, L, H, K, N, Dm, kinds), flush=True)
    _proj_case(B, L, H, K, N, Dm, seed=B * L + H + K + N + Dm, kinds=kinds)


def test_route_few_tokens_ties():
    """Equal logits in every run of columns that the lanes of a head share, and
    rows of -inf and NaN: the first maximum, as with more tokens."""
    H, K, Dm = 3, 37, 64
    S = torch.zeros(H, K, Dm)
    S[0, [5, 6, 20, 36], 0] = 1.0   # four equal maxima
    S[1, :, 0] = -float("inf")      # every logit -inf
    S[2, :, 0] = torch.arange(K, dtype=torch.float32) % 7
    S[2, 0, 1] = float("nan")       # a NaN first: nothing exceeds it
    u = torch.zeros(1, 1, Dm)
    u[:, :, 0] = 1.0
    for T in (1, 40, 65):
        _, idx = pdssm.route(u.expand(T, 1, Dm).bfloat16().contiguous().to(DEV), S.bfloat16().to(DEV))
        assert (idx[:, 0].cpu() == torch.tensor([5, 0, 0])).all(), T


@pytest.mark.parametrize("H,K,N,Dm,T,big", [
    (16, 16, 64, 1056, 5200, "wide"),    # a half tail slice
    (2, 100, 8, 64, 33000, "dma256"),    # a head over four waves of the few-token kernel
    (5, 7, 32, 608, 18817, "wide"),      # half slices, partial tiles
    (3, 50, 16, 32, 200, "dma128"),      # a contraction of half a slice
])
def test_project_same_bits_in_any_call(H, K, N, Dm, T, big):
    """A token's logits, choices, b, c and D have the same bits whatever kernel
    the call's size selects."""
    rule = project_rule().kernel
    g = torch.Generator().manual_seed(T + Dm)
    u = torch.randn((1, T, Dm), generator=g).bfloat16().to(DEV)
    S = (torch.randn((H, K, Dm), generator=g) / Dm ** 0.5).bfloat16().to(DEV)
    W = [(torch.randn((H, 2 * N, Dm), generator=g) / Dm ** 0.5).bfloat16().to(DEV) for _ in range(3)]
    assert rule(T, Dm, H, K, N) == big
    ref = pdssm.project(u, S, *W)
    for t, kernel in ((1, "thin1"), (31, "thin1"), (33, "thin2"), (64, "thin2"), (65, "dma128")):
        assert rule(t, Dm, H, K, N) == kernel
        for first in (0, T - t):
            got = pdssm.project(u[:, first:first + t].contiguous(), S, *W)
            for k in got:
                assert torch.equal(got[k], ref[k][:, first:first + t]), (k, t, first)


@pytest.mark.parametrize("K", [5, 32, 37, 128, 200])
def test_route_large_tiles_ties(K):
    """Equal logits in every run of columns that lanes or waves share, rows of
    -inf, infinities and a NaN in the 256 x 256 tiles: the first maximum."""
    H, N, Dm, T = 6, 256, 192, 8500
    assert project_rule().kernel(T, Dm, H, K, N) == "wide"
    S = torch.zeros(H, K, Dm)
    at = sorted({K // 7 + 1, K // 4, K // 3, K // 2, K - 1})  # equal maxima
    S[0, at, 0] = 1.0
    S[1, :, 0] = -float("inf")      # every logit -inf
    S[2, :, 0] = torch.arange(K, dtype=torch.float32) % 7
    S[2, 0, 1] = float("nan")       # a NaN first: nothing exceeds it
    S[3, K - 2:, 0] = float("inf")  # the first of two infinities
    S[4, K // 2, 1] = float("nan")  # a NaN later: it exceeds nothing
    S[4, K - 1, 0] = 1.0
    S[5, :, 0] = -1.0
    S[5, K - 1, 0] = -0.5
    u = torch.zeros(1, T, Dm)
    u[:, :, 0] = 1.0
    W = torch.zeros(H, 2 * N, Dm).bfloat16().to(DEV)
    for logits in (True, False):
        out = pdssm.project(u.bfloat16().to(DEV), S.bfloat16().to(DEV), W, W, W, logits=logits)
        want = torch.tensor([at[0], 0, 0, K - 2, K - 1, K - 1], dtype=torch.int32)
        assert (out["idx"][0].cpu() == want).all(), K
        if logits:
            lg = out["logits"][0]
            ref = torch.stack([S[h, :, 0] for h in (0, 1, 3, 5)]).to(DEV)  # u has one entry: the scores themselves
            ref[1] = -float("inf")
            got = lg[:, [0, 1, 3, 5]]
            assert torch.equal(got[:, [0, 3]], ref[[0, 3]].expand(T, 2, K))
            assert (got[:, 1] == -float("inf")).all() and (got[:, 2, K - 2:] == float("inf")).all()
