"""The fp32 products as products of bf16 terms: every tile form and group count, operands that are not finite
or overflow, and the error against float64 (less than the fp32 matrix instruction's on the same operands:
4.1e-7 at K 512, 5.7e-7 at K 1024), also of short sums and of operands whose terms are all long."""
import pytest
import torch

import paper_2006_16668_amd as moe

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _ffn(E, R, M, H, edit=None):
    g = torch.Generator(device=DEV).manual_seed(E * R + M + H)
    buf = torch.randn(E, 1, R, M, device=DEV, generator=g)
    wi = torch.randn(E, M, H, device=DEV, generator=g) / M ** 0.5
    wo = torch.randn(E, H, M, device=DEV, generator=g) / H ** 0.5
    if edit:
        edit(buf, wi)
    h = torch.full((E, 1, R, H), float("nan"), device=DEV)
    out = torch.full((E, 1, R, M), float("nan"), device=DEV)
    moe.moe_expert_ffn(moe.MoEShape(1, R, M, H, E, R, "f32"), buf, wi, wo, h, out)
    torch.cuda.synchronize()
    return buf[:, 0], wi, wo, h[:, 0], out[:, 0]


def _error(got, want):
    return float((got.double() - want).norm() / want.norm())


# tiles of h and out on 256 units: 64 x 64 with four groups and with two; with four both; 64 x 128, 64 x 64 with four;
# 64 x 128 both, twice; 64 x 64 without groups both; 128 x 128 both
@pytest.mark.parametrize("E,R,M,H", [(2, 70, 516, 260), (3, 190, 1024, 1028), (16, 128, 512, 1024), (66, 12, 848, 3424),
                                     (2, 3000, 1024, 1536), (64, 257, 64, 132), (64, 130, 132, 132)])
def test_error_against_float64(E, R, M, H):
    buf, wi, wo, h, out = _ffn(E, R, M, H)
    # the leading products' sum is rounded twice per 16 k: about 0.1 x 2^-24 sqrt(K) on these operands, allowed twice
    # that; plus a last place
    bound = lambda K: 2.0 ** -24 * (1 + 0.2 * K ** 0.5)
    assert _error(h, torch.relu(buf.double() @ wi.double())) < bound(M)
    assert _error(out, h.double() @ wo.double()) < bound(H)


# tiles of h: 64 x 64 with two groups, twice; 64 x 128, twice; 64 x 64 without groups; 128 x 128
@pytest.mark.parametrize("E,R,M,H", [(2, 70, 132, 260), (3, 300, 160, 1028), (40, 200, 128, 1024), (2, 3000, 144, 1536),
                                     (64, 257, 64, 132), (64, 130, 132, 132)])
def test_infinities_nan_and_overflow(E, R, M, H):
    inf, nan = float("inf"), float("nan")

    def edit(buf, wi):
        buf[0, 0, 3, 5], buf[1, 0, R - 1, M - 1], buf[1, 0, 7, 0] = inf, -inf, nan
        buf[0, 0, 40] = 0                                      # finite, near the largest: some products overflow
        buf[0, 0, 40, 5] = 3e38
        wi[0, 5, ::7] = 2
        wi[E - 1, 2, H - 2] = inf
        wi[0, M // 2, 9] = 3.4e38

    buf, wi, _, h, _ = _ffn(E, R, M, H, edit)
    want = torch.bmm(buf, wi)                                  # fp32 (no order of the sums changes what overflows)
    ok = torch.isfinite(want)
    assert 0 < int((~ok).sum()) < ok.numel() // 4
    assert torch.equal(torch.isfinite(h) | ~ok, torch.ones_like(ok))        # a finite sum stays one
    pos, neg, und = want == inf, want == -inf, torch.isnan(want)
    assert bool((h[pos] == inf).all()) and bool((h[neg] == 0).all())
    assert bool((h[und] == 0).all())                           # relu of NaN, as maxnum gives it
    exact = torch.relu(buf.double() @ wi.double())
    scale = exact[ok].abs() + 1e-3 * torch.linalg.vector_norm(buf.double(), dim=-1, keepdim=True).expand_as(exact)[ok]
    fin = torch.isfinite(scale)
    assert float(((h[ok].double() - exact[ok]).abs() / scale)[fin].max()) < 1e-3


def _chain(a, b):
    """a [E,R,K] b [E,K,N] summed k by k, one fp32 rounding per product and sum: the fp32 instruction's way."""
    s = torch.zeros(a.shape[0], a.shape[1], b.shape[2], device=DEV)
    for k in range(a.shape[2]):
        s = (s.double() + a[:, :, k, None].double() * b[:, None, k].double()).float()
    return s


# one step of 16 k; of two groups (32) and of four (64), which meet in LDS after it
@pytest.mark.parametrize("K", [4, 8, 12, 16, 32, 64])
def test_short_sums(K):
    buf, wi, _, h, _ = _ffn(2, 70, K, 260)
    want = torch.relu(buf.double() @ wi.double())
    assert _error(h, want) <= _error(torch.relu(_chain(buf, wi)), want)


@pytest.mark.parametrize("E,R,M,H", [(2, 70, 4, 260), (2, 70, 512, 260), (64, 130, 132, 132)])
def test_long_mantissas(E, R, M, H):
    # truncated terms left 2^-21 of these products out, of every product the same
    c = 1 + 2.0 ** -7 - 2.0 ** -23

    def edit(buf, wi):
        buf.fill_(c), wi.fill_(c)

    h = _ffn(E, R, M, H, edit)[3]
    want = M * c * c
    # their three terms are exact in two, so are the products: the sums' own roundings, half a last place each
    assert float((h.double() - want).abs().max()) < want * 2.0 ** -24 * (1 + 2.0 ** -6)


def _step(x, wg, wi, wo, dy, C):
    """A training step of one group with every token sent where wg says."""
    _, S, M = x.shape
    E, _, H = wi.shape
    sh = moe.MoEShape(1, S, M, H, E, C, "f32")
    u, y, aux = torch.full((1, S), 0.5, device=DEV), torch.empty_like(x), torch.empty(1, device=DEV)
    fws = torch.empty(moe.moe_train_workspace_bytes(sh), dtype=torch.uint8, device=DEV)
    bws = torch.empty(moe.moe_backward_workspace_bytes(sh), dtype=torch.uint8, device=DEV)
    dx, dwg, dwi, dwo = (torch.full_like(t, float("nan")) for t in (x, wg, wi, wo))
    moe.moe_forward_train(sh, x, wg, u, wi, wo, y, aux, fws)
    moe.moe_backward(sh, x, wg, wi, wo, dy, torch.zeros(1, device=DEV), fws, dx, dwg, dwi, dwo, bws)
    torch.cuda.synchronize()
    return y, dx, dwi, dwo


def test_weight_gradients_of_few_tokens():
    # expert e keeps e + 1 tokens.  A token is a unit vector, its row of h a row of wi, its weight 1: h and dout are exact
    E, M, H = 16, 160, 132
    kept = [e + 1 for e in range(E)]
    expert = torch.repeat_interleave(torch.arange(E), torch.tensor(kept)).to(DEV)
    S = len(expert)
    g = torch.Generator(device=DEV).manual_seed(5)
    wi = torch.rand(E, M, H, device=DEV, generator=g) + 0.5
    wo, dy = torch.randn(E, H, M, device=DEV, generator=g), torch.randn(1, S, M, device=DEV, generator=g)
    x = torch.eye(S, M, device=DEV).view(1, S, M)
    wg = torch.zeros(M, E, device=DEV)
    wg[torch.arange(S, device=DEV), expert] = 200
    dwo = _step(x, wg, wi, wo, dy, max(kept))[3]
    first = 0
    for e in range(E):
        t = torch.arange(first, first + kept[e], device=DEV)
        first += kept[e]
        a, b = wi[e, t].t().contiguous()[None], dy[0, t][None]
        want = (a.double() @ b.double())[0]
        # 1 %: the smaller products' sum is rounded too, at 2^-8 of the result
        assert _error(dwo[e], want) <= 1.01 * _error(_chain(a, b)[0], want), e
        if kept[e] == 1:
            assert float(((dwo[e].double() - want) / want).abs().max()) < 2.0 ** -24 * (1 + 2.0 ** -6)


@pytest.mark.parametrize("E,R,M,H", [(2, 70, 516, 132), (64, 130, 132, 132)])
@pytest.mark.parametrize("small", ["a", "b"])
def test_operands_near_the_smallest(E, R, M, H, small):
    # of these the smallest terms (2^-16 of an operand and less) are below bf16's range, some below fp32's normal one
    def edit(buf, wi):
        a, b = (2.0 ** -124, 2.0 ** 60) if small == "a" else (2.0 ** 60, 2.0 ** -124)
        buf.mul_(a), wi.mul_(b)

    buf, wi, _, h, _ = _ffn(E, R, M, H, edit)
    want = torch.relu(buf.double() @ wi.double())
    assert _error(h, want) <= _error(torch.relu(_chain(buf, wi)), want)


def _same(got, want, tol):
    """Infinities and NaN where float64 has them, every other element within tol of the norm of its kind."""
    want = want.float()
    for v in (torch.isnan, torch.isposinf, torch.isneginf):
        assert torch.equal(v(got), v(want)), v.__name__
    big = want.abs() > 1e30                                    # (sums that a single huge term decides)
    ok = torch.isfinite(want) & ~big
    assert not ok.any() or _error(got[ok], want[ok].double()) < tol
    big &= torch.isfinite(want)
    assert not big.any() or _error(got[big], want[big].double()) < tol


# tiles of 128 x 128 throughout; 64 x 128 (weight gradients 128 x 128); 64 x 64 with two groups (weight gradients without)
@pytest.mark.parametrize("E,C,M,H", [(16, 512, 1024, 2048), (66, 12, 848, 3424), (3, 70, 132, 260)])
def test_training_step_with_infinities(E, C, M, H):
    """Masked and plain data gradients and weight gradients over kept rows with operands that are not finite."""
    inf, nan = float("inf"), float("nan")
    S = E * C - 5 if E > 3 else E * C - 1                      # (one expert with empty positions)
    g = torch.Generator(device=DEV).manual_seed(E + C)
    expert = torch.arange(S, device=DEV) % E
    x = torch.randn(1, S, M, device=DEV, generator=g)
    x[0, :, M - E:] = 0
    x[0, torch.arange(S, device=DEV), M - E + expert] = 1
    wg = torch.zeros(M, E, device=DEV)
    wg[M - E + torch.arange(E), torch.arange(E)] = 200
    wi = torch.randn(E, M, H, device=DEV, generator=g) / M ** 0.5
    wo = torch.randn(E, H, M, device=DEV, generator=g) / H ** 0.5
    dy = torch.randn(1, S, M, device=DEV, generator=g)
    wi[0, 5, 3], wi[0, 2, 1] = inf, nan
    dy[0, 1, 7], dy[0, 1 + E, 9] = inf, nan                    # of expert 1
    dy[0, 2, 11] = 3e38                                        # of expert 2: some products overflow
    y, dx, dwi, dwo = _step(x, wg, wi, wo, dy, C)
    for e in range(min(E, 4)):
        t = torch.nonzero(expert == e).flatten()
        xe, de = x[0, t].double(), dy[0, t].double()
        h = (xe @ wi[e].double()).float().double()
        h = torch.where(h > 0, h, 0.0)                         # relu of NaN, as maxnum gives it
        dh = torch.where(h > 0, (de @ wo[e].double().t()).float().double(), 0.0)
        # a few of up to 2 million h may be on the other side of 0: a share p of them shows as sqrt(p)
        tol = 2e-3
        _same(y[0, t], h @ wo[e].double(), tol)
        _same(dwo[e], h.t() @ de, tol)
        _same(dwi[e], xe.t() @ dh, tol)
        want = dh @ wi[e].double().t()
        # tokens whose gate gradient is finite too
        ok = torch.isfinite((y[0, t].double() * de).sum(-1).float()) & torch.isfinite(want).all(-1)
        _same(dx[0, t][ok], want[ok], tol)
