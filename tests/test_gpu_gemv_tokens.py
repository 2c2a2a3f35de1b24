"""The several-token dot pass on the matrix cores (tq_gemv, tq_gemv2, tq_gemv_mx with more
than one token) against the single-token kernels on the same quantized activations.

Bar: exact block sums equal and y bitwise equal, token by token: both take each row's fp32
block terms in the same order (the single-token kernels' own parity with the oracle is
asserted in their tests). MXFP4 takes its block sums on the scaled fp8 x fp4 unit (scales
of a wide span in groups): y against the oracle, within 1e-6 of the absolute terms (a term's
fp32 roundings of 2^-24 on its way into the sum: at most 8 per block over a wave's 8 blocks at
k = 16384, where they average out, and 4 + 5 + 3 at k = 1280 x 4; 16 of them are 1e-6)."""
import numpy as np
import pytest
import torch

from gpu_util import announce, assert_close, device
from test_gpu_gemv import gpu_quantize

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tq():
    device()
    from paper_2608_08910_amd import tq as _tq
    return _tq


def make(tq, fmt, n, k, seed, e_lo=110, e_hi=130):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    kb = k // 256
    codes = torch.randint(0, 256, (n, kb, 128), dtype=torch.uint8, device="cuda", generator=g)
    if fmt == "folded":
        lo, hi = codes % 9, (codes // 16) % 9  # nine levels per nibble, as 4-bit two's complement
        codes = ((lo + 12) & 15) | (((hi + 12) & 15) << 4)
        m = tq.TqMatrix(n, k, codes, (torch.rand((n, kb), device="cuda", generator=g) + 0.01).half().view(torch.int16))
        return m, lambda q, d, y, s: tq.tq_gemv(m, q, d, torch.zeros(d.shape, dtype=torch.int32, device="cuda"), y, s), (kb,)
    if fmt == "twoplane":
        codes &= 0x55 | ((codes & 0x55) << 1)  # no 2-bit code 2: a trit is 0, 1 or 3
        a = (torch.rand((n, kb, 2), device="cuda", generator=g) - 0.3).half().view(torch.int16)
        m = tq.TqMatrix2(n, k, codes, a)
        return m, lambda q, d, y, s: tq.tq_gemv2(m, q, d, y, s), (kb, 2)
    e8 = torch.randint(e_lo, e_hi, (n * kb * 8 + 1,), dtype=torch.uint8, device="cuda", generator=g)
    m = tq.TqMatrixMx(n, k, codes, e8[1:].view(n, kb * 8))  # scales off any alignment
    return m, lambda q, d, y, s: tq.tq_gemv_mx(m, q, d, y, s), (kb * 8,)


# every tile of the dispatch (16-token x 16-row tiles 1x1, 1x2, 2x1, 2x2, 2x4, 4x4) with
# ragged rows and tokens; rows of 1 to 64 blocks (one, two, four and eight waves per row
# tile, waves with no block, ragged last rounds); 2 to 16 tokens on both sides of the small-
# matrix bound
SHAPES = [(70, 1280, 5), (16, 256, 16), (300, 512, 17), (131, 768, 33), (45, 1024, 64), (8205, 1280, 7), (4107, 2304, 17),
          (8205, 1280, 20), (16397, 2048, 31), (2061, 4352, 509), (16397, 1536, 65), (37, 16384, 130), (2049, 256, 2),
          (2048, 4096, 3), (4099, 4096, 4), (33, 16384, 4), (40007, 256, 40), (1, 256, 300),
          (701, 1024, 7), (901, 256, 16), (1501, 4096, 8), (299, 12544, 5), (16387, 512, 4)]


@pytest.mark.parametrize("fmt", ["folded", "twoplane", "mxfp4"])
@pytest.mark.parametrize("n,k,t", SHAPES)
def test_tokens_match_single_token_calls_bitwise(tq, oracle, fmt, n, k, t):
    announce(f"{fmt} tokens n={n} k={k} t={t}")
    m, call, per = make(tq, fmt, n, k, n + k + t)
    x = np.random.default_rng(t).standard_normal((t, k)).astype(np.float32)
    q, d, _ = gpu_quantize(tq, x * np.exp(np.linspace(-3, 3, t, dtype=np.float32))[:, None])
    y = torch.full((t + 1, n), float("nan"), device="cuda")
    call(q, d, y[:t], None)
    s = torch.full((t, n, *per), -1, dtype=torch.int32, device="cuda")
    ys = torch.full((t, n), float("nan"), device="cuda")
    call(q, d, ys, s)
    # (the VALU chunks of a small matrix keep the single-token order)
    bitwise = fmt != "mxfp4" or (t <= 16 and n * -(-t // 4) * -(-k // 2048) <= (6400 if k > 4096 else 4800))
    if bitwise:
        assert torch.equal(y[:t], ys), "debug output changes y"
    else:
        check_mx_tokens(tq, oracle, m, q, d, y[:t])
        check_mx_tokens(tq, oracle, m, q, d, ys)
    assert bool(torch.isnan(y[t]).all()), "written past the last token"
    for i in sorted({0, 1, t // 2, min(15, t - 1), min(16, t - 1), t - 2, t - 1}):
        y1 = torch.full((1, n), float("nan"), device="cuda")
        s1 = torch.full((1, n, *per), -1, dtype=torch.int32, device="cuda")
        call(q[i:i + 1], d[i:i + 1], y1, s1)
        assert torch.equal(s[i], s1[0]), f"block sums of token {i}"
        assert not bitwise or torch.equal(y[i], y1[0]), f"y of token {i}"


def check_mx_tokens(tq, oracle, m, q, d, y):
    t = y.shape[0]
    i = sorted({0, t // 2, min(16, t - 1), t - 1})
    c4 = tq.tq_mx_unpack_host(m.codes.cpu().numpy(), m.n, m.k)
    yr, ar = oracle.gemv_mx(c4, np.ascontiguousarray(m.scales.cpu().numpy()), q[i].cpu().numpy(), d[i].cpu().numpy())
    assert_close(y[i].cpu().numpy(), yr, ar, rtol=1e-6, what="y")


# scales of a span up to 2^8 (all at once), wider or beyond 2^+-63 (in groups), and both within
# a matrix; a ragged last row tile must not read as far scales
@pytest.mark.parametrize("e_lo,e_hi", [(116, 125), (116, 126), (64, 191), (20, 236), (62, 67), (188, 193)])
@pytest.mark.parametrize("n,k,t", [(70, 1280, 5), (8205, 256, 9), (4107, 2304, 17), (300, 768, 40)])
def test_mx_scale_range(tq, oracle, n, k, t, e_lo, e_hi):
    announce(f"mx scales {e_lo}..{e_hi} n={n} k={k} t={t}")
    m, call, per = make(tq, "mxfp4", n, k, n + t, e_lo, e_hi)
    q, d, _ = gpu_quantize(tq, np.random.default_rng(t).standard_normal((t, k)).astype(np.float32))
    y = torch.full((t, n), float("nan"), device="cuda")
    call(q, d, y, None)
    check_mx_tokens(tq, oracle, m, q, d, y)


# -- MXFP4 on the scaled matrix unit ---------------------------------------------------------
# sizes that the launcher gives each of its tiles (16-token x 16-row tiles, rows of five blocks
# or more): ragged last row tile, ragged tokens
MX_TILES = {"1x1": (4091, 5), "1x2": (8181, 9), "1x4": (16373, 16), "2x1": (4107, 19), "2x2": (8205, 31), "2x4": (16397, 20)}
DOUBLED = torch.tensor([0, 1, 2, 3, 4, 6, 8, 12, 0, -1, -2, -3, -4, -6, -8, -12], dtype=torch.float64)


def mx_exact(c4, e8, q, blocks):
    """fp64 (exact: whole numbers below 2^28 times a power of two) sums of block blocks[t] of token t: [t][n]."""
    n, k = c4.shape
    w = DOUBLED.cuda()[c4.long()].view(n, k // 32, 32) * torch.exp2(e8.double() - 128).view(n, k // 32, 1)
    w = w.view(n, k // 256, 256)
    return torch.stack([w[:, b] @ q[i].double().view(-1, 256)[b] for i, b in enumerate(blocks)])


def mx_upload(tq, c4, e8):
    n, k = c4.shape
    return tq.TqMatrixMx(n, k, torch.from_numpy(tq.tq_mx_pack_host(c4.to(torch.uint8).cpu().numpy())).cuda(), e8.to(torch.uint8))


def mx_extreme(pattern, n, k, t, span):
    """Codes, scales and activations of the largest magnitudes, scales over the whole span."""
    g = torch.Generator(device="cuda")
    g.manual_seed(n + t + span)
    r = lambda lo, hi, sh: torch.randint(lo, hi, sh, device="cuda", generator=g)
    e8 = 120 + span * r(0, 2, (n, k // 32))
    q = (127 - r(0, 2, (t, k))) * torch.where(r(0, 2, (t, k)) == 0, -1, 1)
    big = torch.where(r(0, 64, (n, k)) == 0, 1, 7)  # +-6, and a few of the smallest code
    if pattern == "aligned":  # one sign throughout, the least scale in one chunk of eight
        e8 = torch.where(torch.arange(k // 32, device="cuda") % 8 == torch.arange(n, device="cuda").view(n, 1) % 8, 120, 120 + span)
        q = q.abs() * torch.where(torch.arange(t, device="cuda") % 2 == 0, 1, -1).view(t, 1)
        return big, e8, q
    if pattern == "cancelling":  # chunk pairs of the largest scale cancel to a few units of the least
        e8 = 120 + span * torch.ones_like(e8)
        e8[:, 2::4] = 120
        big = big.view(n, k // 128, 4, 32)
        big[:, :, 1] = big[:, :, 0] | 8
        q = q.view(t, k // 128, 4, 32)
        q[:, :, 1] = q[:, :, 0]
        return big.reshape(n, k), e8, q.reshape(t, k)
    return big | 8 * r(0, 2, (n, k)), e8, q


@pytest.mark.parametrize("pattern", ["aligned", "cancelling", "mixed"])
@pytest.mark.parametrize("tile", list(MX_TILES))
def test_mx_block_sums_are_exact_over_the_span(tq, tile, pattern):
    # the largest codes and activations, scales that span 2^8: a block's sum is exact and
    # rounded to fp32 once (d = 1 for one block of each token, 0 for the others, so that y is
    # that sum)
    (n, t), k = MX_TILES[tile], 1280
    announce(f"mx exact sums {tile} {pattern}")
    c4, e8, q = mx_extreme(pattern, n, k, t, 8)
    blocks = [(3 * i + 1) % 5 for i in range(t)]
    d = torch.zeros((t, 5), device="cuda")
    d[torch.arange(t), torch.tensor(blocks)] = 1.0
    y = torch.full((t, n), float("nan"), device="cuda")
    tq.tq_gemv_mx(mx_upload(tq, c4, e8), q.to(torch.int8), d, y)
    assert torch.equal(y, mx_exact(c4, e8, q, blocks).float())


def mx_groups(e8, k):
    """Group of each chunk's scale ([n][k/32]) by the rule of tq.h: all 0 in a block whose scales span at most
    2^8 within 2^+-63, else by distance from the block's largest, nine powers of two a group."""
    e = e8.view(e8.shape[0], k // 256, 8).int()
    hi, lo = e.amax(2, keepdim=True), e.amin(2, keepdim=True)
    far = (hi > 190) | (lo < 64) | (hi - lo > 8)
    return torch.where(far, (hi - e) // 9, 0).view(e8.shape)


@pytest.mark.parametrize("e_lo,e_hi", [(100, 110), (100, 126), (40, 64), (185, 205)])
@pytest.mark.parametrize("tile", list(MX_TILES))
def test_mx_far_scales_add_group_by_group(tq, tile, e_lo, e_hi):
    # scales too far apart or too large or small: each group's sum exact and rounded once, added
    # up from the largest scales down, before d (d = 1 for one block of each token, 0 for the others; the fp64
    # sums here are exact: below 2^(19 + 26) units)
    (n, t), k = MX_TILES[tile], 1280
    announce(f"mx far scales {tile} {e_lo}..{e_hi}")
    g = torch.Generator(device="cuda")
    g.manual_seed(n + t + e_lo)
    c4 = torch.randint(0, 16, (n, k), device="cuda", generator=g)
    e8 = torch.randint(e_lo, e_hi, (n, k // 32), device="cuda", generator=g)
    q = torch.randint(-127, 128, (t, k), device="cuda", generator=g)
    blocks = [(3 * i + 1) % 5 for i in range(t)]
    d = torch.zeros((t, 5), device="cuda")
    d[torch.arange(t), torch.tensor(blocks)] = 1.0
    y = torch.full((t, n), float("nan"), device="cuda")
    tq.tq_gemv_mx(mx_upload(tq, c4, e8), q.to(torch.int8), d, y)
    grp = mx_groups(e8, k).repeat_interleave(32, 1)
    want = torch.zeros((t, n), device="cuda")
    for p in range(int(grp.max()) + 1):
        want = (want.double() + mx_exact(torch.where(grp == p, c4, 0), e8, q, blocks).float().double()).float()
    assert torch.equal(y, want)


@pytest.mark.parametrize("k", [256, 1024, 2304, 5120])
@pytest.mark.parametrize("tile", list(MX_TILES))
def test_mx_rows_are_their_own(tq, tile, k):
    # a row's bits depend neither on its neighbours' scales (near ones among far ones and the
    # other way round, far in some of their blocks) nor on the block-sum output
    n, t = MX_TILES[tile]
    announce(f"mx rows {tile} k={k}")
    g = torch.Generator(device="cuda")
    g.manual_seed(n + t + k)
    c4 = torch.randint(0, 16, (n, k), device="cuda", generator=g)
    near = torch.randint(116, 125, (n, k // 32), device="cuda", generator=g)
    far = torch.where(torch.rand((n, k // 256, 1), device="cuda", generator=g).repeat(1, 1, 8).view(n, -1) < 0.5,
                      torch.randint(104, 132, (n, k // 32), device="cuda", generator=g), near)
    q = torch.randint(-127, 128, (t, k), device="cuda", generator=g).to(torch.int8)
    d = torch.rand((t, k // 256), device="cuda", generator=g)

    def run(e8, s=None):
        y = torch.full((t, n), float("nan"), device="cuda")
        tq.tq_gemv_mx(mx_upload(tq, c4, e8), q, d, y, s)
        return y

    sums = lambda: torch.full((t, n, k // 32), -1, dtype=torch.int32, device="cuda")
    y_near, y_far = run(near), run(far)
    for share in (1 / 16, 1 / 2, 15 / 16):
        pick = torch.rand(n, device="cuda", generator=g) < share
        e8, s = torch.where(pick.view(n, 1), far, near), sums()
        y = run(e8)
        assert torch.equal(y, torch.where(pick, y_far, y_near))
        assert torch.equal(y, run(e8, s)), "debug output changes y"
        w = DOUBLED.cuda()[c4].view(n, k // 32, 32).float()  # exact in fp32 (below 2^16)
        i = t // 2
        assert torch.equal(s[i], (w * q[i].float().view(k // 32, 32)).sum(2).int()), "block sums"


@pytest.mark.parametrize("e_lo,e_hi", [(116, 125), (110, 131), (20, 60)])
@pytest.mark.parametrize("n,k,t", [(512, 16384, 40), (2048, 4096, 17)])
def test_mx_loses_no_precision(tq, n, k, t, e_lo, e_hi):
    # error against fp64 no larger than that of the single-token pass on the same data
    announce(f"mx precision n={n} k={k} t={t} {e_lo}..{e_hi}")
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    c4 = torch.randint(0, 16, (n, k), device="cuda", generator=g)
    e8 = torch.randint(e_lo, e_hi, (n, k // 32), device="cuda", generator=g)
    q = torch.randint(-127, 128, (t, k), device="cuda", generator=g).to(torch.int8)
    d = torch.rand((t, k // 256), device="cuda", generator=g)
    m = mx_upload(tq, c4, e8)
    y, y1 = torch.empty((t, n), device="cuda"), torch.empty((t, n), device="cuda")
    tq.tq_gemv_mx(m, q, d, y)
    for i in range(t):
        tq.tq_gemv_mx(m, q[i:i + 1], d[i:i + 1], y1[i:i + 1])
    w = DOUBLED.cuda()[c4].view(n, k // 32, 32) * torch.exp2(e8.double() - 128).view(n, k // 32, 1)
    r = (q.double().view(t, k // 256, 256) * d.double().view(t, -1, 1)).view(t, k) @ w.view(n, k).t()
    assert float((y - r).norm()) <= float((y1 - r).norm())


@pytest.mark.parametrize("tile", list(MX_TILES))
def test_mx_near_scales_match_the_oracle(tq, oracle, tile):
    # the scaled unit alone, two blocks for some waves and one for the others
    (n, t), k = MX_TILES[tile], 2304
    announce(f"mx near scales {tile}")
    m, call, _ = make(tq, "mxfp4", n, k, n + t, 116, 125)
    q, d, _ = gpu_quantize(tq, np.random.default_rng(t).standard_normal((t, k)).astype(np.float32))
    y = torch.full((t + 1, n), float("nan"), device="cuda")
    call(q, d, y[:t], None)
    check_mx_tokens(tq, oracle, m, q, d, y[:t])
    assert bool(torch.isnan(y[t]).all()), "written past the last token"


@pytest.mark.parametrize("e8", [125, 40])
@pytest.mark.parametrize("tile", list(MX_TILES))
def test_mx_every_code_times_every_activation(tq, tile, e8):
    # row r: one code (r / 256) % 16 at column r % 256 of a block, zeros elsewhere; token values
    # -127 .. 127 throughout: each product exact, on near scales and on far ones
    (n, t), k = MX_TILES[tile], 1280
    announce(f"mx codes x activations {tile} e8={e8}")
    r = torch.arange(n, device="cuda")
    code, col = (r // 256) % 16, (r * 257) % 1280
    c4 = torch.zeros((n, k), dtype=torch.int64, device="cuda")
    c4[r, col] = code
    m = mx_upload(tq, c4, torch.full((n, k // 32), e8, device="cuda"))
    d = torch.ones((t, k // 256), device="cuda")
    for v0 in range(-127, 128, t):
        v = torch.arange(v0, v0 + t, device="cuda").clamp(max=127)
        y = torch.full((t, n), float("nan"), device="cuda")
        tq.tq_gemv_mx(m, v.view(t, 1).repeat(1, k).to(torch.int8), d, y)
        want = v.double().view(t, 1) * DOUBLED.cuda()[code] * 2.0 ** (e8 - 128)
        assert torch.equal(y.double(), want), f"activations {v0} .. {int(v[-1])}"
