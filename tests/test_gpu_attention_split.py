"""Both attention kernels around the rule that chooses between them: few workgroups (the key stages dealt out over the waves
of a workgroup) and many (all four waves walk every stage)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def q8():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_06188_amd import q8 as mod
    return mod


def reference(qkv, B, S, heads, d, mask):
    """Plain attention in 64 bits on the CPU."""
    q, k, v = qkv.cpu().double().view(B, S, 3, heads, d).permute(2, 0, 3, 1, 4).contiguous()
    s = torch.matmul(q, k.transpose(-1, -2).contiguous()) / d ** 0.5
    if mask is not None:
        s = s + mask.cpu().double().view(B, 1, 1, S).clamp(min=-1e30)
    return torch.matmul(s.softmax(-1), v).permute(0, 2, 1, 3).reshape(B * S, heads * d)


@pytest.mark.parametrize("B,S,heads,d,mask", [
    # one stage; a stage and a key; fewer stages than waves; as many; one more; ragged last stages; several a wave
    (1, 1, 1, 4, "none"), (2, 31, 2, 8, "some"), (1, 33, 3, 64, "low"), (2, 96, 2, 64, "some"), (3, 128, 2, 32, "low"), (1, 129, 4, 48, "some"),
    (1, 161, 2, 64, "low"), (2, 255, 2, 40, "some"), (1, 300, 2, 128, "low"), (1, 290, 3, 96, "some"), (1, 1000, 2, 64, "low"),
    # 256 / 260 workgroups, 512 / 520 of eight stages, 384 of one
    (16, 128, 4, 64, "some"), (5, 416, 4, 64, "some"), (13, 128, 5, 64, "some"), (16, 256, 4, 64, "low"), (13, 256, 5, 64, "low"), (96, 30, 4, 32, "some"), (65, 128, 1, 80, "low"),
    # many workgroups: the other kernel on ragged sequences, its first stages masked with the lowest number
    (40, 93, 12, 64, "some"), (40, 93, 12, 32, "low"), (33, 70, 8, 128, "low"), (24, 130, 8, 96, "some"),
])
def test_attention_on_both_sides_of_the_split(q8, B, S, heads, d, mask):
    g = torch.Generator(device="cuda").manual_seed(B * 7919 + S * 31 + heads + d)
    qkv = torch.randn((B * S, 3 * heads * d), generator=g, device="cuda")
    m = None
    if mask == "some":
        m = torch.where(torch.rand((B, S), generator=g, device="cuda") < 0.3, -10000.0, 0.0)
    elif mask == "low":      # left padding with the lowest number of the type: whole stages of it before the first key
        m = torch.zeros((B, S), device="cuda")
        m[:, : (2 * S) // 3] = torch.finfo(torch.float32).min
    if m is not None:
        m[:, S - 1] = 0.0
    n, guard = B * S * heads * d, 64
    buf = torch.full((n + guard,), 7.0, device="cuda")
    ctx, slots = buf[:n].view(B * S, heads * d), torch.full((q8.AMAX_SLOTS,), 9e9, device="cuda")
    q8.q8_attention(qkv, B, S, heads, d, ctx=ctx, mask=m, amax_slots=slots)
    scale = torch.tensor([40.0], device="cuda")
    codes = torch.full((n + guard,), 5, dtype=torch.int8, device="cuda")
    q8.q8_attention(qkv, B, S, heads, d, mask=m, q_scale=scale, q_out=codes[:n])
    torch.cuda.synchronize()
    ref = reference(qkv, B, S, heads, d, m)
    got = ctx.cpu().double()
    # probabilities and outputs carry a few roundings of 2^-24 each, the scores one of their own size (|s| < 8): 2e-6 of the
    # largest |V| is the bar of the other attention tests
    assert (got - ref).abs().max().item() <= 2e-6 * qkv[:, 2 * heads * d:].abs().max().item()
    assert slots.max().item() == ctx.abs().max().item()
    assert bool((buf[n:] == 7.0).all()) and bool((codes[n:] == 5).all())
    q_ref = torch.empty((n,), dtype=torch.int8, device="cuda")
    q8.q8_quantize(ctx.reshape(-1), scale, q_ref)
    np.testing.assert_array_equal(codes[:n].cpu().numpy(), q_ref.cpu().numpy())


@pytest.mark.parametrize("B,S,heads,d", [
    (1, 33, 2, 64), (2, 93, 3, 64), (1, 130, 2, 64), (1, 70, 2, 32), (2, 45, 1, 128),          # the stages dealt out
    (2, 33, 140, 64), (2, 93, 44, 64), (2, 130, 30, 64), (2, 70, 50, 32), (2, 45, 70, 128),    # four waves on every stage
])
def test_attention_reads_no_row_behind_its_sequence(q8, B, S, heads, d):
    """Ragged last stages: the rows behind the last sequence are NaN, and so is every sequence but the first one in a second
    call; a key row that does not exist would come in as 0 x NaN."""
    g = torch.Generator(device="cuda").manual_seed(S * 31 + heads + d)
    n, HD = B * S, heads * d
    buf = torch.full((n + 64, 3 * HD), float("nan"), device="cuda")
    buf[:n] = torch.randn((n, 3 * HD), generator=g, device="cuda")
    clean = buf[:n].clone()
    vmax = clean[:, 2 * HD:].abs().max().item()
    ref = reference(clean, B, S, heads, d, None)
    ctx = torch.empty((n, HD), device="cuda")
    q8.q8_attention(buf[:n], B, S, heads, d, ctx=ctx)
    assert (ctx.cpu().double() - ref).abs().max().item() <= 2e-6 * vmax
    if B > 1:
        buf[S:] = float("nan")
        q8.q8_attention(buf[:n], B, S, heads, d, ctx=ctx)
        assert (ctx[:S].cpu().double() - ref[:S]).abs().max().item() <= 2e-6 * vmax
        assert bool(ctx[S:].isnan().all())


@pytest.mark.parametrize("B,heads", [(4, 12), (32, 64)])   # the stages dealt out; four waves on every stage
def test_attention_products_are_as_good_as_one_rounding(q8, B, heads):
    """Scores of a single nonzero column: nothing averages out, so what a product loses against binary32 shows.  Every query
    scores 32 keys near 100 (log2 units), a few tenths apart; the yardstick is the same attention with each score the
    binary32 product of its two binary32 factors and everything behind it in 64 bits.  The six largest partial products,
    summed in one accumulator, are 15 % further off."""
    S, d, scale = 32, 64, 0.5
    g = torch.Generator().manual_seed(heads)
    x = torch.zeros((B, S, 3, heads, d))
    x[:, :, 0, :, 5] = 8 + 8 * torch.rand((B, S, heads), generator=g)
    x[:, :, 1, :, 5] = 13 * (1 + 0.01 * torch.rand((B, S, heads), generator=g))
    x[:, :, 2] = torch.randn((B, S, heads, d), generator=g)
    qkv = x.view(B * S, -1)
    q, k, v = x[:, :, 0, :, 5], x[:, :, 1, :, 5], x[:, :, 2].double().permute(0, 2, 1, 3)
    def ctx_of(s):   # s: [B, heads, queries, keys], log2 units
        p = torch.exp2(s.double() - s.double().amax(-1, keepdim=True))
        return torch.matmul(p / p.sum(-1, keepdim=True), v).permute(0, 2, 1, 3).reshape(B * S, heads * d)
    c = torch.tensor(scale, dtype=torch.float32) * torch.tensor(1.44269504088896341, dtype=torch.float32)
    ref = ctx_of(scale * 1.4426950408889634 * q.double().permute(0, 2, 1)[..., None] * k.double().permute(0, 2, 1)[:, :, None, :])
    rounded = ctx_of((q * c).permute(0, 2, 1)[..., None] * k.permute(0, 2, 1)[:, :, None, :])
    ctx = torch.empty((B * S, heads * d), device="cuda")
    q8.q8_attention(qkv.cuda(), B, S, heads, d, ctx=ctx, scale=scale)
    err, bar = (ctx.cpu().double() - ref).pow(2).mean().sqrt().item(), (rounded - ref).pow(2).mean().sqrt().item()
    assert err <= 1.03 * bar, f"{err:.3e} against {bar:.3e}"


# few heads: the stages dealt out; many: four waves on every stage
RANGE_SHAPES = [(2, 70, 2, 64), (1, 45, 2, 128), (2, 70, 50, 64), (3, 45, 60, 32), (1, 130, 40, 128), (33, 16, 64, 64)]   # the last: more workgroups than slots


@pytest.mark.parametrize("B,S,heads,d", RANGE_SHAPES)
def test_attention_over_the_whole_finite_range(q8, B, S, heads, d):
    """Numbers at both ends of the type, where a sum of three bf16 numbers does not hold 24 bits: V columns of 1e-36 and below,
    a V row and a K row next to the largest float, tiny K against huge Q.  Bar: 2e-6 of the column's largest |V|, as
    everywhere, and one unit of the subnormal numbers for every key."""
    g = torch.Generator().manual_seed(S + heads)
    HD = heads * d
    x = torch.randn((B, S, 3, heads, d), generator=g)
    mask = torch.zeros((B, S))

    def check(name, x, mask):
        qkv = x.reshape(B * S, 3 * HD).cuda()
        ctx, slots = torch.empty((B * S, HD), device="cuda"), torch.full((q8.AMAX_SLOTS,), 9e9, device="cuda")
        q8.q8_attention(qkv, B, S, heads, d, ctx=ctx, mask=mask.cuda(), amax_slots=slots)
        ref = reference(qkv, B, S, heads, d, mask).view(B, S, heads, d)
        vmax = x[:, :, 2].double().abs()
        if mask.min() < 0:
            vmax = vmax * (mask.view(B, S, 1, 1) == 0)
        err = (ctx.cpu().double().view(B, S, heads, d) - ref).abs()
        worst = (err - S * 2.0 ** -149) / vmax.amax(1, keepdim=True)
        assert worst.max().item() <= 2e-6, (name, worst.max().item())
        assert slots.max().item() == ctx.abs().max().item(), name
        # stored scale: the codes of the same results
        scale = torch.tensor([40.0], device="cuda")
        codes, want = torch.empty(B * S * HD, dtype=torch.int8, device="cuda"), torch.empty(B * S * HD, dtype=torch.int8, device="cuda")
        q8.q8_attention(qkv, B, S, heads, d, mask=mask.cuda(), q_scale=scale, q_out=codes)
        q8.q8_quantize(ctx.reshape(-1), scale, want)
        assert torch.equal(codes, want), name

    y = x.clone()
    y[:, :, 2, :, 1::3] *= 1e-36
    y[:, :, 2, :, 2::3] *= 1e-30
    check("small V columns", y, mask)
    y = x.clone()
    y[:, :, 2] *= 3e-37
    check("small V", y, mask)
    y, m = x.clone(), torch.full((B, S), -10000.0)
    m[:, S // 2] = 0.0
    y[:, S // 2, 2] = 3.4e38 * torch.sign(y[:, S // 2, 2])
    check("one key, V next to the largest float", y, m)
    y = x.clone()
    y[:, :, 0, :, 0], y[:, :, 1, :, 0] = 1e-38 * y[:, :, 0, :, 0], 3.4e38 * torch.sign(y[:, :, 1, :, 0])
    check("K next to the largest float, Q small", y, mask)
    y = x.clone()
    y[:, :, 0, :, 0] *= 1e36
    y[:, :, 1, :, 0] *= 1e-36
    check("Q huge, K small", y, mask)


@pytest.mark.parametrize("B,S,heads,d", RANGE_SHAPES)
def test_attention_of_infinities_and_nans(q8, B, S, heads, d):
    """An infinity in V makes its column infinite and no other; a key whose score is -inf has no weight; a NaN spreads no
    further than its column."""
    g = torch.Generator().manual_seed(S + heads)
    HD = heads * d
    x = torch.randn((B, S, 3, heads, d), generator=g)
    x[:, :, 0, :, 0] = x[:, :, 0, :, 0].abs() + 0.1
    y = x.clone()
    y[0, 3, 2, :, 2] = float("inf")
    ctx = torch.empty((B * S, HD), device="cuda")
    q8.q8_attention(y.reshape(B * S, -1).cuda(), B, S, heads, d, ctx=ctx)
    got = ctx.cpu().double().view(B, S, heads, d)
    ref = reference(x.reshape(B * S, -1), B, S, heads, d, None).view(B, S, heads, d)
    assert bool((got[0, :, :, 2] == float("inf")).all())
    got[0, :, :, 2] = ref[0, :, :, 2]
    assert (got - ref).abs().max().item() <= 2e-6 * x[:, :, 2].abs().max().item()
    # a NaN in V makes its column NaN and no other, and the abs-max passes over it
    y = x.clone()
    y[0, 3, 2, :, 2] = float("nan")
    slots = torch.full((q8.AMAX_SLOTS,), 9e9, device="cuda")
    q8.q8_attention(y.reshape(B * S, -1).cuda(), B, S, heads, d, ctx=ctx, amax_slots=slots)
    got = ctx.cpu().double().view(B, S, heads, d)
    assert bool(got[0, :, :, 2].isnan().all())
    assert slots.max().item() == got.nan_to_num(nan=0.0).abs().max().item()
    got[0, :, :, 2] = ref[0, :, :, 2]
    assert (got - ref).abs().max().item() <= 2e-6 * x[:, :, 2].abs().max().item()
    y = x.clone()
    y[:, 5, 1, :, 0] = float("-inf")
    mask = torch.zeros((B, S))
    mask[:, 5] = -1e30
    q8.q8_attention(y.reshape(B * S, -1).cuda(), B, S, heads, d, ctx=ctx)
    ref = reference(x.reshape(B * S, -1), B, S, heads, d, mask)
    assert (ctx.cpu().double() - ref).abs().max().item() <= 2e-6 * x[:, :, 2].abs().max().item()


@pytest.mark.parametrize("B,S,heads,d,offset", [(2, 70, 2, 64, 0), (2, 70, 50, 64, 0), (2, 70, 2, 64, 1), (2, 70, 2, 5, 0), (1, 9, 1, 130, 0)])
def test_attention_of_a_sequence_that_is_masked_out(q8, B, S, heads, d, offset):
    """Every key of the first sequence carries the lowest number: the mean of V, whichever kernel runs (both MFMA kernels; a
    view four bytes into its buffer and other widths: the generic one)."""
    g = torch.Generator().manual_seed(d)
    HD = heads * d
    x = torch.randn((B, S, 3, heads, d), generator=g)
    mask = torch.zeros((B, S))
    mask[0] = torch.finfo(torch.float32).min
    buf = torch.empty(x.numel() + offset, device="cuda")
    buf[offset:] = x.reshape(-1).cuda()
    ctx = torch.empty((B * S, HD), device="cuda")
    q8.q8_attention(buf[offset:], B, S, heads, d, ctx=ctx, mask=mask.cuda())
    got = ctx.cpu().double().view(B, S, HD)
    ref = reference(x.reshape(B * S, -1), B, S, heads, d, None).view(B, S, HD)
    ref[0] = x[0, :, 2].double().reshape(S, HD).mean(0)
    assert (got - ref).abs().max().item() <= 2e-6 * x[:, :, 2].abs().max().item()


@pytest.mark.parametrize("B,S,heads,d,mask", [
    # two workgroups a compute unit: width 64 with three stages (staged), four (dealt out), one; width 32 with two and three
    (32, 96, 4, 64, "some"), (32, 128, 4, 64, "some"), (43, 128, 3, 64, "low"), (128, 20, 4, 64, "some"), (64, 33, 4, 32, "low"), (32, 90, 4, 32, "some"), (57, 90, 3, 32, "low"),
])
def test_attention_where_two_workgroups_share_a_compute_unit(q8, B, S, heads, d, mask):
    test_attention_on_both_sides_of_the_split(q8, B, S, heads, d, mask)


@pytest.mark.parametrize("B,S,heads,d", [(1, 200, 2, 64), (2, 330, 2, 32), (1, 290, 2, 128), (4, 330, 44, 64), (6, 290, 40, 32), (3, 200, 50, 128)])
@pytest.mark.parametrize("levels", [(-60, -60, -200, -20, 0), (-7, 20, 0, 75, 90), (0, 5, -30), (-150,), (60,), (-20, 3, 40, -40)])
def test_attention_reference_on_both_sides_of_zero(q8, B, S, heads, d, levels):
    """Stages whose scores lie around given levels: a maximum near zero, far below and far above it, one that jumps from far below to
    zero or beyond, and one that climbs.  Both kernels."""
    g = torch.Generator().manual_seed(S + heads + d + len(levels))
    qkv = torch.randn((B * S, 3 * heads * d), generator=g).cuda()
    m = torch.tensor([float(levels[min(j // 32, len(levels) - 1)]) for j in range(S)]).repeat(B, 1).cuda()
    ctx = torch.empty((B * S, heads * d), device="cuda")
    q8.q8_attention(qkv, B, S, heads, d, ctx=ctx, mask=m)
    ref = reference(qkv, B, S, heads, d, m)
    # a score of up to 2^7.8 (log2 units) is rounded where the mask enters, in the sums of the small products, where the sums meet and where the
    # maximum is subtracted: seven times 2^-17.2 at worst, 2.3e-6 in the mean square; 1e-5 of the largest |V| is the bar of such scores
    assert (ctx.cpu().double() - ref).abs().max().item() <= 1e-5 * qkv[:, 2 * heads * d:].abs().max().item()


@pytest.mark.parametrize("B,S,heads,d,mask", [(16, 380, 4, 32, "some"), (64, 96, 4, 28, "low"), (13, 480, 4, 32, "some"), (16, 190, 5, 64, "some"), (10, 200, 7, 64, "low")])
def test_attention_on_both_sides_of_the_split_by_width(q8, B, S, heads, d, mask):
    """Four waves on every stage: 768 and 780 workgroups of width 32 and below.  The stages dealt out: 480 and 490 of width 64, of six and of
    seven stages."""
    test_attention_on_both_sides_of_the_split(q8, B, S, heads, d, mask)


@pytest.mark.parametrize("value", [-10000.0, torch.finfo(torch.float32).min])
@pytest.mark.parametrize("B,S,heads,d", [
    (3, 1, 2, 64), (2, 1, 3, 20), (2, 1, 2, 128), (2, 70, 2, 64), (3, 170, 2, 32), (1, 300, 2, 128), (2, 33, 2, 5),      # the stages dealt out; any width
    (45, 1, 20, 64), (60, 1, 20, 32), (40, 1, 12, 128), (9, 70, 40, 64), (7, 170, 30, 32), (5, 130, 30, 128),         # four waves on every stage
])
def test_attention_of_one_visible_key_is_its_v(q8, B, S, heads, d, value):
    """One-token sequences, and masks that leave one key: its probability is exactly 1, so the result is its V row bit for bit."""
    g = torch.Generator().manual_seed(B + 31 * S + heads + d)
    x = torch.randn((B, S, 3, heads, d), generator=g)
    x[:, :, 2] *= 10.0 ** torch.randint(-3, 4, (B, S, heads, d), generator=g)
    visible = torch.randint(0, S, (B,), generator=g)
    mask = torch.full((B, S), value)
    mask[torch.arange(B), visible] = 0.0
    ctx = torch.empty((B * S, heads * d), device="cuda")
    q8.q8_attention(x.reshape(B * S, -1).cuda(), B, S, heads, d, ctx=ctx, mask=mask.cuda() if S > 1 else None)
    expected = x[torch.arange(B), visible, 2].reshape(B, 1, heads * d).expand(B, S, heads * d)
    np.testing.assert_array_equal(ctx.cpu().view(B, S, heads * d).numpy(), expected.numpy())


@pytest.mark.parametrize("B", [1, 4])   # the stages dealt out; four waves on every stage
def test_attention_scores_of_one_term_keep_their_lowest_products(q8, B):
    """Scores c k of a single term near 4 (log2 units).  c = 1 + m + l and k = 4 (1 + m + l) in bf16 parts, every m near its largest;
    in half of the heads the l of k is positive, in the other half negative, everything else alike.  What a kernel leaves out of the products m l and
    l m moves the two halves apart: by 2 x 4 x 2^-8 x 2^-17 x 0.78 = 1.9e-7 if it forms neither.  A score is rounded to 2^-22 at worst and the
    result through which it is seen to a few 2^-24 (1.6e-7 in the mean square together), so that the difference of two means over
    512 heads each is 1e-8 of noise: 5e-8 is the bar."""
    heads, d, S = 1024, 4, 2
    g = torch.Generator().manual_seed(3)
    c = np.float32(1 + 2.0 ** -8 * 0.97)
    log2e = np.float32(1.44269504088896341)
    scale = float(np.float32(c / log2e))
    c = np.float32(np.float32(scale) * log2e)
    m = (2.0 ** -8 * (0.55 + 0.4 * torch.rand(heads, generator=g, dtype=torch.float64))).bfloat16().double()
    low = 2.0 ** -17 * (0.65 + 0.3 * torch.rand(heads, generator=g, dtype=torch.float64))
    low[1::2] *= -1
    k = (4 * (1 + m + low)).float()
    x = torch.zeros((B, S, 3, heads, d))
    x[:, :, 0, :, 1] = 1.0
    x[:, 1, 1, :, 1] = k
    x[:, 0, 2, :, 0] = 1.0
    ctx = torch.empty((B * S, heads * d), device="cuda")
    q8.q8_attention(x.reshape(B * S, -1).cuda(), B, S, heads, d, ctx=ctx, scale=scale)
    p = ctx.cpu().double().view(B * S, heads, d)[:, :, 0]   # 1 / (1 + 2^s)
    error = (torch.log2(1 / p - 1) - float(c) * k.double()).mean(0)
    assert abs((error[0::2].mean() - error[1::2].mean()).item()) <= 5e-8


@pytest.mark.parametrize("B,S,heads,d", [(3, 70, 2, 64), (3, 93, 2, 32), (3, 130, 80, 64), (3, 70, 60, 128)])
def test_attention_of_a_nan_in_the_mask(q8, B, S, heads, d):
    """A NaN score makes every result of its sequence NaN, none of another one, and the abs-max passes over it."""
    g = torch.Generator(device="cuda").manual_seed(S + heads)
    qkv = torch.randn((B * S, 3 * heads * d), generator=g, device="cuda")
    mask = torch.zeros((B, S), device="cuda")
    clean, ctx, slots = torch.empty((B * S, heads * d), device="cuda"), torch.empty((B * S, heads * d), device="cuda"), torch.full((q8.AMAX_SLOTS,), 9e9, device="cuda")
    q8.q8_attention(qkv, B, S, heads, d, ctx=clean, mask=mask)
    mask[1, S // 2] = float("nan")
    q8.q8_attention(qkv, B, S, heads, d, ctx=ctx, mask=mask, amax_slots=slots)
    got, want = ctx.view(B, S, -1), clean.view(B, S, -1)
    assert bool(got[1].isnan().all()) and torch.equal(got[0], want[0]) and torch.equal(got[2], want[2])
    assert slots.max().item() == max(want[0].abs().max().item(), want[2].abs().max().item())


def test_attention_of_a_nan_in_the_mask_takes_no_longer(q8):
    """Nothing is formed a second time for a NaN: the plain evaluation of a sequence takes tens of times as long."""
    B, S, heads, d = 1, 1024, 24, 64
    qkv = torch.randn((B * S, 3 * heads * d), device="cuda")
    ctx, mask = torch.empty((B * S, heads * d), device="cuda"), torch.zeros((B, S), device="cuda")

    def best_ms():
        times = []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            q8.q8_attention(qkv, B, S, heads, d, ctx=ctx, mask=mask)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    clean = best_ms()
    mask[0, 5] = float("nan")
    assert best_ms() <= 4 * clean
