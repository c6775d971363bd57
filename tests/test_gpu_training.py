"""GPU parity of the training-side entry points against the CPU oracle: fake quantization
(Section 2.2), the moving average of max|x| under Eq. 4 and the straight-through gradient
(Eq. 5).  Every operation here is a fixed sequence of correctly rounded binary32 operations,
so the comparison is bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import q8_oracle as O  # noqa: E402
from paper_1910_06188_amd import synth  # noqa: E402


@pytest.fixture(scope="module")
def q8():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_06188_amd import q8 as mod
    return mod


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    return t.detach().cpu().numpy()


def scalar(v):
    return torch.tensor([v], dtype=torch.float32, device="cuda")


def same_bits(a, b):
    return a.astype(np.float32).tobytes() == b.astype(np.float32).tobytes()


@pytest.mark.parametrize("n", [0, 1, 3, 4, 5, 255, 1024, 4099, 1_000_003, 3_145_728])
def test_fake_quantize_bit_exact(q8, n):
    g = synth.rng(300 + n % 89)
    x = g.standard_normal(n, dtype=np.float32) * np.float32(1.7)
    if n > 8:
        x[:8] = np.array([0.0, -0.0, 1e-30, -1e-30, 50.0, -50.0, 4.6, -4.6], dtype=np.float32)   # beyond the clamp too
    for s in (np.float32(27.3), np.float32(1.0), np.float32(127.0) / max(np.float32(1e-3), np.abs(x).max() if n else np.float32(1))):
        xd = dev(x)
        y = torch.full((n,), 9.0, device="cuda")
        q8.q8_fake_quantize(xd, scalar(float(s)), y)
        ref = O.fake_quantize(x, s)
        assert same_bits(host(y), ref), (n, float(s))
        # in place
        q8.q8_fake_quantize(xd, scalar(float(s)), xd)
        assert same_bits(host(xd), ref), (n, float(s))


def test_fake_quantize_misaligned_views(q8):
    g = synth.rng(31)
    base = g.standard_normal(5003, dtype=np.float32)
    bd = dev(base)
    s = np.float32(40.0)
    for off in (1, 2, 3):
        for n in (1, 6, 1001, 4999):
            out = torch.zeros(5003 + 4, device="cuda")
            q8.q8_fake_quantize(bd[off:off + n], scalar(float(s)), out[off:off + n])
            got = host(out)
            assert same_bits(got[off:off + n], O.fake_quantize(base[off:off + n], s))
            assert not got[:off].any() and not got[off + n:].any()          # nothing outside the view


def test_ema_sequence_bit_exact(q8):
    g = synth.rng(32)
    state = torch.zeros(2, device="cuda")
    e_ref, started = np.float32(0.0), False
    for step in range(25):
        decay = [0.9, 0.99, 0.5, 0.0, 1.0][step % 5]
        parts = np.abs(g.standard_normal(1 + step * 7, dtype=np.float32)) * np.float32(3.0)
        a_out, s_out = scalar(-1.0), scalar(-1.0)
        q8.q8_ema_update(dev(parts), decay, state, amax_out=a_out, scale_out=s_out)
        a = parts.max()
        e_ref = O.ema_update(e_ref, started, a, np.float32(decay))
        started = True
        st = host(state)
        assert st[0] == e_ref and st[1] == 1.0, step
        assert host(a_out)[0] == a
        assert host(s_out)[0] == O.scale(e_ref)
    # outputs are optional
    q8.q8_ema_update(dev(np.array([2.0], dtype=np.float32)), 0.5, state)
    assert host(state)[0] == O.ema_update(e_ref, True, 2.0, 0.5)


@pytest.mark.parametrize("shape", [(16, 768), (777, 1024), (4096, 768)])
def test_fake_quantize_ema_training_steps(q8, shape):
    """Three training steps of the activation quantizer on changing batches: state, scale and the
    fake-quantized tensor all follow the oracle bit for bit; decay 0 reproduces the weights'
    quantizer (Eq. 3 on the tensor's own max)."""
    g = synth.rng(33 + shape[0])
    state = torch.zeros(2, device="cuda")
    work = torch.zeros(q8.SCAL_WORK, device="cuda")
    e_ref, started = np.float32(0.0), False
    for step, gain in enumerate((1.0, 2.5, 0.4)):
        x = synth.activations(g, *shape) * np.float32(gain)
        y = torch.empty(shape, device="cuda")
        q8.q8_fake_quantize_ema(dev(x), 0.9, state, work, y)
        a = O.absmax(x)
        e_ref = O.ema_update(e_ref, started, a, np.float32(0.9))
        started = True
        s = O.scale(e_ref)
        w = host(work)
        assert w[0] == a and w[1] == s and host(state)[0] == e_ref, step
        assert same_bits(host(y), O.fake_quantize(x, s)), step
    W = synth.weights(g, *shape)
    st2 = torch.zeros(2, device="cuda")
    Wd = dev(W)
    for _ in range(2):                       # second call: state already started, decay 0 forgets it
        out = torch.empty(shape, device="cuda")
        q8.q8_fake_quantize_ema(Wd, 0.0, st2, work, out)
        sw = O.scale(O.absmax(W))
        assert host(work)[1] == sw
        assert same_bits(host(out), O.fake_quantize(W, sw))
    # empty batch: counts as max 0
    st3 = torch.zeros(2, device="cuda")
    q8.q8_fake_quantize_ema(torch.empty(0, device="cuda"), 0.9, st3, work, torch.empty(0, device="cuda"))
    assert host(st3).tolist() == [0.0, 1.0] and host(work)[1] == 1.0


@pytest.mark.parametrize("n", [0, 1, 5, 4099, 2_000_001])
def test_ste_backward_identity(q8, n):
    g = synth.rng(34)
    grad = g.standard_normal(n, dtype=np.float32)
    gd = dev(grad)
    out = torch.full((n,), 7.0, device="cuda")
    q8.q8_ste_backward(gd, out)
    assert same_bits(host(out), O.ste_backward(grad))
    q8.q8_ste_backward(gd, gd)               # aliasing: nothing to do
    assert same_bits(host(gd), grad)
    if n > 3:
        out2 = torch.zeros(n + 2, device="cuda")
        q8.q8_ste_backward(gd[1:], out2[2:n + 1])
        assert same_bits(host(out2)[2:n + 1], grad[1:]) and host(out2)[1] == 0 and host(out2)[n + 1] == 0


def test_training_argument_checks(q8):
    lib = q8.raw()
    x = torch.zeros(8, device="cuda")
    st = torch.zeros(2, device="cuda")
    work = torch.zeros(q8.SCAL_WORK, device="cuda")
    p = lambda t: t.data_ptr()
    assert lib.q8_fake_quantize(p(x), -1, p(x), p(x), None) == 2
    assert lib.q8_fake_quantize(None, 8, p(x), p(x), None) == 1
    assert lib.q8_fake_quantize(p(x) + 1, 4, p(x), p(x), None) == 3
    assert lib.q8_ema_update(p(x), 0, 0.5, p(st), None, None, None) == 2
    assert lib.q8_ema_update(p(x), 1, 1.5, p(st), None, None, None) == 2
    assert lib.q8_ema_update(p(x), 1, float("nan"), p(st), None, None, None) == 2
    assert lib.q8_ema_update(p(x), 1, 0.5, None, None, None, None) == 1
    assert lib.q8_fake_quantize_ema(p(x), 8, 0.5, p(st), None, p(x), None) == 1
    assert lib.q8_fake_quantize_ema(p(x), 8, -0.1, p(st), p(work), p(x), None) == 2
    assert lib.q8_ste_backward(p(x), 8, None, None) == 1
    assert lib.q8_ste_backward(p(x), -2, p(x), None) == 2
    torch.cuda.synchronize()


@pytest.mark.parametrize("n,off", [(1, 0), (3, 1), (4096, 0), (4099, 0), (8192 * 6 + 5, 1), (17_000_003, 0), (17_000_000, 1)])
@pytest.mark.parametrize("in_place", [False, True])
def test_ema_inside_the_fake_quantization(q8, n, off, in_place):
    """The two-launch moving-average quantizer over every path of its kernels -- one workgroup, a ragged last block, more
    blocks than partial maxima, outputs beyond 64 MiB (stored past the cache), 4-byte aligned tensors -- and the gradient
    copy of the same sizes.  Two steps, so that the second one reads a state the first has written."""
    g = torch.Generator(device="cuda").manual_seed(n + off)
    state, work = dev(np.zeros(2, np.float32)), torch.full((q8.SCAL_WORK,), 9e9, device="cuda")
    average, started = np.float32(0), False
    for _ in range(2):
        buf = torch.randn(n + off, generator=g, device="cuda")
        x = buf[off:]
        xc = x.clone()
        y = x if in_place else torch.empty(n + off, device="cuda")[off:]
        q8.q8_fake_quantize_ema(x, 0.9, state, work, y)
        a = np.float32(xc.abs().max().item())
        average = O.ema_update(average, started, a, np.float32(0.9))
        started = True
        s = np.float32(127.0) / average
        assert host(state)[0] == average and host(state)[1] == 1.0
        assert host(work)[0] == a and host(work)[1] == s
        ref = torch.empty_like(xc)
        q8.q8_fake_quantize(xc, dev(np.array([s], np.float32)), ref)    # pinned to the oracle above
        assert torch.equal(y, ref)
        part = slice(max(0, n - 5000), n)
        np.testing.assert_array_equal(host(y[part]), O.fake_quantize(host(xc[part]), s))
    out = torch.full((n + off + 4,), 7.0, device="cuda")
    q8.q8_ste_backward(xc, out[off:off + n])
    assert torch.equal(out[off:off + n], xc) and bool((out[off + n:] == 7.0).all())


@pytest.mark.parametrize("n", [16388, 20_000, 4096 * 5, 4096 * 5 + 4, 131_076, 524_288, 524_292, 16389])
@pytest.mark.parametrize("polls", [64, 0])
def test_dynamic_quantizer_of_small_tensors(q8, n, polls):
    """One launch with a grid of its own size (up to half a million elements), waiting at the barrier and giving up at once
    (every workgroup reads the shares of the others); one element more or a ragged count takes two launches."""
    x = torch.randn(n, generator=torch.Generator(device="cuda").manual_seed(n), device="cuda")
    x[n - 1] = -9.5                                     # the maximum sits in the last workgroup
    q, work, zero = torch.full((n + 64,), 77, dtype=torch.int8, device="cuda"), torch.zeros(q8.SCAL_WORK, device="cuda"), torch.ones(1, device="cuda")
    q8.set_quantize_one_pass(True, polls)
    try:
        for _ in range(3):
            q8.q8_quantize_dynamic(x, q[:n], work, zero_slot=zero)
        torch.cuda.synchronize()
    finally:
        q8.set_quantize_one_pass(True, 64)
    xh = host(x)
    s = O.scale(O.absmax(xh))
    assert host(work)[0] == O.absmax(xh) and host(work)[1] == s and host(zero)[0] == 0.0
    np.testing.assert_array_equal(host(q[:n]), O.quantize(xh, s))
    assert bool((q[n:] == 77).all())


@pytest.mark.parametrize("n,off", [(1, 0), (2, 1), (7, 3), (1536, 0), (1537, 1), (100_003, 2), (1_572_864, 0), (1_572_869, 1), (6_000_001, 0)])
@pytest.mark.parametrize("enabled,polls", [(True, 64), (True, 0), (False, 64)])
def test_absmax_in_one_launch(q8, n, off, enabled, polls):
    """The abs-max and its scale in one launch (one workgroup, a few, as many as there are slots and several trips each; the
    first workgroup waiting, and scanning every share that is not there at its first look) and in three."""
    buf = torch.randn(n + off, generator=torch.Generator(device="cuda").manual_seed(n), device="cuda")
    x = buf[off:]
    a, s = torch.full((3,), 5.0, device="cuda"), torch.full((3,), 6.0, device="cuda")
    q8.set_quantize_one_pass(enabled, polls)
    try:
        for pos, value in ((n - 1, -9.5), (0, 11.25), (n // 2, 12.0)):
            x[pos] = value
            for _ in range(2):
                q8.q8_absmax(x, a[1:2], s[1:2])
            torch.cuda.synchronize()
            xh = host(x)
            assert host(a)[1] == O.absmax(xh) and host(s)[1] == O.scale(O.absmax(xh))
        q8.q8_absmax(x, a[1:2])                                   # no scale asked for
        assert host(a)[1] == O.absmax(xh)
        x.zero_()
        q8.q8_absmax(x, a[1:2], s[1:2])
        assert host(a).tolist() == [5.0, 0.0, 5.0] and host(s).tolist() == [6.0, 1.0, 6.0]
    finally:
        q8.set_quantize_one_pass(True, 64)


def test_absmax_many_launches_on_two_streams(q8):
    """More launches in flight than the ring of slots has entries, sizes mixed over two streams."""
    sizes = [5, 70_000, 1_000_003, 3_000_000]
    xs = [torch.randn(n, device="cuda") for n in sizes]
    peak = [float(x.abs().max()) for x in xs]
    out = torch.zeros((2, 400), device="cuda")
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for i in range(400):
        for j, st in enumerate(streams):
            q8.q8_absmax(xs[(i + j) % 4], out[j, i:i + 1], stream=st)
    torch.cuda.synchronize()
    got = host(out)
    for j in range(2):
        for i in range(400):
            assert got[j, i] == np.float32(peak[(i + j) % 4])


def test_absmax_launches_that_share_a_ring_entry_do_not_stall(q8):
    """Two launches 256 apart use the same slots.  Both wait for the same event and then run at the same time, the older one
    up to some tens of microseconds later, so that their writes to a slot come in any order: the older one's values must not
    stand in for the newer one's, which would then be waited for until the bound of about a second."""
    import time
    n, rounds = 24_000_000, 24
    x = [torch.randn(n, device="cuda") for _ in range(2)]
    peak = [np.float32(v.abs().max().item()) for v in x]
    small = torch.randn(8, device="cuda")
    out, skip, late = torch.zeros((2, rounds), device="cuda"), torch.zeros(1, device="cuda"), torch.zeros(8, device="cuda")
    first, old, new = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream()
    slowest = 0.0
    for i in range(rounds):
        torch.cuda.synchronize()
        gate = torch.cuda.Event()
        with torch.cuda.stream(first):
            torch.cuda._sleep(8_000_000)            # some milliseconds of one thread, in which all but the last launches below come and go
            gate.record()
        old.wait_event(gate)
        with torch.cuda.stream(old):
            for _ in range(i % 8):
                late += 1
        q8.q8_absmax(x[0], out[0, i:i + 1], stream=old)
        for _ in range(255):
            q8.q8_absmax(small, skip, stream=new)
        new.wait_event(gate)
        q8.q8_absmax(x[1], out[1, i:i + 1], stream=new)
        start = time.perf_counter()
        torch.cuda.synchronize()
        slowest = max(slowest, time.perf_counter() - start)
    got = host(out)
    for j in range(2):
        assert (got[j] == peak[j]).all()
    assert slowest < 0.5, slowest
