"""The kernels of small and ragged FC launches: 64x64 tiles with deep rings (variant 7), the direct kernel (variant 8; by itself for few
tiles, for operands that are not 4-byte aligned and for long reductions in few tiles), the tiles with few stage buffers (variants 9 to 13) and the
one-thread-per-output kernel of the very shortest reductions; and the choice among all of them (variant 0).  Every output must carry the bits of
the staged 128x128 kernel on operands zero-padded to a multiple of 128, which the other tests pin to the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import q8_oracle as O
from paper_1910_06188_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def q8():
    from paper_1910_06188_amd import q8 as m
    return m


def at_offset(a, off):
    """A device copy of the int8 array whose first byte lies `off` bytes behind a 16-byte boundary and whose last byte
    ends the allocation's used part."""
    buf = torch.zeros(a.size + off, dtype=torch.int8, device="cuda")
    buf[off:] = torch.from_numpy(a.reshape(-1)).cuda()
    return buf[off:].view(a.shape)


@pytest.mark.parametrize("M,K,N,variant,off", [
    # the direct kernel: every class of row end (bytes, words, one vector, a unit and what follows it) on ragged tiles
    (5, 1, 3, 8, 0), (33, 3, 34, 8, 0), (31, 4, 32, 8, 1), (40, 7, 65, 8, 3), (64, 15, 31, 8, 0), (1, 16, 2, 8, 5), (33, 17, 70, 8, 0),
    (20, 31, 24, 8, 2), (65, 127, 33, 0, 0), (32, 128, 32, 0, 1), (37, 129, 100, 0, 0), (70, 250, 129, 0, 7), (96, 1000, 200, 0, 0),
    (18, 1151, 40, 0, 0), (8, 2048, 96, 8, 0), (130, 3072, 64, 0, 0), (33, 4095, 31, 0, 15),
    # one thread per output, and the direct kernel right behind it
    (5, 1, 3, 0, 0), (33, 31, 70, 0, 1), (64, 32, 2048, 0, 0), (65, 32, 2048, 0, 0), (40, 33, 20, 0, 0),
    # 512 / 513 tiles and beyond: eight, four, two and one wave a tile
    (512, 130, 1024, 0, 0), (513, 130, 1000, 0, 0), (1024, 257, 1024, 0, 0), (1025, 40, 1020, 0, 0), (2048, 100, 1024, 0, 0), (2050, 300, 1030, 0, 1),
    # 64x64 tiles: fewer stages than the ring holds, more of them, ragged edges, interior tiles
    (64, 128, 64, 7, 0), (65, 256, 63, 7, 0), (128, 512, 192, 7, 0), (130, 640, 200, 7, 0), (192, 768, 256, 7, 0), (651, 1152, 130, 7, 0),
    # the rule's own choice on both sides of 256 small and 512 medium tiles
    (256, 256, 1024, 0, 0), (257, 256, 1024, 0, 0), (1024, 256, 2048, 0, 0), (1025, 256, 2048, 0, 0),
])
def test_small_and_ragged_gemm_equals_the_staged_kernel(q8, M, K, N, variant, off):
    g = synth.rng(9000 + M + K + N)
    xh, wh = synth.random_int8(g, (M, K)), synth.random_int8(g, (N, K))
    Kp = (K + 127) // 128 * 128
    pad = lambda a: torch.from_numpy(np.pad(a, ((0, 0), (0, Kp - K)))).cuda()
    xp, wp, x, w = pad(xh), pad(wh), at_offset(xh, off), at_offset(wh, off)
    b = torch.from_numpy(synth.bias(g, N)).cuda()
    res = torch.from_numpy(g.standard_normal((M, N)).astype(np.float32)).cuda()
    one = lambda v: torch.tensor([v], dtype=torch.float32, device="cuda")
    sx, sw, ns = one(24.0), one(900.0), one(9.0)
    guard = 64

    def run(v, x, w, flags, residual=False, dump=False):
        dt = torch.int8 if flags & 4 else torch.float32
        buf = torch.full((M * N + guard,), 77, dtype=dt, device="cuda")
        y, am = buf[:M * N].view(M, N), one(0.0)
        acc = torch.empty((M, N), dtype=torch.int32, device="cuda") if dump else None
        q8.set_gemm_variant(v)
        try:
            if residual:
                q8.q8_linear_residual(x, w, b, sx, sw, res, y, acc_out=acc, out_amax=am if flags & 2 else None, flags=flags)
            else:
                q8.q8_linear(x, w, b, sx, sw, y, acc_out=acc, out_amax=am if flags & 2 else None, next_scale=ns if flags & 4 else None, flags=flags)
        finally:
            q8.set_gemm_variant(0)
        torch.cuda.synchronize()
        assert bool((buf[M * N:] == 77).all()), "wrote behind y"
        return y, am.item(), acc

    for flags, residual in [(f, False) for f in range(8)] + [(0, True), (3, True)]:
        y, am, _ = run(variant, x, w, flags, residual)
        y_ref, am_ref, _ = run(3, xp, wp, flags, residual)
        assert torch.equal(y, y_ref) and am == am_ref, (flags, residual)
    _, _, acc = run(variant, x, w, 3, dump=True)
    bq = O.quantize_bias(b.cpu().numpy(), N, 24.0, [900.0])
    np.testing.assert_array_equal(acc.cpu().numpy(), O.gemm_i8(xh, wh, bq, threads=8))


@pytest.mark.parametrize("M,K,N,off", [(512, 130, 1024, 0), (513, 130, 1000, 0), (1024, 257, 1024, 0), (1025, 40, 1020, 0), (2048, 100, 1024, 0), (2050, 300, 1030, 1), (1100, 1024, 1000, 4)])
def test_direct_gemm_of_many_tiles_equals_the_staged_kernel(q8, M, K, N, off):
    """Eight, four, two and one wave a tile, whatever the automatic choice would take."""
    test_small_and_ragged_gemm_equals_the_staged_kernel(q8, M, K, N, 8, off)


@pytest.mark.parametrize("variant,bm,bn", [(9, 64, 64), (10, 64, 64), (11, 128, 64), (12, 128, 128), (13, 192, 128)])
@pytest.mark.parametrize("dm,dn,K", [(0, 0, 128), (1, 1, 256), (-1, -1, 384), (0, 7, 512), (33, 0, 1152)])
def test_ring_gemm_equals_the_staged_kernel(q8, variant, bm, bn, dm, dn, K):
    """The tiles with few stage buffers: fewer stages than buffers, as many, more; whole tiles, one row or column more or less."""
    test_small_and_ragged_gemm_equals_the_staged_kernel(q8, 2 * bm + dm, K, 3 * bn + dn, variant, 0)


@pytest.mark.parametrize("M,K,N", [(1100, 512, 500), (2050, 384, 1030), (2050, 1920, 520), (2050, 2048, 520), (4100, 256, 1540), (6200, 256, 2050), (2900, 128, 4100)])
def test_ring_gemm_choice_equals_the_staged_kernel(q8, M, K, N):
    """What the rule takes for ragged launches of a few to many tiles per compute unit."""
    test_small_and_ragged_gemm_equals_the_staged_kernel(q8, M, K, N, 0, 0)


@pytest.mark.parametrize("variant", [9, 10, 11, 12, 13])
@pytest.mark.parametrize("M,K,N,off", [(70, 4, 70, 0), (130, 36, 129, 4), (200, 124, 66, 8), (193, 132, 130, 12), (129, 256, 128, 4), (257, 500, 190, 0), (65, 1020, 64, 4)])
def test_ring_gemm_of_any_multiple_of_four(q8, variant, M, K, N, off):
    """Widths that end inside a stage, a 32-byte step or a 16-byte operand, rows 4 bytes aligned: what lies behind the end of K -- the
    next row, or nothing -- does not count."""
    test_small_and_ragged_gemm_equals_the_staged_kernel(q8, M, K, N, variant, off)


@pytest.mark.parametrize("M,K,N,off", [(777, 1000, 520, 0), (513, 36, 545, 4), (512, 1000, 512, 0), (544, 1000, 512, 0), (600, 2100, 500, 0), (700, 2100, 800, 0), (1024, 768, 520, 4), (1024, 998, 520, 0)])
def test_ring_gemm_choice_of_ragged_widths(q8, M, K, N, off):
    """Both sides of the rule: 256 and 272 tiles, short and long reductions, rows that are only 2-byte aligned."""
    test_small_and_ragged_gemm_equals_the_staged_kernel(q8, M, K, N, 0, off)


@pytest.mark.parametrize("M,K,N", [(2112, 128, 4096), (2100, 256, 4100), (3072, 384, 3000), (3073, 128, 4090)])
def test_gemm_choice_around_one_round_of_large_tiles(q8, M, K, N):
    """176 and 187 tiles of 192 x 256 rows and columns, 192, and more than 256."""
    test_small_and_ragged_gemm_equals_the_staged_kernel(q8, M, K, N, 0, 0)


@pytest.mark.parametrize("variant", [-1, 14, 99])
@pytest.mark.parametrize("M,K,N", [(300, 256, 300), (700, 600, 500), (40, 33, 40)])
def test_unknown_gemm_variant_is_an_error(q8, variant, M, K, N):
    """Whatever kernel the shape would get by itself: staged or with few stage buffers, the same for ragged widths, direct."""
    x, w = torch.zeros((M, K), dtype=torch.int8, device="cuda"), torch.zeros((N, K), dtype=torch.int8, device="cuda")
    one, y = torch.ones(1, device="cuda"), torch.full((M, N), 7.0, device="cuda")
    q8.set_gemm_variant(variant)
    try:
        with pytest.raises(RuntimeError, match="launch failed"):
            q8.q8_linear(x, w, None, one, one, y)
    finally:
        q8.set_gemm_variant(0)
    assert bool((y == 7.0).all())


@pytest.mark.parametrize("M,K,N", [(34000, 128, 64), (5000, 128, 840), (5000, 256, 839), (6000, 132, 1500), (12288, 128, 576), (12288, 512, 576), (3000, 512, 2816), (3000, 384, 2816), (3100, 512, 2816), (33000, 128, 2)])
def test_gemm_choice_of_narrow_and_full_rounds_of_large_tiles(q8, M, K, N):
    """176 to 256 tiles of 192 x 256 rows and columns that are a quarter, three quarters and all outputs; 32 MiB of them and less; short reductions."""
    test_small_and_ragged_gemm_equals_the_staged_kernel(q8, M, K, N, 0, 0)


@pytest.mark.parametrize("M,K,N", [(1024, 1152, 1024), (1025, 1152, 1024), (1024, 1024, 1000), (300, 1920, 2300), (3300, 1152, 2304), (3300, 1024, 2304), (3100, 1152, 2304), (3000, 640, 2816), (4097, 384, 2080), (4097, 512, 2080), (2100, 2048, 1500)])
def test_gemm_choice_of_longer_reductions(q8, M, K, N):
    """Both sides of the lines between the staged tiles and those with few buffers: 256 and 272 tiles of 64 x 64 and one stage less, a round of large tiles of 29 and 27 MiB,
    outputs stored for the caches of 384, 512 and 640, wide ones of broken lines."""
    test_small_and_ragged_gemm_equals_the_staged_kernel(q8, M, K, N, 0, 0)


@pytest.mark.parametrize("M,K,N", [(300, 640, 1000), (300, 644, 1000), (290, 1148, 1000), (290, 1156, 1000), (300, 1404, 1000), (300, 1412, 1000), (9000, 316, 20), (9000, 324, 20),
                                   (9000, 572, 32), (9000, 580, 32), (16400, 1604, 10)])
def test_gemm_choice_of_long_ragged_reductions(q8, M, K, N):
    """Both sides of the lines between the direct kernel and the tiles with few stage buffers, per kind of epilogue, in two rounds of 32 x 32 tiles and one
    tile more."""
    test_small_and_ragged_gemm_equals_the_staged_kernel(q8, M, K, N, 0, 0)


def time_of(q8, variant, M, K, N):
    """Microseconds of a plain layer, the smallest of several runs of ten, outputs past the caches."""
    x, w = (torch.randint(-127, 128, s, dtype=torch.int8, device="cuda") for s in ((M, K), (N, K)))
    one = torch.ones(1, device="cuda")
    ys = [torch.empty((M, N), device="cuda") for _ in range(max(2, min(8, (1 << 28) // (M * N))))]
    q8.set_gemm_variant(variant)
    try:
        times = []
        for _ in range(10):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for i in range(10):
                q8.q8_linear(x, w, None, one, one, ys[i % len(ys)])
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b) * 100.0)
        return min(times)
    finally:
        q8.set_gemm_variant(0)


@pytest.mark.parametrize("M,K,N", [(40000, 768, 64), (48000, 128, 128), (36000, 1024, 2), (36000, 768, 64), (30000, 512, 999)])
def test_gemm_choice_is_near_the_best_tile(q8, M, K, N):
    """Shapes that a rule written for another one would take: the automatic choice within a third of the best of the small tiles.  The measured
    times lie 0 to 15 % apart, those of a wrong rule 35 % and more."""
    best = min(time_of(q8, v, M, K, N) for v in (10, 11, 12))
    assert time_of(q8, 0, M, K, N) <= 1.33 * best
