"""GPU parity of the two bandwidth-bound kernels on their own (accumulate, optimizer)."""
import numpy as np
import pytest

import oracle as O
import vf_inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 3, 4, 1023, 1024, 4096 + 5, 203530, 5_000_003])
def test_accumulate_matches_weighted_sum(n):
    import torch
    import paper_2009_09523_amd as vf
    print(f"accumulate n={n}", flush=True)
    sizes = [48, 48, 32, 32, 16, 16, 48, 16]
    off, w = O.partition(sizes, 256)
    g = I.make_flat_gradients(n, len(sizes))
    buf = torch.full((n,), 7.0, device="cuda")            # stale contents must be overwritten
    want32 = np.zeros(n, dtype=np.float32)
    want64 = np.zeros(n)
    for i in range(len(sizes)):
        gi = torch.from_numpy(g[i]).cuda()
        vf.vf_accumulate(buf, gi, float(w[i]), first=(i == 0))
        want64 += (sizes[i] / 256.0) * g[i].astype(np.float64)
    torch.cuda.synchronize()
    got = buf.cpu().numpy()
    assert np.max(np.abs(got - want64)) <= 1e-6 * np.max(np.abs(want64)) + 1e-7
    # the kernel's own order of operations: one fused multiply-add per node, in node order
    acc = np.zeros(n, dtype=np.float64)
    for i in range(len(sizes)):
        acc = (np.float64(w[i]) * g[i].astype(np.float64) + acc).astype(np.float32).astype(np.float64)
    np.testing.assert_array_equal(got, acc.astype(np.float32))


def test_accumulate_empty_and_misaligned():
    import torch
    import paper_2009_09523_amd as vf
    buf = torch.zeros(16, device="cuda")
    g = torch.ones(16, device="cuda")
    vf.vf_accumulate(buf[:0], g[:0], 1.0, first=True)       # n = 0 is a no-op
    with pytest.raises(vf.VfError):
        vf.vf_accumulate(buf[1:9], g[1:9], 1.0, first=True)  # not 16-byte aligned


@pytest.mark.parametrize("n", [5, 4096, 1_000_003])
def test_sgdm_kernel(n):
    import torch
    import paper_2009_09523_amd as vf
    rng = np.random.Generator(np.random.PCG64(n))
    th0 = rng.standard_normal(n).astype(np.float32)
    th, v = th0.astype(np.float64), np.zeros(n)
    tht, vt = torch.from_numpy(th0).cuda(), torch.zeros(n, device="cuda")
    for step in range(3):
        G = rng.standard_normal(n).astype(np.float32)
        vf.vf_sgdm_update(tht, vt, torch.from_numpy(G).cuda(), 0.1, 0.9)
        th, v = O.sgdm_update(th, G, v, 0.1, 0.9)
    torch.cuda.synchronize()
    np.testing.assert_allclose(tht.cpu().numpy(), th, rtol=1e-5, atol=1e-6)
    np.testing.assert_allclose(vt.cpu().numpy(), v, rtol=1e-5, atol=1e-6)


@pytest.mark.parametrize("n", [5, 4096, 1_000_003])
def test_adam_kernel(n):
    import torch
    import paper_2009_09523_amd as vf
    rng = np.random.Generator(np.random.PCG64(n + 1))
    th0 = rng.standard_normal(n).astype(np.float32)
    th, m, u = th0.astype(np.float64), np.zeros(n), np.zeros(n)
    tht = torch.from_numpy(th0).cuda()
    mt, ut = torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")
    for t in range(1, 4):
        G = rng.standard_normal(n).astype(np.float32)
        vf.vf_adam_update(tht, mt, ut, torch.from_numpy(G).cuda(), 1e-3, 0.9, 0.999, 1e-8, t)
        th, m, u = O.adam_update(th, G, m, u, t, 1e-3, 0.9, 0.999, 1e-8)
    torch.cuda.synchronize()
    # beta2 arrives as an fp32 value: 1 - float32(0.999) differs from 0.001 by 1.3e-5 relative
    np.testing.assert_allclose(tht.cpu().numpy(), th, rtol=1e-5, atol=1e-6)
    np.testing.assert_allclose(mt.cpu().numpy(), m, rtol=1e-5, atol=1e-7)
    np.testing.assert_allclose(ut.cpu().numpy(), u, rtol=5e-5, atol=1e-9)


def test_flat_kernels_on_vectors_beyond_the_cache():
    """Vectors of 64 MB and more take the kernels' non-temporal form (here 256 MB): accumulate (two nodes, bit for bit
    against its fma chain), SGD-momentum and Adam (one step each against the oracle), ragged tail included."""
    import torch
    import paper_2009_09523_amd as vf
    n = (64 << 20) + 5
    print(f"flat kernels n={n}", flush=True)
    rng = np.random.Generator(np.random.PCG64(77))
    g0 = rng.standard_normal(n, dtype=np.float32)
    g1 = rng.standard_normal(n, dtype=np.float32)
    w = [np.float32(48) / np.float32(256), np.float32(208) / np.float32(256)]
    buf = torch.full((n,), 7.0, device="cuda")
    vf.vf_accumulate(buf, torch.from_numpy(g0).cuda(), float(w[0]), first=True)
    vf.vf_accumulate(buf, torch.from_numpy(g1).cuda(), float(w[1]), first=False)
    torch.cuda.synchronize()
    acc = (np.float64(w[0]) * g0.astype(np.float64)).astype(np.float32).astype(np.float64)
    acc = (np.float64(w[1]) * g1.astype(np.float64) + acc).astype(np.float32)
    G = buf.cpu().numpy()
    np.testing.assert_array_equal(G, acc)
    del acc
    th0 = rng.standard_normal(n, dtype=np.float32)
    tht, vt = torch.from_numpy(th0).cuda(), torch.zeros(n, device="cuda")
    vf.vf_sgdm_update(tht, vt, buf, 0.1, 0.9)
    th, v = O.sgdm_update(th0.astype(np.float64), G, np.zeros(n), 0.1, 0.9)
    torch.cuda.synchronize()
    np.testing.assert_allclose(tht.cpu().numpy(), th, rtol=1e-5, atol=1e-6)
    np.testing.assert_allclose(vt.cpu().numpy(), v, rtol=1e-5, atol=1e-6)
    del th, v
    tht, mt, ut = torch.from_numpy(th0).cuda(), torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")
    vf.vf_adam_update(tht, mt, ut, buf, 1e-3, 0.9, 0.999, 1e-8, 1)
    th, m, u = O.adam_update(th0.astype(np.float64), G, np.zeros(n), np.zeros(n), 1, 1e-3, 0.9, 0.999, 1e-8)
    torch.cuda.synchronize()
    np.testing.assert_allclose(tht.cpu().numpy(), th, rtol=1e-5, atol=1e-6)
    np.testing.assert_allclose(mt.cpu().numpy(), m, rtol=1e-5, atol=1e-7)
    np.testing.assert_allclose(ut.cpu().numpy(), u, rtol=5e-5, atol=1e-9)


GEMM_SHAPES = [(128, 4096 // 8, 1024 // 4), (48, 1000, 520), (16, 392, 1000), (8, 520, 256), (40, 264, 392),
               (300, 100, 392), (392, 1000, 128), (520, 392, 48), (256, 520, 16), (256, 520, 8), (1, 8, 8),
               (33, 65, 72), (129, 257, 264), (304, 1003, 128), (2048, 2304, 768),
               # the 256-row LDS-direct kernel, ragged on both sides, 256 x 128 tiles ...
               (4000, 3585, 192),
               # ... and 256 x 256 tiles (exactly one round of 256 tiles: the whole-line kernel), with
               # three, one and two stages of 64
               (4000, 3900, 192), (3900, 4000, 64), (4000, 3900, 128)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("M,N,K", GEMM_SHAPES)
def test_gemm_against_float64_matmul(M, N, K, dtype):
    """C = alpha A B^T (+C) on ragged shapes: several tiles, row/column/contraction tails."""
    import torch
    import paper_2009_09523_amd as vf
    print(f"gemm {dtype} M={M} N={N} K={K}", flush=True)
    rng = np.random.Generator(np.random.PCG64(M * 7 + N * 3 + K))
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    lda = ((K + 7) // 8) * 8 + 8
    A = torch.from_numpy(rng.standard_normal((M, lda)).astype(np.float32)).to(tdt).cuda()
    B = torch.from_numpy(rng.standard_normal((N, lda)).astype(np.float32)).to(tdt).cuda()
    C0 = rng.standard_normal((M, N + 3)).astype(np.float32)
    Cd = torch.from_numpy(C0).cuda()
    A64, B64 = A[:, :K].double().cpu().numpy(), B[:, :K].double().cpu().numpy()
    want = A64 @ B64.T
    vf.vf_gemm(A[:, :K], B[:, :K], Cd[:, :N], M, N, K, alpha=0.75, accumulate=False)
    torch.cuda.synchronize()
    got = Cd.cpu().numpy()
    tol = 2e-5 * np.sqrt(K) * np.max(np.abs(want)) if dtype == "f32" else 1e-5 * np.max(np.abs(want)) * np.sqrt(K)
    assert np.max(np.abs(got[:, :N] - 0.75 * want)) <= tol
    np.testing.assert_array_equal(got[:, N:], C0[:, N:])          # nothing written past column N
    vf.vf_gemm(A[:, :K], B[:, :K], Cd[:, :N], M, N, K, alpha=-0.5, accumulate=True)
    torch.cuda.synchronize()
    got2 = Cd.cpu().numpy()
    assert np.max(np.abs(got2[:, :N] - 0.25 * want)) <= 2 * tol


@pytest.mark.parametrize("M,N,K,nsplit", [(128, 512, 4096, 16), (48, 1000, 520, 3), (16, 392, 1000, 4),
                                         (128, 264, 72, 2), (300, 100, 1000, 8),
                                         # whole 64-element stages per slice: the LDS-direct kernel
                                         (128, 4096, 4096, 4), (100, 1000, 1024, 8), (70, 130, 192, 3),
                                         (65, 64, 64, 1), (48, 392, 64, 2), (128, 1000, 4096, 16),
                                         # 256 x 256 tiles, sliced contraction
                                         (1100, 1030, 2048, 16),
                                         # the whole-line kernel (one round of 256 x 256 tiles), slices of 4 and 3 stages
                                         (4000, 3900, 1024, 4), (4000, 3900, 384, 2)])
def test_gemm_split_contraction_slabs_sum_to_product(M, N, K, nsplit):
    import torch
    import paper_2009_09523_amd as vf
    print(f"gemm split M={M} N={N} K={K} nsplit={nsplit}", flush=True)
    rng = np.random.Generator(np.random.PCG64(M + N + K))
    A = torch.from_numpy(rng.standard_normal((M, K)).astype(np.float32)).to(torch.bfloat16).cuda()
    B = torch.from_numpy(rng.standard_normal((N, K)).astype(np.float32)).to(torch.bfloat16).cuda()
    ldc = N + 5
    Cd = torch.full((nsplit, M, ldc), 3.0, device="cuda")
    vf.vf_gemm(A, B, Cd, M, N, K, nsplit=nsplit)
    torch.cuda.synchronize()
    got = Cd.cpu().numpy().astype(np.float64)
    want = A.double().cpu().numpy() @ B.double().cpu().numpy().T
    assert np.all(got[:, :, N:] == 3.0)
    assert np.max(np.abs(got[:, :, :N].sum(axis=0) - want)) <= 1e-5 * np.sqrt(K) * np.max(np.abs(want))


@pytest.mark.parametrize("M,N,K", [(8, 32, 10), (128, 64, 10), (3, 64, 10), (64, 10, 127), (40, 24, 75)])
def test_gemm_ragged_contraction_with_cold_operands(M, N, K):
    """A contraction length that is no multiple of 8 (the last 16-byte vector of a row is masked
    by element), with the operands pushed out of the caches before every launch: the masking must
    not depend on when the loads land."""
    import torch
    import paper_2009_09523_amd as vf
    print(f"gemm cold M={M} N={N} K={K}", flush=True)
    rng = np.random.Generator(np.random.PCG64(M * 11 + N * 5 + K))
    lda = ((K + 7) // 8) * 8
    A = torch.from_numpy(rng.standard_normal((M, lda)).astype(np.float32)).to(torch.bfloat16).cuda()
    B = torch.from_numpy(rng.standard_normal((N, lda)).astype(np.float32)).to(torch.bfloat16).cuda()
    want = A[:, :K].double().cpu().numpy() @ B[:, :K].double().cpu().numpy().T
    flush = torch.empty(768 * 1024 * 1024 // 4, device="cuda")        # larger than every cache level
    first = None
    for k in range(20):
        Cd = torch.full((M, N), 5.0, device="cuda")
        flush.fill_(float(k))
        vf.vf_gemm(A[:, :K], B[:, :K], Cd, M, N, K)
        torch.cuda.synchronize()
        got = Cd.cpu().numpy()
        assert np.max(np.abs(got - want)) <= 1e-5 * np.sqrt(K) * np.max(np.abs(want)), k
        if first is None:
            first = got
        assert got.tobytes() == first.tobytes(), k


@pytest.mark.parametrize("M,N,K,nsplit", [(70, 131, 193, 1), (64, 66, 63, 1), (200, 130, 1000, 3), (65, 64, 130, 4),
                                         (300, 1003, 71, 1), (700, 2000, 321, 1), (700, 3000, 321, 1), (768, 6144, 321, 1),
                                         (3000, 700, 131, 1), (1030, 4100, 1001, 2), (4096, 4100, 211, 1), (515, 2050, 2049, 8)])
def test_gemm_bf16_contraction_tails(M, N, K, nsplit):
    """Contraction slices that are no whole number of 64-element stages, on the 64 x 64 kernels and on the 256-row one
    (and slices with no element at all): what lies in the rows' padding (here NaN) must not be read into the product."""
    import torch
    import paper_2009_09523_amd as vf
    print(f"gemm bf16 tail M={M} N={N} K={K} nsplit={nsplit}", flush=True)
    gen = torch.Generator().manual_seed(M + 3 * N + 7 * K)
    ld = (K + 7) // 8 * 8 + 8
    A, B = torch.full((M, ld), float("nan")), torch.full((N, ld), float("nan"))
    A[:, :K] = torch.randn((M, K), generator=gen)
    B[:, :K] = torch.randn((N, K), generator=gen)
    A, B = A.to(torch.bfloat16), B.to(torch.bfloat16)
    Cd = torch.full((nsplit, M, N), 3.0, device="cuda")
    vf.vf_gemm(A.cuda()[:, :K], B.cuda()[:, :K], Cd if nsplit > 1 else Cd[0], M, N, K, nsplit=nsplit)
    torch.cuda.synchronize()
    a, b = A[:, :K].double(), B[:, :K].double()
    # exact products, fp32 sums: at most K roundings of partial sums no larger than sum |a||b|
    bound = K * 2.0 ** -24 * (a.abs() @ b.abs().T)
    assert torch.all((Cd.double().sum(0).cpu() - a @ b.T).abs() <= bound)


@pytest.mark.parametrize("pad", [0, 1, 4])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (16, 256, 784), (17, 33, 65), (31, 10, 3), (100, 500, 1000), (784, 65, 16),
                                   (256, 769, 256), (256, 1601, 40), (36, 256, 4099), (515, 1024, 515), (1000, 1100, 200),
                                   (1030, 2100, 20)])
def test_gemm_f32_tiles(M, N, K, pad):
    """Every tile of the fp32 product at its edges: rows, columns and contractions that end inside a tile, a
    chunk, a 16-byte vector; what lies in the rows' padding (here NaN) must not be read into the product."""
    import torch
    import paper_2009_09523_amd as vf
    print(f"gemm f32 M={M} N={N} K={K} pad={pad}", flush=True)
    rng = np.random.Generator(np.random.PCG64(M + 3 * N + 7 * K + pad))
    A = np.full((M, K + pad), np.nan, np.float32)
    B = np.full((N, K + pad), np.nan, np.float32)
    A[:, :K] = rng.standard_normal((M, K))
    B[:, :K] = rng.standard_normal((N, K))
    C0 = rng.standard_normal((M, N + 2)).astype(np.float32)
    Cd = torch.from_numpy(C0).cuda()
    vf.vf_gemm(torch.from_numpy(A).cuda()[:, :K], torch.from_numpy(B).cuda()[:, :K], Cd[:, :N], M, N, K, alpha=0.5,
               accumulate=True)
    torch.cuda.synchronize()
    got = Cd.cpu().numpy()
    a, b = A[:, :K].astype(np.float64), B[:, :K].astype(np.float64)
    # fp32 sums of K products: at most K roundings of partial sums no larger than sum |a||b|
    bound = K * 2.0 ** -24 * 0.5 * (np.abs(a) @ np.abs(b).T) + 2.0 ** -23 * (1 + np.abs(C0[:, :N]))
    assert np.all(np.abs(got[:, :N] - (0.5 * (a @ b.T) + C0[:, :N])) <= bound + 2.0 ** -23 * np.abs(a @ b.T))
    np.testing.assert_array_equal(got[:, N:], C0[:, N:])


def _time_us(f, repeats=5):
    """The fastest of a few runs of f, in microseconds."""
    import torch
    f()
    best = float("inf")
    for _ in range(repeats):
        a, b = torch.cuda.Event(True), torch.cuda.Event(True)
        a.record(), f(), b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3)
    return best


@pytest.mark.parametrize("M,N,K,limit_us", [(5, 13, 4099, None), (65, 130, 33, None), (64, 8192, 1024, 700)])
def test_gemm_f32_of_operands_out_of_32_bit_reach(M, N, K, limit_us):
    """Rows 32 MB and more apart: a workgroup of the kernel with 32-bit offsets cannot reach them.  Right, and as fast as
    the tiled kernel is (64 x 8192 x 1024: 197 us; one thread per output took 1695 us, and the forward product of a
    weight of 2 GiB, 64 x 32768 x 16384, 27 ms instead of 4)."""
    import torch
    import paper_2009_09523_amd as vf
    print(f"gemm f32 far M={M} N={N} K={K}", flush=True)
    pitch = (1 << 23) + 3
    gen = torch.Generator().manual_seed(5)
    A = torch.empty(M * pitch, device="cuda").as_strided((M, K), (pitch, 1))
    a, B = torch.randn((M, K), generator=gen), torch.randn((N, K), generator=gen)
    A.copy_(a)
    C0 = torch.randn((M, N), generator=gen)
    Bd, C = B.cuda(), C0.cuda()
    vf.vf_gemm(A, Bd, C, M, N, K, alpha=0.5, accumulate=True)
    torch.cuda.synchronize()
    exact = a.double() @ B.double().T
    # fp32 sums of K products: at most K roundings of partial sums no larger than sum |a||b|
    bound = K * 2.0 ** -24 * 0.5 * (a.abs().double() @ B.abs().double().T) + 2.0 ** -23 * (1 + C0.abs() + exact.abs())
    assert torch.all((C.cpu().double() - (0.5 * exact + C0.double())).abs() <= bound)
    if limit_us:
        us = _time_us(lambda: vf.vf_gemm(A, Bd, C, M, N, K))
        assert us < limit_us, us


@pytest.mark.parametrize("M,N,K,ratio", [(8192, 8192, 16, 3.2), (4096, 4096, 64, 4.3), (8192, 8192, 255, 12.5)])
def test_gemm_f32_of_a_short_contraction_keeps_up_with_memory(M, N, K, ratio):
    """A large result over few elements is bound by reading and writing the result: its time as a multiple of what an
    element-wise pass over as much memory takes on the same card: 2.1, 3.1 and 8.5 (as on the tiled kernel alone); 4.9, 5.7
    and 18 when four wavefronts shared a 64 x 64 tile whose contraction only one of them had anything of.  The limits
    lie halfway (on the logarithm).  255: no vector reads."""
    import torch
    import paper_2009_09523_amd as vf
    print(f"gemm f32 short M={M} N={N} K={K}", flush=True)
    A, B, C = torch.randn((M, K), device="cuda"), torch.randn((N, K), device="cuda"), torch.zeros((M, N), device="cuda")
    product = _time_us(lambda: [vf.vf_gemm(A, B, C, M, N, K, accumulate=True) for _ in range(4)])
    add = _time_us(lambda: [C.add_(1.0) for _ in range(4)])
    print(f"{product / 4:.1f} us, {product / add:.2f} of the pass", flush=True)
    assert product < ratio * add


def test_gemm_bf16_of_operands_of_2_gib():
    """Rows of an operand further than 2 GiB apart, on the 128 x 128 tiles: the first and the last rows' products (the
    operand's last element is 2.1 GiB behind its first)."""
    import torch
    import paper_2009_09523_amd as vf
    M, N, K, pitch = 1100, 1030, 520, 1024000
    print(f"gemm bf16 far M={M} N={N} K={K} pitch={pitch}", flush=True)
    gen = torch.Generator().manual_seed(3)
    a, b = (torch.randn((r, K), generator=gen).to(torch.bfloat16) for r in (M, N))
    A = torch.empty(M * pitch, device="cuda", dtype=torch.bfloat16).as_strided((M, K), (pitch, 1))
    A.copy_(a)
    C = torch.zeros((M, N), device="cuda")
    vf.vf_gemm(A, b.cuda(), C, M, N, K)
    torch.cuda.synchronize()
    a, b = a.double(), b.double()
    # exact products, fp32 sums: at most K roundings of partial sums no larger than sum |a||b|
    assert torch.all((C.double().cpu() - a @ b.T).abs() <= K * 2.0 ** -24 * (a.abs() @ b.abs().T))
