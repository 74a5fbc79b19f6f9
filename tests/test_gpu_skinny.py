"""Products with few rows of op(A) or columns of op(B), both K-contiguous:
their own kernel, against the oracle and against the tiled path (the same
product with another plan forced), over row counts around its blocks of 4, 8 and
16, ragged widths and K, element types, mantissa bits, batches and strides,
unaligned views, and operand values of every class."""
import numpy as np
import pytest

import paper_2305_17190_amd as pam
import pam_workloads as wl
from gpu_util import check_gemm, device, note, oracle_gemm, to_dev
from oracle import pam_ref

pytestmark = pytest.mark.gpu


def run_both(a, b, bits=23):
    """The product by the library's choice and by a forced plan (which, with a
    whole-tile count, is no plan of the library's own)."""
    c = pam.bmm(a, b, trans_b=True, mantissa_bits=bits)
    tiled = pam.bmm(a, b, trans_b=True, plan=(64, 64, 1, 4, 1))
    return c.cpu().numpy(), tiled.cpu().numpy()


@pytest.mark.parametrize("few", [1, 3, 4, 5, 8, 9, 16, 17, 32, 33])
@pytest.mark.parametrize("wide,k", [(1, 1), (15, 63), (17, 64), (130, 65), (300, 515), (64, 1030)])
@pytest.mark.parametrize("swap", [False, True])
def test_row_counts_widths_and_k(few, wide, k, swap):
    m, n = (wide, few) if swap else (few, wide)
    g = np.random.default_rng(1000 + few + wide + k)
    a, b = g.standard_normal((m, k)).astype(np.float32), g.standard_normal((n, k)).astype(np.float32)
    a[g.random(a.shape) < 0.2] = 0.0
    note(f"skinny m={m} n={n} k={k}")
    c, tiled = run_both(to_dev(a)[None], to_dev(b)[None])
    c_ref, s_ref = oracle_gemm(a.ravel(), b.ravel(), False, True, m, n, k, k, k, batches=[0])
    check_gemm(c, c_ref, s_ref, k, "skinny")
    check_gemm(tiled, c_ref, s_ref, k, "tiled")
    if few <= 32 and k >= 515 and m * n >= 64:   # two kernels: their sums have another order
        assert not np.array_equal(c, tiled)


@pytest.mark.parametrize("few,wide,k", [(1, 40, 16384), (3, 35, 16385), (7, 20, 33000), (12, 17, 40000)])
def test_long_k_folds_its_sums(few, wide, k):
    """A lane's sum is folded into the outputs every 32 chunks of 512 k steps:
    sums that are exact in any order equal the oracle bit for bit.  (Without a
    workspace, so that the product's plan has no K slices to win with.)"""
    import torch
    note(f"skinny long K few={few} wide={wide} k={k}")
    a, b = wl.exact_sum_values((few, k), 1250), wl.exact_sum_values((wide, k), 1251)
    ad, bd = to_dev(a), to_dev(b)
    c = torch.full((few, wide), float("nan"), device=device())
    st = pam.load().pam_gemm_batched(0, 1, few, wide, k, ad.data_ptr(), k, 0, bd.data_ptr(), k, 0, c.data_ptr(), wide, 0,
                                     1, torch.cuda.current_stream().cuda_stream)
    assert st == 0
    c_ref, _ = oracle_gemm(a, b, False, True, few, wide, k, k, k)
    assert np.array_equal(c.cpu().numpy().astype(np.float64), c_ref[0])


def best_times(products):
    """Least time of 20 calls of each of the products, in turn."""
    import torch
    best = {}
    for _ in range(5):
        for name, (x, w) in products.items():
            pam.gemm(x, w, trans_b=True)
            t0, t1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            t0.record()
            for _ in range(20):
                pam.gemm(x, w, trans_b=True)
            t1.record()
            t1.synchronize()
            best[name] = min(best.get(name, 1e9), t0.elapsed_time(t1))
    print(best, flush=True)
    return best


@pytest.mark.parametrize("few", [8, 32])
def test_tiny_values_do_not_take_the_complete_definition(few):
    """Tiny normals cost a rounding more per term, as in the tiled kernel, not
    the complete definition of every term near them (which took 6 to 10 times as
    long): at most 3 times the time of clean operands."""
    import torch
    note(f"skinny tiny values few={few}")
    g = torch.Generator(device=device()).manual_seed(1260)
    x = torch.randn((few, 4096), generator=g, device=device())
    w = torch.randn((4096, 4096), generator=g, device=device())
    spiced = torch.where(torch.rand(w.shape, generator=g, device=device()) < 1e-3, torch.full_like(w, 1.5e-38), w)
    best = best_times({"clean": (x, w), "tiny": (x, spiced)})
    assert best["tiny"] < 3.0 * best["clean"], best


@pytest.mark.parametrize("few", [8, 16])
def test_bf16_takes_no_longer_than_float32(few):
    """bfloat16 weights are half the bytes and the same work: not 1.25 times the
    time of float32 ones (1.5 times when their loads were waited for at once)."""
    import torch
    note(f"skinny bf16 time few={few}")
    g = torch.Generator(device=device()).manual_seed(1270)
    x, w = (torch.randn((r, 4096), generator=g, device=device()).to(torch.bfloat16) for r in (few, 4096))
    best = best_times({"bf16": (x, w), "float32": (x.float(), w.float())})
    assert best["bf16"] < 1.25 * best["float32"], best


@pytest.mark.parametrize("few", [2, 7, 12])
@pytest.mark.parametrize("bits", [23, 7, 3])
def test_batches_strides_and_narrow_mantissas(few, bits):
    import torch
    batch, n, k = 5, 70, 90
    g = np.random.default_rng(1100 + few + bits)
    a = g.standard_normal((batch, few, k)).astype(np.float32)
    b = g.standard_normal((batch, n, k)).astype(np.float32)
    note(f"skinny batch few={few} bits={bits}")
    # rows one element past alignment, gaps between rows and matrices
    abuf = torch.full((batch, few + 1, k + 3), float("nan"), device=device())
    abuf[:, :few, 1:k + 1] = to_dev(a)
    bbuf = torch.full((batch, n + 2, k + 1), float("nan"), device=device())
    bbuf[:, :n, :k] = to_dev(b)
    out = torch.full((batch, few, n + 1), float("nan"), device=device())[:, :, :n]
    pam.bmm(abuf[:, :few, 1:k + 1], bbuf[:, :n, :k], trans_b=True, out=out, mantissa_bits=bits)
    ar, br = (a, b) if bits == 23 else (pam_ref.round_mantissa_ref(x, bits) for x in (a, b))
    c_ref, s_ref = oracle_gemm(ar, br, False, True, few, n, k, k, k, few * k, n * k, batches=list(range(batch)))
    check_gemm(out.cpu().numpy(), c_ref, s_ref, k, f"skinny batch bits={bits}")
    # a zero stride broadcasts an operand
    one = pam.bmm(abuf[:1, :few, 1:k + 1].expand(batch, few, k), bbuf[:, :n, :k], trans_b=True, mantissa_bits=bits)
    assert torch.equal(one[0].view(torch.int32), out[0].contiguous().view(torch.int32))


@pytest.mark.parametrize("few,n,k", [(1, 40, 700), (6, 33, 130), (16, 260, 77)])
def test_bf16_equals_the_widened_product(few, n, k):
    import torch
    g = torch.Generator().manual_seed(1200 + few)
    a = torch.randn((few, k), generator=g).to(torch.bfloat16).to(device())
    b = torch.randn((n, k), generator=g).to(torch.bfloat16).to(device())
    note(f"skinny bf16 few={few} n={n} k={k}")
    for x, y in ((a, b), (b, a)):
        c16, c32 = pam.gemm(x, y, trans_b=True), pam.gemm(x.float(), y.float(), trans_b=True)
        assert torch.equal(c16.view(torch.int32), c32.view(torch.int32))


@pytest.mark.parametrize("few", [1, 4, 11])
@pytest.mark.parametrize("kind", ["finite", "huge", "nonfinite"])
def test_every_operand_class(few, kind):
    """Zeros, denormals, tiny and boundary values; then |x| >= 2^64 (in A only:
    no partial sum overflows); then inf and NaN too."""
    n, k = 50, 150
    g = np.random.default_rng(1300 + few)
    pats = wl.special_bit_patterns()
    mag = np.abs(pats)
    pats = pats[mag < 2.0 ** 64] if kind == "finite" else pats[mag < 2.0 ** 66] if kind == "huge" else \
        pats[~((mag >= 2.0 ** 64) & np.isfinite(pats))]
    a = g.standard_normal((few, k)).astype(np.float32)
    b = g.standard_normal((n, k)).astype(np.float32)
    for x in (a, b) if kind != "huge" else (a,):
        pick = g.random(x.shape) < (0.3 if kind == "finite" else 0.02)
        x[pick] = g.choice(pats, size=int(pick.sum()))
    note(f"skinny classes few={few} kind={kind}")
    c_ref, s_ref = oracle_gemm(a.ravel(), b.ravel(), False, True, few, n, k, k, k, batches=[0])
    c, tiled = run_both(to_dev(a)[None], to_dev(b)[None])
    check_gemm(c, c_ref, s_ref, k, f"skinny {kind}")
    check_gemm(tiled, c_ref, s_ref, k, f"tiled {kind}")
