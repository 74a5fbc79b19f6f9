"""Matrix products at the edges of the operand copies: rows shorter than the
16-byte pieces (four float32 or eight bfloat16 elements), last pieces that end
with the row, operands that start at any element, K tails of every length in
a chunk and K slices that end inside one, under every tile shape.  Everything
around an operand is NaN: a copy that took an element of it would show."""
import numpy as np
import pytest

import paper_2305_17190_amd as pam
from gpu_util import check_gemm, device, note, oracle_gemm, to_dev

pytestmark = pytest.mark.gpu

# (A whole-tile count beside one split changes nothing but keeps the plan from
# being the library's own, which a small product would not run.)
PLANS = [(128, 128, 1, 1, 1), (128, 64, 1, 1, 1), (128, 64, 1, 2, 1), (64, 64, 1, 1, 1), (64, 64, 1, 4, 1)]


def placed(x, shift, gap, dtype):
    """x on the GPU, `shift` elements into a NaN buffer, rows `gap` apart."""
    import torch
    rows, cols = x.shape
    buf = torch.full((shift + rows * (cols + gap) + 8,), float("nan"), dtype=dtype, device=device())
    view = buf[shift:shift + rows * (cols + gap)].view(rows, cols + gap)[:, :cols]
    view.copy_(to_dev(x).to(dtype))
    return view


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("ta,tb", [(False, False), (False, True), (True, False), (True, True)])
@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (3, 2, 3), (5, 3, 7), (7, 9, 5), (130, 6, 2), (2, 131, 9), (65, 67, 31),
                                   (129, 70, 47), (8, 4096 // 32, 77)])
def test_short_rows_and_tails(m, n, k, ta, tb, bf16):
    import torch
    dtype = torch.bfloat16 if bf16 else torch.float32
    g = np.random.default_rng(900 + m + n + k)
    a = g.standard_normal((k, m) if ta else (m, k)).astype(np.float32)
    b = g.standard_normal((n, k) if tb else (k, n)).astype(np.float32)
    if bf16:
        a, b = (torch.from_numpy(x).to(dtype).float().numpy() for x in (a, b))
    for shift, gap in ((0, 0), (1, 0), (3, 1), (2, 2)):
        note(f"edges m={m} n={n} k={k} ta={ta} tb={tb} bf16={bf16} shift={shift} gap={gap}")
        c = pam.gemm(placed(a, shift, gap, dtype), placed(b, shift, gap, dtype), trans_a=ta, trans_b=tb,
                     out=placed(np.zeros((m, n), np.float32), shift, gap, torch.float32))
        c_ref, s_ref = oracle_gemm(a.ravel(), b.ravel(), ta, tb, m, n, k, a.shape[1], b.shape[1], batches=[0])
        check_gemm(c.cpu().numpy()[None], c_ref, s_ref, k, "edges")


@pytest.mark.parametrize("plan", PLANS + [(128, 64, 3, 2, 0), (64, 64, 3, 4, 0), (128, 128, 2, 1, 1)])
@pytest.mark.parametrize("k", [3, 33, 101, 197])
def test_tails_under_every_tile_shape(k, plan):
    import torch
    m, n = 133, 131
    g = np.random.default_rng(950 + k)
    a, b = g.standard_normal((m, k)).astype(np.float32), g.standard_normal((k, n)).astype(np.float32)
    a[:, k // 2] = 0.0
    note(f"K tail k={k} plan={plan}")
    c = pam.bmm(placed(a, 1, 0, torch.float32)[None], placed(b, 1, 0, torch.float32)[None], plan=plan)
    c_ref, s_ref = oracle_gemm(a.ravel(), b.ravel(), False, False, m, n, k, k, n, batches=[0])
    check_gemm(c.cpu().numpy(), c_ref, s_ref, k, "tails")


@pytest.mark.parametrize("plan", PLANS + [(128, 64, 3, 2, 0), (64, 64, 3, 4, 0)])
@pytest.mark.parametrize("thin", [1, 2, 3, 5, 7])
@pytest.mark.parametrize("bf16", [False, True])
def test_operands_of_fewer_columns_than_a_piece(thin, plan, bf16):
    """Both operands not K-contiguous and thinner than a 16-byte piece: pieces run
    on over the rows' gaps (NaN here) and start earlier at the operand's end."""
    import torch
    dtype = torch.bfloat16 if bf16 else torch.float32
    for k, gap in ((1, 0), (2, 1), (17, 0), (64, 3), (129, 0), (200, 1)):
        g = np.random.default_rng(970 + k + thin)
        a, b = (g.standard_normal((k, c)).astype(np.float32) for c in (133, thin))
        a[k // 3] = 0.0
        if bf16:
            a, b = (torch.from_numpy(x).to(dtype).float().numpy() for x in (a, b))
        note(f"thin n={thin} k={k} gap={gap} plan={plan} bf16={bf16}")
        for x, y in ((a, b), (b, a)):
            m, n = x.shape[1], y.shape[1]
            xd, yd = placed(x, 1, gap, dtype), placed(y, 3, gap, dtype)
            c = pam.bmm(xd[None], yd[None], trans_a=True, plan=None if bf16 else plan)
            c_ref, s_ref = oracle_gemm(x.ravel(), y.ravel(), True, False, m, n, k, m, n, batches=[0])
            check_gemm(c.cpu().numpy(), c_ref, s_ref, k, "thin")
            if bf16:
                wide = pam.bmm(placed(x, 2, gap, torch.float32)[None], placed(y, 1, gap, torch.float32)[None], trans_a=True)
                assert torch.equal(c.view(torch.int32), wide.view(torch.int32))


def test_thin_operands_are_copied_beside_the_compute():
    """An operand of three columns against one of four: 1.47 times the time when
    its elements were loaded one by one before each chunk's compute, now 1.15."""
    import torch
    note("thin operand time")
    g = torch.Generator(device=device()).manual_seed(990)
    a = torch.randn((4096, 4096), generator=g, device=device())
    best = {}
    for _ in range(5):
        for n in (3, 4):
            b = torch.randn((4096, n), generator=g, device=device())
            pam.gemm(a, b)
            t0, t1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            t0.record()
            for _ in range(50):
                pam.gemm(a, b)
            t1.record()
            t1.synchronize()
            best[n] = min(best.get(n, 1e9), t0.elapsed_time(t1))
    print(best, flush=True)
    assert best[3] < 1.3 * best[4], best
