"""The elementwise streams at every length modulo a 16-byte group and every
offset of each pointer from a 16-byte boundary, with guard elements around the
output that must stay as they are."""
import numpy as np
import pytest

import paper_2305_17190_amd as pam
import pam_workloads as wl
from gpu_util import device, note, to_dev
from oracle import pa_ref, pam_ref

pytestmark = pytest.mark.gpu

OPS = {"mul": (pam.mul, pam_ref.pam_mul_ref, 2), "pad": (pam.pad, pa_ref.pad_ref, 2),
       "palog2": (pam.palog2, pa_ref.palog2_ref, 1), "paexp2": (pam.paexp2, pa_ref.paexp2_ref, 1)}


@pytest.mark.parametrize("op", sorted(OPS))
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 1023, 1024, 1025, 1026, 1027, 4099])
def test_tails_and_offsets(op, n):
    import torch
    fn, ref, arity = OPS[op]
    host = [wl.random_bit_patterns(n, 60 + n + i) for i in range(arity)]
    want = ref(*host).view(np.uint32)
    for shifts in ((0, 0, 0), (1, 0, 0), (0, 2, 0), (0, 0, 3), (1, 3, 2), (3, 3, 3)):
        note(f"{op} n={n} offsets {shifts}")
        args = []
        for x, shift in zip(host, shifts):
            buf = torch.zeros(n + 8, device=device())
            buf[shift:shift + n] = to_dev(x)
            args.append(buf[shift:shift + n])
        out = torch.full((n + 8,), 7.0, device=device())
        fn(*args, out=out[shifts[2]:shifts[2] + n])
        got = out.cpu().numpy()
        assert np.array_equal(got[shifts[2]:shifts[2] + n].view(np.uint32), want)
        assert np.all(got[:shifts[2]] == 7.0) and np.all(got[shifts[2] + n:] == 7.0)
