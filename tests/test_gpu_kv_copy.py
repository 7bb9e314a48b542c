"""sd_kv_write / sd_kv_read move bytes exactly: ragged starts and ends within a
page, whole pages, more pages than one launch carries, caller rows that are
only 2-byte aligned (the element-wise kernel), and no neighbour touched."""
import numpy as np
import pytest
import torch

import workload as wl
from gpu_harness import make_verifier
from workload.device import DeviceWeights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shift", [0, 1, 4])  # elements the caller's buffers are off a 256-byte boundary
@pytest.mark.parametrize("pos0,n", [(0, 1), (0, 16), (3, 9), (5, 11), (15, 2), (16, 16), (7, 300), (0, 4200), (33, 4150)])
def test_rows_round_trip(pos0, n, shift):
    m = wl.MODELS["tiny-bf16"]
    P = pos0 + n + 5
    w = wl.custom_workload("tiny-bf16", [P, 64], [1, 1], seed=3)
    dw = DeviceWeights(m, w.seed)
    v = make_verifier(w, dw)
    per = m.n_kv_heads * m.head_dim
    g = torch.Generator(device="cuda").manual_seed(100 * pos0 + n)

    def rows(cnt):
        flat = torch.randint(-30000, 30000, (cnt * per + shift,), dtype=torch.int16, device="cuda", generator=g)
        return flat[shift:].view(cnt, m.n_kv_heads, m.head_dim)

    def read(u, cnt):
        k, x = rows(cnt), rows(cnt)
        v.read_kv(u, 1, 0, k, x)
        return k.cpu().numpy(), x.cpu().numpy()

    k0, v0, ko, vo = rows(P), rows(P), rows(64), rows(64)
    v.reset_user(0, P, 0)
    v.reset_user(1, 64, 0)
    v.write_kv(0, 1, 0, k0, v0)
    v.write_kv(1, 1, 0, ko, vo)
    k1, v1 = rows(n), rows(n)
    v.write_kv(0, 1, pos0, k1, v1)
    ek, ev = k0.cpu().numpy().copy(), v0.cpu().numpy().copy()
    ek[pos0:pos0 + n], ev[pos0:pos0 + n] = k1.cpu().numpy(), v1.cpu().numpy()
    gk, gv = read(0, P)
    assert np.array_equal(gk, ek) and np.array_equal(gv, ev)
    gk, gv = read(1, 64)
    assert np.array_equal(gk, ko.cpu().numpy()) and np.array_equal(gv, vo.cpu().numpy())
    # a ragged read writes its own rows only
    k2, v2 = rows(n + 2), rows(n + 2)
    a, b = k2.cpu().numpy(), v2.cpu().numpy()
    v.read_kv(0, 1, pos0, k2[1:n + 1], v2[1:n + 1])
    a[1:n + 1], b[1:n + 1] = ek[pos0:pos0 + n], ev[pos0:pos0 + n]
    assert np.array_equal(k2.cpu().numpy(), a) and np.array_equal(v2.cpu().numpy(), b)
    v.close()
