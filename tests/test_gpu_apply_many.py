"""The aggregated apply where its two forms meet (21 M parameters and more: longer stretches of every stream) and at partly filled last
workgroups of either, against single applies and pulls: the same bits."""
import ctypes

import pytest

from paper_1908_11848_amd import binding as B
from gpu_util import empty, stream_ptr

pytestmark = pytest.mark.gpu
LINE = 5 * 2 ** 22


@pytest.mark.parametrize("n", [1, 3, 4, 1000, 1023, 1024, 1027, 50_001, LINE - 4, LINE - 1, LINE, LINE + 3, LINE + 4, LINE + 8 * 1024 + 2049 * 4 + 1, LINE + 7 * 8192 - 4])
@pytest.mark.parametrize("m,after", [(1, [1, 1]), (3, [2, 3]), (16, [1, 16, 16])])
def test_same_bits_as_single_applies(n, m, after):
    import torch
    g = torch.Generator(device="cuda").manual_seed(n + m)
    w = torch.randn(n, device="cuda", generator=g)
    G = [1e-2 * torch.randn(n, device="cuda", generator=g) for _ in range(m)]
    torch.cuda.synchronize()
    L, s, nd = B.lib(), stream_ptr(), len(after)
    w1, w2, stamps = w.clone(), w.clone(), torch.zeros(2 + 2 * nd, dtype=torch.int64, device="cuda")
    one, many = [empty(n) for _ in after], [empty(n) for _ in after]
    for j in range(m):
        assert L.dsspk_apply(s, w1.data_ptr(), G[j].data_ptr(), n, 0.01, stamps.data_ptr(), 7 + j) == 0
        for d, a in enumerate(after):
            if a == j + 1:
                assert L.dsspk_pull(s, one[d].data_ptr(), w1.data_ptr(), n, stamps[2 + d:].data_ptr(), stamps.data_ptr()) == 0
    ptr = lambda ts: (ctypes.c_void_p * len(ts))(*[t.data_ptr() for t in ts])
    assert L.dsspk_apply_many(s, w2.data_ptr(), m, ptr(G), n, 0.01, nd, ptr(many), (ctypes.c_int * nd)(*after),
                              ptr([stamps[2 + nd + d:] for d in range(nd)]), stamps[1:].data_ptr(), 7) == 0
    torch.cuda.synchronize()
    assert torch.equal(w1, w2) and all(torch.equal(a, b) for a, b in zip(one, many))
    st = stamps.tolist()
    assert st[0] == st[1] == 6 + m and st[2:2 + nd] == st[2 + nd:]
