"""moe_permute around the numbers of pairs (4096) and of 16-byte pieces of x (2^23) up to which one launch does all of it, the
numbers of pairs (1024, 2048) where its wavefronts take longer chunks, and the sizes where a thread copies to all slots of a
token, to some or to one: whole numbers, exact."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2602_11686_amd import binding as B
from gpu_common import host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,E,k,dtype", [(1, 8, 1, 1, torch.bfloat16), (1, 24, 256, 8, torch.bfloat16),
                                           (64, 2048, 128, 8, torch.bfloat16), (255, 136, 3, 1, torch.bfloat16),
                                           (1365, 20, 7, 3, torch.float32), (1366, 20, 7, 3, torch.float32),
                                           (4096, 64, 256, 1, torch.bfloat16), (4097, 64, 256, 1, torch.bfloat16),
                                           (819, 4, 65, 5, torch.float32), (512, 256, 16, 8, torch.bfloat16),
                                           (512, 8192, 6, 3, torch.bfloat16), (513, 8192, 6, 3, torch.bfloat16),
                                           (300, 8192, 70, 2, torch.float32),
                                           (128, 4096, 16, 8, torch.bfloat16), (129, 4096, 16, 8, torch.bfloat16),
                                           (1024, 1040, 9, 2, torch.bfloat16), (683, 1800, 30, 3, torch.bfloat16),
                                           (205, 5000, 256, 5, torch.bfloat16), (8, 4096, 8, 7, torch.bfloat16),
                                           (1024, 65536, 5, 1, torch.bfloat16), (1025, 65536, 5, 1, torch.bfloat16), (2048, 8200, 9, 2, torch.bfloat16)])
def test_permute(T, d, E, k, dtype):
    rng = np.random.default_rng(T + E)
    # skewed: low experts are picked more often, some not at all
    ids = np.stack([rng.choice(E, size=k, replace=False, p=None if t % 3 else np.linspace(2, 1, E) / np.linspace(2, 1, E).sum())
                    for t in range(T)]).astype(np.int32)
    x = torch.randn(T, d, device="cuda").to(dtype)
    counts, offsets, rop, por, _ = O.permute(np.zeros((T, d)), ids, E)
    s = B.Shape(T, d, 8, E, k, dtype)
    ws = torch.empty(B.moe_workspace_bytes(s), dtype=torch.uint8, device="cuda")
    for with_rows in (True, False):
        i32 = lambda n: torch.full((n,), -9, dtype=torch.int32, device="cuda")
        c, o, r, p = i32(E), i32(E + 1), i32(T * k), i32(T * k)
        xp = torch.full((T * k, d), float("nan"), dtype=dtype, device="cuda") if with_rows else None
        B.moe_permute(s, x, torch.from_numpy(ids).cuda(), c, o, r, p, xp, ws)
        for got, want in ((c, counts), (o, offsets), (r, rop), (p, por)):
            np.testing.assert_array_equal(host(got), want)
        if with_rows:
            assert torch.equal(xp, x[torch.from_numpy(np.asarray(por) // k).cuda().long()])
