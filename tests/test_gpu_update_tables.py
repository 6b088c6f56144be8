"""Many-tensor update at the counts where its argument table changes size (4, 16 and 48 tensors per launch): every tensor
must come out with the bits of the single-tensor update, which is held against the oracle elsewhere."""
import numpy as np
import pytest
import torch

from paper_1710_03740_amd import binding as mpt

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grad32", [False, True])
@pytest.mark.parametrize("count", [1, 4, 5, 16, 17, 48, 49])
def test_every_tensor_is_updated_as_by_itself(count, grad32):
    g = torch.Generator(device="cuda").manual_seed(count)
    entries, single = [], []
    for k in range(count):
        n = 1 + (k * 37) % 600
        w = torch.empty(n, device="cuda").normal_(generator=g)
        m = torch.empty(n, device="cuda").normal_(generator=g)
        grad = torch.empty(n, device="cuda").normal_(generator=g)
        if not grad32:
            grad = grad.half()
        entries.append((w, m, grad, torch.zeros(n, device="cuda", dtype=torch.float16)))
        single.append((w.clone(), m.clone(), grad, torch.zeros(n, device="cuda", dtype=torch.float16)))
    flag = torch.zeros(1, device="cuda", dtype=torch.int32)
    mpt.mpt_master_update_multi(entries, 0.25, 0.1, 0.9, flag)
    for e in single:
        mpt.mpt_master_update(*e, 0.25, 0.1, 0.9, flag)
    for k, (a, b) in enumerate(zip(entries, single)):
        for x, y in zip(a, b):
            assert np.array_equal(x.cpu().numpy().view(np.uint8), y.cpu().numpy().view(np.uint8)), k
