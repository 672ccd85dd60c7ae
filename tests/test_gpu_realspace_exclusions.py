"""The check of exclusion lists is remembered for the tensors it was made on, not
for whatever later lies at their addresses."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_new_lists_at_old_addresses_are_checked():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2009_12617_amd as P
    n, box = 3000, np.diag([36.0] * 3)
    rng = np.random.default_rng(4)
    pos = torch.from_numpy(rng.random((n, 3)) * 36.0).to("cuda")
    q = torch.from_numpy(rng.uniform(-1.0, 1.0, size=n)).to("cuda")
    idx = (np.arange(n).reshape(-1, 2)[:, ::-1]).astype(np.int32).reshape(-1)  # partners in pairs
    real = P.RealSpace(n)

    def lists(end):
        off = np.minimum(np.arange(n + 1), end).astype(np.int32)  # (in range for any end <= n)
        return torch.from_numpy(off).to("cuda"), torch.from_numpy(idx).to("cuda")

    real(pos, q, box, 0.36, 8.0, exclusions=lists(n))  # (freed on return)
    torch.cuda.synchronize()
    bad = lists(n - 2)  # offsets that do not end at the number of partners
    with pytest.raises(ValueError):
        real(pos, q, box, 0.36, 8.0, exclusions=bad)
    real(pos, q, box, 0.36, 8.0, exclusions=lists(n))
