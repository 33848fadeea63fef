"""Gradient on the beamlet rows for more rows than a launch of wide workgroups can count threads for."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [(2 ** 32 - 1) // 512, (2 ** 32 - 1) // 512 + 1, 9_000_000])
def test_every_row_is_summed(rows):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_4417_amd import CSR
    at = np.array([0, 1, 611_328, rows // 2, rows - 2, rows - 1])          # the rows with entries, one each
    ip = torch.zeros(rows + 1, dtype=torch.int64)
    ip[torch.from_numpy(at + 1)] = 1
    ip = torch.cumsum(ip, 0).cuda()
    idx = torch.arange(len(at), dtype=torch.int32, device="cuda")
    val = torch.arange(1, len(at) + 1, dtype=torch.float32, device="cuda")
    r = torch.full((len(at),), 0.5, device="cuda")
    want = np.zeros(rows, np.float32)
    want[at] = 0.5 * np.arange(1, len(at) + 1)
    got = CSR(ip, idx, val, len(at)).gradient(r)
    np.testing.assert_array_equal(got.cpu().numpy(), want)
