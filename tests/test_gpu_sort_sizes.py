"""The sort at the sizes where its scan changes form: one tile of 4096 keys and
one key more, the last size whose digit counts one workgroup scans and one key
more.  Whole numbers: exact."""
import pytest
import torch

import paper_2012_13173_amd as hcg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 4096, 4097, 50_000, 1 << 19, (1 << 19) + 1])
@pytest.mark.parametrize("bits", [3, 19, 32])
def test_sort_at_the_edges_of_its_scan(n, bits):
    g = torch.Generator().manual_seed(n + bits)
    keys = torch.randint(0, 1 << bits, (n,), generator=g, dtype=torch.int64)
    print(f"sort n={n} bits={bits}", flush=True)
    bits32 = torch.where(keys < 1 << 31, keys, keys - (1 << 32)).to(torch.int32)  # as uint32
    out, perm = hcg.hcg_sort_keys(bits32.cuda(), bits)
    torch.cuda.synchronize()
    want, order = torch.sort(keys, stable=True)
    assert torch.equal(out.cpu().to(torch.int64) & 0xFFFFFFFF, want)
    assert torch.equal(perm.cpu().to(torch.int64), order)
