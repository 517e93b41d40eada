"""Labels in the caller's format: soft rows leave a workgroup of k_labels as one run of words, 256, 128, 64, 32 or 16 rows of it by
the number of columns; up to 1 MB of them go straight to pinned memory.  Rows at the ends of workgroups, odd column counts."""
import numpy as np
import pytest
import torch

import paper_2604_06596_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C", [2, 3, 4, 5, 8, 9, 16, 17, 31, 33, 50, 64])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 255, 256, 257, 4099, 12000])
def test_every_row_and_column_reaches_its_place(n, C):
    rng = np.random.default_rng(n * 100 + C)
    sv = rng.permutation(n)[: (n + 1) // 2].astype(np.int32)
    sc = rng.integers(0, C, sv.size).astype(np.int32)
    want = np.full((n, C), np.float32(1.0) / np.float32(C), np.float32)
    want[sv] = 0
    want[sv, sc] = 1
    arrays = [np.zeros(n + 1, np.int64), np.zeros(0, np.int32), np.zeros(0, np.float32), sv, sc]
    for device in (False, True):
        a = [torch.as_tensor(x).cuda() if device else x for x in arrays]
        with P.DynLP(n, a[0], a[1], a[2], C, a[3], a[4], device_ptrs=device) as d:
            for soft, hard in ((True, True), (True, False), (False, True)):
                so, ho = (x.cpu().numpy() if torch.is_tensor(x) else x for x in d.get_labels(soft=soft, hard=hard))
                assert (so is None) == (not soft) and (ho is None) == (not hard)
                if soft:
                    assert np.array_equal(so, want)
                if hard:  # equal columns: the lowest class
                    assert np.array_equal(ho, np.argmax(want, 1))
