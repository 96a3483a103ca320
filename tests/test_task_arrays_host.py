"""Task arrays hold the same tags whether they are filled field by field (up to 16 tasks) or
column by column: the low 32 bits of any integer, as a C field takes them."""
import numpy as np
import pytest

import paper_2005_10445_amd as acq
from paper_2005_10445_amd import _capi


@pytest.mark.parametrize("n", [1, 16, 17, 40])
@pytest.mark.parametrize("tag", [5, -1, 2 ** 31 - 1, 2 ** 32 + 3, -2 ** 40 + 9, 2 ** 63 - 1, 2 ** 63, 2 ** 80 + 7, -2 ** 70 + 1])
def test_tags_of_any_size(n, tag):
    tasks = [(10 + i, i) for i in range(n - 1)] + [(99, tag)]
    arr = acq._task_array(_capi.AcqTrackTask, np.dtype(_capi.AcqTrackTask), "block", tasks,
                          lambda blocks: [(1000 + b, 2 * b) for b in blocks])
    assert len(arr) == n
    for i in range(n - 1):
        assert (arr[i].block, arr[i].n, arr[i].tag) == (1010 + i, 20 + 2 * i, i)
    want = (tag + 2 ** 31) % 2 ** 32 - 2 ** 31
    assert (arr[n - 1].block, arr[n - 1].n, arr[n - 1].tag) == (1099, 198, want)
