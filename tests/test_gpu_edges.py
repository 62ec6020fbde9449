"""Kernels at the sizes where their split of the work changes: edges of
chunks and batches, remainders, the smallest and the largest."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import numpy as np

from gpu_util import dev_bytes, host_words
from oracle import splitmix
from paper_2608_15764_amd import ilpsweep as isw

SEED = 0x1D5EED00 + 33
FILL_CHUNK = 4 << 10            # bytes one wave of the fill writes


@pytest.mark.parametrize("nbytes", [8, FILL_CHUNK - 16, FILL_CHUNK - 4, FILL_CHUNK,
                                    FILL_CHUNK + 4, FILL_CHUNK + 16, 7 * FILL_CHUNK - 12,
                                    4099 * FILL_CHUNK + 4092 * 4])
def test_fill_at_chunk_edges(nbytes):
    print("fill", nbytes, flush=True)
    buf = dev_bytes((nbytes + 15) // 16 * 16 + 4096).zero_()
    isw.sweep_fill_u32(buf, nbytes, SEED)
    torch.cuda.synchronize()
    assert np.array_equal(host_words(buf)[:nbytes // 4], splitmix.words(SEED, 0, nbytes // 4))
    assert not buf[nbytes:].any()
