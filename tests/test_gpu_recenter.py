"""Bit centering at the edges of its norm's chunks: groups of 32 addends, chunks of 2048, and the sizes where the
workgroup gets wider; the same bits as the oracle's one addition after the other."""
import pytest

import test_gpu_parity as parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,K,d,R", [(8, 1, 1, 3), (16, 1, 31, 1), (8, 1, 32, 1), (8, 1, 33, 1), (16, 1, 1024, 1),
                                     (8, 1, 1025, 1), (16, 1, 2047, 1), (8, 1, 2048, 2), (8, 1, 2049, 1),
                                     (16, 3, 1365, 1), (8, 1, 4097, 1), (8, 10, 10000, 2)])
def test_recenter_at_the_edges_of_the_chunks(b, K, d, R):
    parity.test_recenter_bit_exact(b, K, d, R)
