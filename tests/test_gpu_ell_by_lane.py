"""Rank 4 with many samples (from 16,384 on): a lane per column part.  Columns of every length around the parts'
and blocks' bounds as in the other form's test, ranks 4 and 3 (padded), both workgroup sizes, sample counts at both
sides of the rule."""
import pytest

pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import test_gpu_ell_edges as edges  # noqa: E402


@pytest.mark.parametrize("m,n,q,threads", [(260, 1041, 4, 1024), (260, 1041, 3, 512), (140, 316, 4, 1024),
                                           (140, 306, 4, 1024), (200, 330, 4, 512)])
def test_parts_blocks(m, n, q, threads):
    edges.test_parts_items_steps(m, n, q, threads)
