"""Rank 8 with many samples (a bucket's mean from 28,672 samples and 512 rows on): a lane per column part.  Columns of
every length around the parts' and blocks' bounds as in the other form's test, ranks 8 and 5 (padded), both workgroup
sizes, samples and rows at both sides of the rule."""
import pytest

pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import test_gpu_ell_edges as edges  # noqa: E402


@pytest.mark.parametrize("m,n,q,threads", [(600, 1041, 8, 1024), (600, 1041, 5, 512), (512, 362, 8, 1024),
                                           (511, 362, 8, 1024), (512, 350, 8, 512), (520, 362, 6, 512)])
def test_parts_blocks(m, n, q, threads):
    edges.test_parts_items_steps(m, n, q, threads)
