"""Every tile shape of the grouped matrix-core kernel at the edges of its inner
loop: one to all column blocks of 16 in use (whole tiles, ragged last slices of
merged ones), rows past the slice, one, two and three chunks of inner indices
and fewer than a chunk, and operand elements that are not finite."""
import numpy as np
import pytest

from paper_2211_17028_amd import tn
from tests.test_gpu_parity import _random_mfma_job

pytestmark = pytest.mark.gpu


def _launch(torch, job, tiles, tile):
    d = tn.mfma_group_descriptors([job], tiles)
    tn.kernel_mfma_group(tile, d)
    if job.get("ksplit", 1) > 1:
        tn.kernel_mfma_split_reduce(tile, d)
    torch.cuda.synchronize()
    return job["C"].cpu().numpy()


# (m, n, k, slices, slices sharing an operand, merge, split); column counts as parts of a tile's width
SHAPES = [
    ("whole", lambda bm, bn: (bm, bn, 5, 2, 1, 0, 1)),
    ("two_by_two_tiles", lambda bm, bn: (bm + 1, bn + 1, 4, 1, 1, 0, 1)),
    ("one_chunk", lambda bm, bn: (bm, bn, 3, 3, 1, 0, 1)),
    ("three_chunks_of_parts", lambda bm, bn: (bm, bn, 6, 2, 1, 0, 4)),
    ("short_inner", lambda bm, bn: (bm - 1, bn, 1, 2, 1, 0, 1)),
    ("no_inner", lambda bm, bn: (bm, bn - 1, 0, 2, 1, 0, 1)),
    ("a_quarter_of_the_columns", lambda bm, bn: (bm, bn - 2, 6, 3, 1, 0, 1)),
    ("half_of_the_columns", lambda bm, bn: (bm, bn - 1, 6, 3, 1, 0, 1)),
    ("one_and_three_quarters", lambda bm, bn: (bm, bn - 2, 5, 10, 5, 1, 1)),
    ("three_quarters", lambda bm, bn: (bm, bn - 2, 5, 6, 3, 1, 1)),
    ("ragged_rows", lambda bm, bn: (bm - 2, bn, 5, 10, 5, 2, 1)),
    ("few_rows_split", lambda bm, bn: (3, bn - 1, 7, 3, 1, 0, 8)),
]


@pytest.mark.parametrize("tile", range(8))
@pytest.mark.parametrize("name,shape", SHAPES, ids=[s[0] for s in SHAPES])
def test_every_tile_shape(tile, name, shape):
    import torch
    bm, bn = (int(np.log2(v)) for v in tn.MFMA_TILE_SHAPES[tile])
    m_log, n_log, k_log, n_slices, share, merge, ksplit = shape(bm, bn)
    print("tile", tile, name, (m_log, n_log, k_log, n_slices, share, merge, ksplit), flush=True)
    rng = np.random.default_rng([tile, m_log, n_log, k_log, merge])
    job, tiles, ref = _random_mfma_job(torch, rng, m_log, n_log, k_log, n_slices, share, merge, tile, ksplit)
    got = _launch(torch, job, tiles, tile).reshape(ref.shape)
    # 2 k products of normal numbers (the largest of many about 16): an error of at most
    # 2^-24 x 16 for each of a few sums, growing like sqrt(2 k) sums of size sqrt(2 k)
    k = 1 << k_log
    assert np.abs(got - ref).max() <= 2.0 ** -24 * 16 * (k + 4)
    assert np.array_equal(got.view(np.float32), _launch(torch, job, tiles, tile).reshape(ref.shape).view(np.float32))


@pytest.mark.parametrize("tile", range(8))
@pytest.mark.parametrize("k_log,merge", [(1, 0), (2, 1), (2, 2), (4, 0)])
def test_values_that_are_not_finite_stay_in_their_rows_and_columns(tile, k_log, merge):
    """Padding lanes read elements of the tile's first row and column: not finite
    ones spoil the outputs they belong to and no others."""
    import torch
    bm, bn = (int(np.log2(v)) for v in tn.MFMA_TILE_SHAPES[tile])
    m_log, n_log = (bm - 2 if merge == 2 else bm - 1), (bn - 2 if merge == 1 else bn - 1)
    print("not finite", tile, k_log, merge, flush=True)
    rng = np.random.default_rng([tile, k_log, merge])
    job, tiles, ref = _random_mfma_job(torch, rng, m_log, n_log, k_log, 3, 3 if merge else 1, merge, tile, 1)
    # row 0 of A's first slice, column 0 of B's first slice, alternately NaN and infinite
    k = np.arange(1 << k_log)
    at = lambda pos: sum(((k >> j) & 1) << p for j, p in enumerate(pos))          # noqa: E731
    bad = torch.from_numpy(np.where(k % 2, np.nan, np.inf).astype(np.complex64)).cuda()
    job["A"][torch.from_numpy(at(job["a_k"])).cuda()] = bad
    job["B"][torch.from_numpy(at(job["b_k"])).cuda()] = bad
    got = _launch(torch, job, tiles, tile).reshape(ref.shape)
    clean = np.ones(ref.shape, bool)
    for s in range(3):
        if merge == 1 or s == 0:         # merge 1: all slices read A's first slice
            clean[s, 0, :] = False
        if merge == 2 or s == 0:
            clean[s, :, 0] = False
    assert not np.isfinite(got[~clean]).any()
    assert np.abs(got[clean] - ref[clean]).max() <= 2.0 ** -24 * 16 * ((1 << k_log) + 4)
