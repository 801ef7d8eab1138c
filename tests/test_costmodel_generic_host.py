"""The cost model's features of GENERIC saturated candidates describe the
kernels that are generated (no GPU needed): instructions after sharing, the LDS
element, rows per thread, planes loaded for their neighbours."""
import numpy as np

from paper_2306_13002_amd import stencil as S, synth


def feats(n, tile, shape, r, pattern, dtype):
    taps = synth.box_taps(r) if shape == "box" else synth.star_taps(r)
    cids, _ = synth.sharing_ids(taps, pattern, iter(synth.uniform_f64(9, 5, (4096,))))
    kw = dict(dtype=dtype, radius=r, taps=taps, cids=cids, coef=[1.0 / len(taps)] * (max(cids) + 1))
    return S.features("generic", n, ("saturated", tile, "xcd"), **kw)


def test_symmetric_box_counts_its_shared_sums():
    f = feats((256, 256, 256), (64, 16, 16), "box", 3, "symmetric", "f64")
    # 70 FMAs per point (groups per plane: 10 classes x 7) and fewer adds than
    # half the 273 of unshared sums, over 22 planes per 16 written
    assert 70 * 22 / 16 < f[19] < (70 + 273 / 2) * 22 / 16
    assert f[14] == np.float32((64 + 6) * (16 + 6) / (64 * 16) * 22 / 16)
    assert f[15] == 2 * 70 * 22 * 8


def test_distinct_box_counts_its_taps():
    f = feats((256, 256, 256), (64, 16, 16), "box", 2, "distinct", "f32")
    assert f[19] == 125  # slots that are not live are skipped


def test_stars_in_f32_hold_f32_in_lds():
    f = feats((256, 256, 256), (32, 16, 16), "star", 4, "reflection", "f32")
    assert f[15] == 2 * 40 * 24 * 4


def test_rows_per_thread_follow_the_grid():
    many = feats((256, 256, 256), (64, 4, 8), "box", 2, "distinct", "f64")  # two rows per thread: more accumulators
    few = feats((64, 20, 16), (64, 4, 8), "box", 2, "distinct", "f64")      # one
    assert many[16] > few[16]


def test_tiles_that_are_not_offered_still_have_features():
    assert np.all(np.isfinite(feats((64, 64, 64), (16, 16, 8), "star", 1, "distinct", "f64")))
