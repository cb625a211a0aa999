"""The branches of the launch rules that the parity cases' own shapes do not reach, at their edges."""
import numpy as np
import pytest

from paper_2408_10746_amd import inputs
from paper_2408_10746_amd.inputs import Workload

pytestmark = pytest.mark.gpu

from tests.test_gpu_parity import TOL, check_against_oracle, make_session  # noqa: E402


# 256 x 256 tiles (many layers: the smaller tiles would need a second round of the compute units), gradients that are no
# contractions as whole rows.  Tails: p1 88 of 256 token rows and a last 64-token step of few valid tokens, d = 3.5 tiles;
# p2 adapter rows of one and a quarter tiles, d = 3.25 tiles.
@pytest.mark.parametrize("w", [
    Workload("p1", L=20, d=896, n_max=230, B=3, r=256, C=4, N=3, cache_dtype="bf16", len_lo=170),
    Workload("p2", L=16, d=832, n_max=301, B=2, r=320, C=5, N=2, cache_dtype="bf16", len_lo=299),
], ids=lambda w: w.name)
def test_wide_contractions_on_large_tiles(w):
    lens, ids = inputs.lengths(w), np.arange(w.B)
    acts, labels = inputs.batch_acts(w, ids), inputs.labels(w)[ids]
    sess = make_session(w, lens=lens)
    sess.cache_fill(ids, acts, lens)
    check_against_oracle(w, sess, ids, acts, lens, labels, inputs.random_params(w, up_scale=0.3), TOL["bf16"], what=w.name)


# fp32: 16-row tiles with 8, 6 (the second column chunk part empty), 4 and 6 column blocks per workgroup; K of 2 .. 10
# units over eight wavefronts, a last row tile of a few rows
@pytest.mark.parametrize("w", [
    Workload("f1", L=2, d=96, n_max=130, B=32, r=128, C=3, N=32, cache_dtype="f32", len_lo=128),
    Workload("f2", L=2, d=160, n_max=68, B=32, r=160, C=2, N=32, cache_dtype="f32", len_lo=62),
    Workload("f3", L=3, d=64, n_max=68, B=32, r=128, C=2, N=32, cache_dtype="f32", len_lo=62),
    Workload("f4", L=2, d=32, n_max=130, B=32, r=96, C=5, N=32, cache_dtype="f32", len_lo=128),
    Workload("f5", L=2, d=288, n_max=9, B=3, r=64, C=2, N=3, cache_dtype="f32", len_lo=1),
], ids=lambda w: w.name)
def test_fp32_contractions(w):
    lens, ids = inputs.lengths(w), np.arange(w.B)
    acts, labels = inputs.batch_acts(w, ids), inputs.labels(w)[ids]
    sess = make_session(w, lens=lens)
    sess.cache_fill(ids, acts, lens)
    check_against_oracle(w, sess, ids, acts, lens, labels, inputs.random_params(w, up_scale=0.3), TOL["f32"], what=w.name)
