"""The video kernel with waves of 64, 48 and 32 rows, against the fp64 oracle:
row counts whose tiles hold 256, 192 and 128 rows at this head count (and the
remainders in their last tiles), over partial pages, single keys, streams
longer than the 128-unit entry window, attained logit bounds, and logits far
below their bound."""
import numpy as np
import pytest

from paper_2607_04443_amd import synth
import test_gpu_video_edges as edges

pytestmark = pytest.mark.gpu
# three heads: 380 rows take tiles of 256 rows, 250 and 500 of 192, 300 of 128
ROWS = [380, 250, 500, 300]


def _bits(seed, n_q, n_keys, H=3):
    rng = np.random.default_rng(seed)
    return tuple(synth.normal_bf16(rng, (n, H, 128)) for n in (n_q, n_keys, n_keys))


@pytest.mark.parametrize("n_q", ROWS)
@pytest.mark.parametrize("n_keys", [1, 33, 63, 64, 65, 64 * 4, 64 * 5 + 7])
def test_key_counts(ws, n_q, n_keys):
    edges._check(ws, *_bits(n_q + n_keys, n_q, n_keys), label=f"{n_q} rows, {n_keys} keys")


@pytest.mark.parametrize("n_q", [250, 500])
def test_long_streams(ws, n_q):
    # 64 heads x 20 pages over two or three tiles: shares of several heads, streams past 128 units
    edges._check(ws, *_bits(n_q, n_q, 64 * 20 - 9, H=64), label=f"{n_q} rows, shares across heads")
    edges._check(ws, *_bits(n_q, n_q, 64 * 1000 - 23, H=1), label=f"{n_q} rows, a long stream")


@pytest.mark.parametrize("n_q", [250, 380])
@pytest.mark.parametrize("stretch", [3.0, 9.0])
def test_lowered_shift(ws, n_q, stretch):
    edges.test_shift_below_an_attained_bound(ws, n_q, stretch)


@pytest.mark.parametrize("n_keys", [1, 64 * 3 + 24])
@pytest.mark.parametrize("n_q", ROWS)
def test_running_maximum(ws, n_q, n_keys):
    edges.test_rows_out_of_the_shift_s_reach(ws, n_q, n_keys, n_q == 250)
