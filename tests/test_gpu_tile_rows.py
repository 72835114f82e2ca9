"""The video kernel in query tiles of 256, 192 and 128 rows (waves of 64, 48 and
32), against the fp64 oracle: whole tiles and the remainders in their last ones,
over partial pages, single keys, streams longer than the 128-unit entry
window, and logits far below their bound.  Each case states its tile."""
import numpy as np
import pytest

from paper_2607_04443_amd import synth
import test_gpu_video_edges as edges

pytestmark = pytest.mark.gpu
# three heads, one to six pages: rows per query tile
TILE = {380: 256, 250: 192, 500: 192, 300: 128}
ROWS = list(TILE)


def _bits(seed, n_q, n_keys, H=3):
    rng = np.random.default_rng(seed)
    return tuple(synth.normal_bf16(rng, (n, H, 128)) for n in (n_q, n_keys, n_keys))


@pytest.mark.parametrize("n_q", ROWS)
@pytest.mark.parametrize("n_keys", [1, 33, 63, 64, 65, 64 * 4, 64 * 5 + 7])
def test_key_counts(ws, n_q, n_keys):
    edges._check(ws, *_bits(n_q + n_keys, n_q, n_keys), label=f"{n_q} rows, {n_keys} keys", tile=TILE[n_q])


# shares of several heads (64 groups of 20 and 10 units), then streams of 143
# units (one of 1900 rows: every 31st row compared, for the oracle's time)
@pytest.mark.parametrize("H,n_q,pages,tile,every", [(64, 250, 20, 128, 1), (64, 500, 20, 192, 1), (64, 500, 10, 192, 1),
                                                    (1, 250, 1000, 128, 1), (1, 500, 1000, 128, 1),
                                                    (3, 1900, 1000, 192, 31)])
def test_long_streams(ws, H, n_q, pages, tile, every):
    edges._check(ws, *_bits(n_q, n_q, 64 * pages - 9, H=H), label=f"{H} heads, {n_q} rows, {pages} pages", tile=tile,
                 every=every)


@pytest.mark.parametrize("n_q", [250, 300, 380])
@pytest.mark.parametrize("stretch", [3.0, 9.0])
def test_attained_bounds(ws, n_q, stretch):
    edges.test_shift_below_an_attained_bound(ws, n_q, 0, TILE[n_q], stretch, False)


@pytest.mark.parametrize("n_keys", [1, 64 * 3 + 24])
@pytest.mark.parametrize("n_q", ROWS)
def test_running_maximum(ws, n_q, n_keys):
    # (two heads take the same tiles)
    edges.test_rows_out_of_the_shift_s_reach(ws, n_q, 0, TILE[n_q], n_keys, n_q == 250)
