"""Queries normed in the video kernel.  Rows of a query tile past the end of
their call (or of their query group) leave the rows before them alone: a
ragged call with eps = 0 (a row of zeros then has an infinite reciprocal
norm) gives bit for bit what a call with the tile filled gives.  And the mean
square is an fp32 one: rows of 2^-64 (squares below fp32's normal range) are
normed like any other."""
import numpy as np
import pytest

from helpers import assert_gates, bf16_f64, dev_f32, dev_i32, from_dev, to_dev
from paper_2607_04443_amd import synth

pytestmark = pytest.mark.gpu
H, KEYS = 2, 64 * 5 + 9
ANY = -(2 ** 31)


@pytest.fixture(scope="module")
def setup(ws):
    rng = np.random.default_rng(synth.SEED_BASE + 801)
    cache = ws.Cache(H, KEYS // 64 + 4, max_q_tokens=1024)
    k, v = (to_dev(synth.normal_bf16(rng, (KEYS, H, 128))) for _ in range(2))
    cache.append(0, ws.WS_KIND_COND, k, v)
    q = to_dev(synth.normal_bf16(rng, (256, H, 128)))
    pos = dev_i32(rng.integers(0, 200, size=(256, 3)))
    gamma = dev_f32(rng.uniform(0.5, 1.5, 128))
    yield cache, q, pos, gamma, ws.mask_spec(0, ANY, (ws.WS_KIND_COND,))
    cache.close()


def _unit(ws, s, n, splits):
    import torch
    cache, q, pos, gamma, mask = s
    cache.set_option(ws.WS_OPT_VIDEO_KV_SPLITS, splits)
    out = torch.full((n, H, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    cache.unit_attention(q[:n], out, mask, ws.WS_APPEND_NORM_ROPE, pos[:n], gamma, 0.0)
    return from_dev(out)


@pytest.mark.parametrize("splits", [1, 2])  # (forced ranges: tiles of 256 rows, shares that ignore the row count)
@pytest.mark.parametrize("n_q", [1, 24, 100, 131, 200, 250])
def test_ragged_call_equals_the_filled_tile(ws, setup, n_q, splits):
    full = _unit(ws, setup, 128 if n_q <= 128 else 256, splits)  # waves of 32 and of 64 rows
    np.testing.assert_array_equal(_unit(ws, setup, n_q, splits), full[:n_q])


def test_ragged_groups_equal_the_filled_tiles(ws, setup):
    import torch
    cache, q, pos, gamma, mask = setup
    cache.set_option(ws.WS_OPT_VIDEO_KV_SPLITS, 1)
    out = torch.full((231, H, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    rows = list(range(200)) + list(range(31))
    cache.unit_attention_groups(q[rows], out, [(200, mask), (31, mask)], ws.WS_APPEND_NORM_ROPE, pos[rows], gamma, 0.0)
    got = from_dev(out)
    np.testing.assert_array_equal(got[:200], _unit(ws, setup, 256, 1)[:200])
    np.testing.assert_array_equal(got[200:], _unit(ws, setup, 128, 1)[:31])


@pytest.mark.parametrize("e", [64, 66, 68, 70])
def test_tiny_rows_are_normed(ws, setup, e):
    import torch
    cache, q, pos, gamma, mask = setup
    cache.set_option(ws.WS_OPT_VIDEO_KV_SPLITS, 1)
    out = torch.full_like(q, float("nan"))
    cache.unit_attention(q * 2.0 ** -e, out, mask, ws.WS_APPEND_NORM_ROPE, pos, gamma, 0.0)
    # scaling every row by a power of two leaves its RMS norm as it was, up to
    # the bits that squares near 2^-2e lose (at least 9 of 24 remain, of 128 squares)
    assert_gates(bf16_f64(from_dev(out)), bf16_f64(_unit(ws, setup, 256, 1)), label=f"rows of 2^-{e}")
