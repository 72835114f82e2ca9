"""The append launch at the edges of its tiles and of its rotary bands, against
the fp64 oracle: partial pages and partial groups of 16 rows, bands that are
empty or end inside a thread's four pairs, several tiles per block, and empty
slots with eps = 0 (which must stay zero, not 0 * inf)."""
import numpy as np
import pytest

import oracle
from helpers import bf16_f64, dev_f32, dev_i32, from_dev, to_dev
from paper_2607_04443_amd import synth

pytestmark = pytest.mark.gpu


def _close(got, ref):
    # one bf16 ulp plus the fp32 error of a rotated pair that cancels to near zero
    ulp = np.exp2(np.floor(np.log2(np.maximum(np.abs(ref), 2.0 ** -126))) - 7)
    err = np.abs(got - ref)
    assert (err <= ulp + 2.0 ** -15).all(), float(err.max())


@pytest.mark.parametrize("pairs", [(22, 21, 21), (64, 0, 0), (0, 1, 63), (5, 59, 0)])
@pytest.mark.parametrize("heads,n", [(1, 1), (3, 15), (3, 65), (70, 16 * 64 + 17)])
def test_rows_bands_and_empty_slots(ws, pairs, heads, n):
    import torch
    rng = np.random.default_rng(synth.SEED_BASE + 17 * n + heads)
    k, v, q = (synth.normal_bf16(rng, (n, heads, 128)) for _ in range(3))
    pos = rng.integers(0, 200, size=(n, 3)).astype(np.int32)
    gamma = rng.uniform(0.5, 1.5, 128).astype(np.float32)
    cache = ws.Cache(heads, n // 64 + 4, max_q_tokens=max(64, n), rope_pairs=pairs)
    try:
        kd, vd, qd, pd, gd = to_dev(k), to_dev(v), to_dev(q), dev_i32(pos), dev_f32(gamma)
        q_out = torch.full_like(qd, float("nan"))
        cache.step_append([dict(unit=0, kind=ws.WS_KIND_VIDEO, k=kd, v=vd, mode=ws.WS_APPEND_NORM_ROPE,
                                positions=pd, gamma=gd, eps=0.0)],
                          [dict(q=qd, q_out=q_out, positions=pd, gamma=gd, eps=0.0, scale=1.0)])
        k_got, v_got = cache.export(0, ws.WS_KIND_VIDEO)
        np.testing.assert_array_equal(v_got, v)
        k_got, q_got = bf16_f64(k_got), bf16_f64(from_dev(q_out))
        for h in {0, heads // 2, heads - 1}:
            g = gamma.astype(np.float64)
            _close(k_got[:, h], oracle.query_prologue(k[:, h], oracle.MODE_NORM_ROPE, pos, g, 0.0, pairs))
            _close(q_got[:, h], np.log2(np.e) * oracle.query_prologue(q[:, h], oracle.MODE_NORM_ROPE, pos, g, 0.0,
                                                                      pairs))
        # a NaN in an empty slot or in a tile's largest norm would reach the outputs
        out = torch.full_like(qd, float("nan"))
        cache.unit_attention(q_out, out, ws.mask_spec(0, -(2 ** 31), (ws.WS_KIND_VIDEO,)), ws.WS_QUERY_PREPARED)
        assert torch.isfinite(out).all()
        assert cache.check() == 0
    finally:
        cache.close()
