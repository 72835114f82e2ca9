"""Audio calls of few pages, whose one key range per head goes to the output
without a merge: against the fp64 oracle on both sides of the page count where
that ends, and against the same call cut into ranges; rows of several query
tiles, strided outputs, no visible key."""
import numpy as np
import pytest

import oracle
from helpers import Loaded, assert_gates, bf16_f64, from_dev, to_dev
from paper_2607_04443_amd import synth
from test_gpu_video_edges import COND, _workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_q", [1, 4, 17, 64])
@pytest.mark.parametrize("n_keys", [1, 65, 64 * 4, 64 * 8 + 1, 64 * 12, 64 * 12 + 1, 64 * 17])
def test_one_range_against_the_oracle_and_a_merge(ws, n_q, n_keys):
    import torch
    rng = np.random.default_rng(700 + 64 * n_q + n_keys)
    H = 3
    q, k, v = (synth.normal_bf16(rng, (n, H, 128)) for n in (n_q, n_keys, n_keys))
    L = Loaded(ws, _workload(H, k, v), max_pages=n_keys // 64 + 8, max_q_tokens=64)
    try:
        pos = np.zeros((n_q, 3), np.int32)
        ref = L.oracle(q, pos, 0, COND, mode=oracle.MODE_RAW)
        got = {}
        for splits in (0, 1, 2):  # the library's choice, one range, two with a merge
            L.cache.set_option(ws.WS_OPT_AUDIO_KV_SPLITS, splits)
            got[splits] = L.run("audio", q, pos, 0, COND, mode=ws.WS_APPEND_RAW)
            assert_gates(got[splits], ref, label=f"{n_q} rows, {n_keys} keys, {splits} ranges")
        # a strided output, with guard values around every row
        L.cache.set_option(ws.WS_OPT_AUDIO_KV_SPLITS, 1)
        wide = torch.full((n_q, H + 2, 128), 7.0, dtype=torch.bfloat16, device="cuda")
        out = wide[:, 1:H + 1]
        L.cache.audio_attention(to_dev(q), out, ws.mask_spec(0, -(2 ** 31), COND), ws.WS_APPEND_RAW)
        np.testing.assert_array_equal(bf16_f64(from_dev(out.contiguous())), got[1])
        assert (wide[:, 0] == 7.0).all() and (wide[:, -1] == 7.0).all()
        # nothing visible: zeros
        L.cache.audio_attention(to_dev(q), out, ws.mask_spec(0, 0, (ws.WS_KIND_AUDIO,)), ws.WS_APPEND_RAW)
        assert (out == 0).all()
    finally:
        L.close()


@pytest.mark.parametrize("n_keys", [50, 64 * 8, 64 * 12])
def test_a_nan_row_is_the_same_with_one_range_and_with_a_merge(ws, n_keys):
    """A query row of NaN gives a row of zeros however its keys are cut, and
    leaves the other rows alone."""
    rng = np.random.default_rng(760 + n_keys)
    H = 3
    q, k, v = (synth.normal_bf16(rng, (n, H, 128)) for n in (5, n_keys, n_keys))
    q[2] = 0x7fc0
    L = Loaded(ws, _workload(H, k, v), max_pages=n_keys // 64 + 8, max_q_tokens=64)
    try:
        pos = np.zeros((5, 3), np.int32)
        rest = [0, 1, 3, 4]
        ref = L.oracle(q[rest], pos[rest], 0, COND, mode=oracle.MODE_RAW)
        for splits in (0, 1, 2):
            L.cache.set_option(ws.WS_OPT_AUDIO_KV_SPLITS, splits)
            got = L.run("audio", q, pos, 0, COND, mode=ws.WS_APPEND_RAW)
            assert (got[2] == 0).all(), (splits, got[2])
            assert_gates(got[rest], ref, label=f"{n_keys} keys, {splits} ranges")
    finally:
        L.close()
