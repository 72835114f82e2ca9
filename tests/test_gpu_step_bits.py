"""A step gives the bits of the separate calls, and the same bits whichever
workspace its partials go to: short audio windows (one key range per head)
beside a video call with and without a merge, and steps near the static
workspace's limit."""
import numpy as np
import pytest

from helpers import from_dev, to_dev
from paper_2607_04443_amd import synth
from test_gpu_riders import ALL, VIDEO, Step
from test_gpu_video_edges import COND

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pages", [7, 8, 12, 13])
@pytest.mark.parametrize("splits", [1, 2])  # video ranges per head: without and with a merge
@pytest.mark.parametrize("prepared", [True, False])
def test_audio_rows_that_do_not_ride_equal_the_audio_call(ws, pages, splits, prepared):
    import torch
    rng = np.random.default_rng(820 + pages)
    H, n_keys = 3, 64 * pages - 5
    qv, qa, k, v = (to_dev(synth.normal_bf16(rng, (n, H, 128))) for n in (200, 5, n_keys, n_keys))
    cache = ws.Cache(H, pages + 4, max_q_tokens=256)
    try:
        cache.append(0, ws.WS_KIND_COND, k, v)
        cache.set_option(ws.WS_OPT_VIDEO_KV_SPLITS, splits)
        cache.set_option(ws.WS_OPT_STEP_SEPARATE_AUDIO, 1)
        mask = ws.mask_spec(0, -(2 ** 31), COND)
        mode = ws.WS_QUERY_PREPARED if prepared else ws.WS_APPEND_RAW
        if prepared:
            qv, qa = qv * 0.125, qa * 0.125
        sv, sa, v1, a1, v2, a2 = (torch.full_like(x, float("nan")) for x in (qv, qa) * 3)
        cache.unit_attention(qv, sv, mask, mode)
        cache.audio_attention(qa, sa, mask, mode)
        cache.step_attention(dict(q=qv, out=v1, mask=mask, mode=mode), dict(q=qa, out=a1, mask=mask, mode=mode))
        cache.step_attention_noalloc(dict(q=qv, out=v2, mask=mask, mode=mode), dict(q=qa, out=a2, mask=mask, mode=mode))
        for got, want in ((v1, sv), (a1, sa), (v2, sv), (a2, sa)):
            np.testing.assert_array_equal(from_dev(got), from_dev(want))
    finally:
        cache.close()


@pytest.mark.parametrize("n_v", [1040, 1060, 1064])
def test_riders_do_not_depend_on_the_workspace(ws, n_v):
    """Three forced video ranges of 40 heads: the static workspace has room for
    fewer ranges of the audio rows than the cache's (at 1064 rows: for one of
    their own pages beside the three shared ones)."""
    import torch
    S = Step(ws, 40, (20, 54), 64, 4, 3, 83)
    try:
        S.cache.set_option(ws.WS_OPT_VIDEO_KV_SPLITS, 3)
        u = S.unit
        qv, qa = to_dev(S.queries(n_v)), to_dev(S.queries(4))
        outs = []
        for fn in (S.cache.step_attention, S.cache.step_attention_noalloc):
            ov, oa = torch.full_like(qv, float("nan")), torch.full_like(qa, float("nan"))
            S.cache.timing_enable(4)
            fn(dict(q=qv, out=ov, mask=ws.mask_spec(u, u - 3, VIDEO), mode=ws.WS_QUERY_PREPARED),
               dict(q=qa, out=oa, mask=ws.mask_spec(u, u - 3, ALL), mode=ws.WS_QUERY_PREPARED))
            torch.cuda.synchronize()
            rec = S.cache.timing_read()
            assert [r["path"] for r in rec] == ["video", "audio_riders"], rec
            outs.append((from_dev(ov), from_dev(oa)))
        for a, b in zip(*outs):
            np.testing.assert_array_equal(a, b)
    finally:
        S.close()
