"""Query rows whose logits reach past what a shift fixed in advance serves
(their running maximum is raised as the pages come): each row's result is its
own, whatever rows share its wave, riders among them; values keep the range
of fp32; and the rounding of the softmax weights is that of weights taken
under a row's running maximum, not under a bound."""
import numpy as np
import pytest

import oracle
from helpers import Loaded, bf16_f64
from paper_2607_04443_amd import synth
from test_gpu_riders import ALL, VIDEO, Step
from test_gpu_video_edges import COND, _workload

pytestmark = pytest.mark.gpu


def _bits(x):
    return synth.bf16_bits(np.asarray(x, np.float32))


def _run(ws, q, k, v, splits=1, running=0):
    """RAW video queries over RAW keys; bf16 bits as float64."""
    L = Loaded(ws, _workload(q.shape[1], k, v), max_pages=k.shape[0] // 64 + 8, max_q_tokens=max(64, len(q)))
    try:
        L.cache.set_option(ws.WS_OPT_VIDEO_KV_SPLITS, splits)
        L.cache.set_option(ws.WS_OPT_VIDEO_RUNNING_MAX, running)
        return L.run("video", q, np.zeros((len(q), 3), np.int32), 0, COND, mode=ws.WS_APPEND_RAW)
    finally:
        L.close()


@pytest.mark.parametrize("n_v,n_a", [(124, 8), (120, 4), (200, 16), (300, 4)])
@pytest.mark.parametrize("stretch_v,stretch_a", [(1.0, 10.0), (10.0, 1.0), (3.0, 30.0)])
@pytest.mark.parametrize("splits", [0, 2])
def test_video_rows_do_not_depend_on_riders(ws, n_v, n_a, stretch_v, stretch_a, splits):
    """Prepared rows of std 0.15 have logit bounds of about 20 in log2 units;
    stretched by 3 and 10 they pass 40 and 180."""
    S = Step(ws, 3, (5, 60), 100, 4, 4, 81)
    try:
        S.cache.set_option(ws.WS_OPT_VIDEO_KV_SPLITS, splits)
        u = S.unit
        vmask, amask = (u, u - 3, VIDEO), (u, u - 3, ALL)
        qv = _bits(stretch_v * synth.bf16_to_f32(S.queries(n_v)))
        qa = _bits(stretch_a * synth.bf16_to_f32(S.queries(n_a)))
        fv, fa, rec = S.step(qv, qa, vmask, amask)
        print(rec)
        np.testing.assert_array_equal(fv, S.separate_video(qv, vmask))
        for got, q, mask in ((fv, qv, vmask), (fa, qa, amask)):
            ratio = np.abs(bf16_f64(got) - S.oracle(q, mask)) / S.bound(q, mask)
            assert ratio.max() <= 1.0, ratio.max()
    finally:
        S.close()


@pytest.mark.parametrize("n_q", [60, 200])
@pytest.mark.parametrize("stretch", [3.0, 6.0, 20.0])
def test_rows_are_independent(ws, n_q, stretch):
    """Sharp and ordinary rows mixed in every subtile against calls of one kind each."""
    rng = np.random.default_rng(900 + n_q)
    n_keys = 64 * 9 + 40
    q, k, v = (synth.normal_bf16(rng, (n, 2, 128)) for n in (n_q, n_keys, n_keys))
    sharp = np.zeros(n_q, bool)
    sharp[rng.permutation(n_q)[:n_q // 3]] = True
    q_sharp = _bits(stretch * synth.bf16_to_f32(q))
    mixed = np.where(sharp[:, None, None], q_sharp, q)
    got, mild, all_sharp = (_run(ws, x, k, v) for x in (mixed, q, q_sharp))
    np.testing.assert_array_equal(got[~sharp], mild[~sharp])
    np.testing.assert_array_equal(got[sharp], all_sharp[sharp])


@pytest.mark.parametrize("n_q", [60, 200])
@pytest.mark.parametrize("attained,exponent", [(True, 112), (False, 112), (False, -80)])
def test_values_keep_their_range(ws, n_q, attained, exponent):
    """Values scaled by a power of two give the output scaled by it, bit for
    bit: softmax weights stay within 2^8 and the row's largest is not small."""
    rng = np.random.default_rng(950 + n_q)
    n_keys = 64 * 9 + 40
    q, k, v = (synth.normal_bf16(rng, (n, 2, 128)) for n in (n_q, n_keys, n_keys))
    if attained:  # every row's dominant key is five times its own direction
        for i in range(n_q):
            k[(i * 29 + 300) % n_keys] = _bits(5.0 * synth.bf16_to_f32(q[i]))
    else:
        q = _bits(4.0 * synth.bf16_to_f32(q))
    one = _run(ws, q, k, v)
    scaled = _run(ws, q, k, _bits(np.ldexp(synth.bf16_to_f32(v), exponent)))
    assert np.isfinite(scaled).all()
    np.testing.assert_array_equal(np.ldexp(scaled, -exponent), one)


@pytest.mark.parametrize("stretch", [3.0, 4.0, 7.0])
@pytest.mark.parametrize("n_q,pages", [(120, 20), (240, 80)])
def test_weights_are_rounded_under_a_running_maximum(ws, n_q, pages, stretch):
    """The distance from the 64-bit result is that of the same sums in 64 bits
    with P rounded to bf16 under the stated maximum (of the first 32 keys, and
    raised by every 32 keys that exceed it by more than 8), to 1%: under a
    shift unrelated to the row's weights it is 1.3% to 4.9% larger where the
    row maximum reaches 40 to 65, its largest weight being rounded too."""
    rng = np.random.default_rng(int(1000 * stretch) + n_q)
    H, n_keys = 4, 64 * pages
    q, k, v = (synth.normal_bf16(rng, (n, H, 128)) for n in (n_q, n_keys, n_keys))
    q = _bits(stretch * synth.bf16_to_f32(q))
    got = _run(ws, q, k, v)
    qf, kf, vf = bf16_f64(_bits(synth.bf16_to_f32(q) * np.float32(np.log2(np.e) / np.sqrt(128)))), bf16_f64(k), bf16_f64(v)
    exact, lazy = np.empty_like(got), np.empty_like(got)
    for h in range(H):
        s = qf[:, h] @ kf[:, h].T
        p = np.exp2(s - s.max(axis=1, keepdims=True))
        exact[:, h] = (p @ vf[:, h]) / p.sum(1, keepdims=True)
        m, o, l = s[:, :32].max(1), 0.0, 0.0
        for c in range(0, n_keys, 32):
            top = s[:, c:c + 32].max(1)
            up = np.where(top > m + 8, top - m, 0.0)
            m = m + up
            pb = bf16_f64(_bits(np.exp2(s[:, c:c + 32] - m[:, None])))
            o = o * np.exp2(-up)[:, None] + pb @ vf[c:c + 32, h]
            l = l * np.exp2(-up) + pb.sum(1)
        lazy[:, h] = bf16_f64(_bits(o / l[:, None]))
    mine, want = (np.linalg.norm(x - exact) / np.linalg.norm(exact) for x in (got, lazy))
    print(f"stretch {stretch} rows {n_q} pages {pages}: {mine:.6f}, in 64 bits {want:.6f}, {mine / want:.4f}", flush=True)
    assert abs(mine / want - 1) <= 0.01
