"""The video kernel at the edges of its tiles, its page stream and its softmax
shift, against the fp64 oracle with the parity gates: subtiles of 16 rows,
waves of 32 (tiles up to 128 rows) and 64 rows, ragged pages, streams longer
than the 128-unit entry window, shares that cross several heads, and rows under
a running maximum whose logit bound is attained or far above every logit."""
import numpy as np
import pytest

import oracle
from helpers import Loaded, assert_gates, bf16_f64, video_waves
from paper_2607_04443_amd import synth

pytestmark = pytest.mark.gpu
COND = (synth.KIND_COND,)


def _workload(H, k, v):
    cfg = synth.Config("edges", 20, H, (1, 1), k.shape[0], 0)
    wl = synth.make_workload(cfg)
    wl.cached[0].k, wl.cached[0].v = k, v
    return wl


def _check(ws, q, k, v, splits=0, label="", tile=None, prepared=False, every=1):
    """RAW rows (or, prepared, the same rows with the scale folded in, which take
    the other of the two video kernels), in query tiles of `tile` rows; every
    `every`-th row against the oracle."""
    n_q, H = q.shape[0], q.shape[1]
    if tile is not None:
        assert video_waves(H, n_q, -(-k.shape[0] // 64), splits)[0] == tile, label
    L = Loaded(ws, _workload(H, k, v), max_pages=k.shape[0] // 64 + 8, max_q_tokens=max(64, n_q))
    try:
        pos = np.zeros((n_q, 3), np.int32)
        L.cache.set_option(ws.WS_OPT_VIDEO_KV_SPLITS, splits)
        if prepared:
            q = synth.bf16_bits(synth.bf16_to_f32(q) * np.float32(np.log2(np.e) / np.sqrt(128.0)))
        got = L.run("video", q, pos, 0, COND, mode=ws.WS_QUERY_PREPARED if prepared else ws.WS_APPEND_RAW)
        ref = oracle.unit_attention(L.ocache, q[::every], 0, mode=oracle.MODE_RAW,
                                    scale=np.log(2.0) if prepared else None, kind_mask=1 << synth.KIND_COND)[0]
        assert_gates(got[::every], ref, label=label)
        return got
    finally:
        L.close()


@pytest.mark.parametrize("n_q", [15, 16, 17, 32, 48, 64, 65, 96, 127, 130, 160, 192, 193, 255, 256, 257, 300, 385])
def test_row_counts(ws, n_q):
    rng = np.random.default_rng(100 + n_q)
    H, n_keys = 3, 64 * 3 + 1 + n_q % 63
    q, k, v = (synth.normal_bf16(rng, (n, H, 128)) for n in (n_q, n_keys, n_keys))
    _check(ws, q, k, v, label=f"{n_q} rows, {n_keys} keys")


@pytest.mark.parametrize("n_keys", [1, 4, 8, 31, 32, 33, 63, 64, 65, 96, 128, 129, 300, 384])
@pytest.mark.parametrize("n_q", [30, 200])
def test_key_counts(ws, n_q, n_keys):
    rng = np.random.default_rng(200 + n_keys)
    q, k, v = (synth.normal_bf16(rng, (n, 2, 128)) for n in (n_q, n_keys, n_keys))
    _check(ws, q, k, v, label=f"{n_q} rows, {n_keys} keys")


@pytest.mark.parametrize("n_q", [20, 140])
@pytest.mark.parametrize("pages,splits", [(128, 1), (129, 1), (150, 1), (193, 1), (262, 1), (270, 2)])
def test_streams_longer_than_the_entry_window(ws, n_q, pages, splits):
    """One share per head and range: a stream of `pages` / `splits` units."""
    rng = np.random.default_rng(300 + pages)
    n_keys = 64 * pages - 23
    q, k, v = (synth.normal_bf16(rng, (n, 2, 128)) for n in (n_q, n_keys, n_keys))
    _check(ws, q, k, v, splits, label=f"{pages} pages in {splits}")


@pytest.mark.parametrize("H,n_q,n_keys", [(64, 1300, 64 * 2 + 5), (96, 2600, 40), (50, 900, 64 * 7)])
def test_shares_across_heads(ws, H, n_q, n_keys):
    rng = np.random.default_rng(400 + H)
    q, k, v = (synth.normal_bf16(rng, (n, H, 128)) for n in (n_q, n_keys, n_keys))
    _check(ws, q, k, v, label=f"{H} heads x {n_q} rows")


# Rows, forced key ranges (1: tiles of 256 rows) and the tile: waves of 32 rows
# twice (a short last tile, a narrow tile), of 64 and of 48.
WAVES = [(40, 0, 256), (200, 0, 128), (200, 1, 256), (250, 0, 192)]


@pytest.mark.parametrize("n_q,splits,tile", WAVES)
@pytest.mark.parametrize("stretch", [3.0, 5.0, 9.0])
@pytest.mark.parametrize("prepared", [False, True])
def test_shift_below_an_attained_bound(ws, n_q, splits, tile, stretch, prepared):
    """Each query's dominant key is `stretch` times its own direction: the
    logit bound (16.3 stretch in log2 units, above 40) is attained where a row's
    maximum is raised to it, and every other weight is below 2^-20 of it, so
    each row returns its key's V."""
    rng = np.random.default_rng(500 + n_q)
    H, n_keys = 2, 331 if n_q < 331 else 389  # (a prime above the row count: a key per row)
    q, k, v = (synth.normal_bf16(rng, (n, H, 128)) for n in (n_q, n_keys, n_keys))
    qf = synth.bf16_to_f32(q)
    q = synth.bf16_bits(qf / np.sqrt((qf * qf).mean(-1, keepdims=True)))
    for i in range(n_q):
        k[(i * 29 + 3) % n_keys] = synth.bf16_bits(stretch * synth.bf16_to_f32(q[i]))
    got = _check(ws, q, k, v, splits, f"needles x {stretch}", tile, prepared)
    # the other keys together weigh at most 388 2^-20: an output rounding
    want = bf16_f64(v[(np.arange(n_q) * 29 + 3) % n_keys])
    assert (np.abs(got - want) <= 2.0 ** -8 * np.abs(want) + 0.005).all()


@pytest.mark.parametrize("n_keys", [1, 64 * 3 + 24])
@pytest.mark.parametrize("n_q,splits,tile,mixed", [(40, 0, 256, False), (200, 0, 128, True), (200, 1, 256, True),
                                                   (250, 0, 192, True)])
def test_rows_out_of_the_shift_s_reach(ws, n_q, splits, tile, n_keys, mixed):
    """Every key points away from the queries and is 7 times as long: the bound
    is about 114 in log2 units and every logit about minus that, so no shift
    near the bound serves (`mixed`: with ordinary rows of a tenth the length,
    which have a fixed shift, in the same waves)."""
    rng = np.random.default_rng(600 + n_q + n_keys)
    H = 2
    base = rng.standard_normal((1, H, 128)).astype(np.float32)
    base /= np.sqrt((base * base).mean(-1, keepdims=True))
    qf = np.repeat(base, n_q, axis=0)
    if mixed:
        qf[1::2] *= 0.1
    q = synth.bf16_bits(qf)
    k = synth.bf16_bits(-7.0 * base + 0.02 * rng.standard_normal((n_keys, H, 128)).astype(np.float32))
    v = synth.normal_bf16(rng, (n_keys, H, 128))
    s = np.log2(np.e) / np.sqrt(128.0)
    logits = s * np.einsum("qhd,khd->qhk", bf16_f64(q), bf16_f64(k))
    assert logits[0].max() < -100, logits[0].max()
    got = _check(ws, q, k, v, splits, f"out of reach, {n_keys} keys, mixed {mixed}", tile)
    if n_keys == 1:
        np.testing.assert_array_equal(got, bf16_f64(np.repeat(v, n_q, axis=0)))


# What the last tile holds: rows per tile, rows per wave, waves without rows.
@pytest.mark.parametrize("grid,n_a,audio_tokens,splits,waves", [
    ((12, 21), 4, 4, 1, (256, 64, 0)),    # every wave has rows, the last attends the riders' pages afterwards
    ((12, 21), 4, 4, 3, (256, 64, 0)),    # the same in three ranges
    ((12, 21), 4, 40, 1, (256, 64, 0)),   # one range per head takes all of them
    ((12, 21), 4, 4, 0, (192, 32, 2)),    # 64 rows in the last tile
    ((8, 15), 8, 4, 0, (256, 32, 0)),     # 128 rows, none idle
    ((9, 9), 5, 4, 0, (256, 32, 1)),      # 86 rows
    ((10, 17), 17, 12, 1, (256, 64, 1)),  # 187 rows, two passes of 16 riders
    ((10, 17), 17, 12, 0, (128, 32, 2)),  # 59 rows in the last tile
])
def test_rider_pages_in_busy_and_idle_waves(ws, grid, n_a, audio_tokens, splits, waves):
    from test_gpu_riders import ALL, VIDEO, Step
    S = Step(ws, 6, grid, 100, audio_tokens, 4, 71)
    try:
        S.cache.set_option(ws.WS_OPT_VIDEO_KV_SPLITS, splits)
        u, n_v = S.unit, grid[0] * grid[1]
        vmask, amask = (u, u - 3, VIDEO), (u, u - 3, ALL)
        assert video_waves(6, n_v, 2 + 4 * -(-n_v // 64), splits, n_a) == waves
        qv, qa = S.queries(n_v), S.queries(n_a)
        fv, fa, rec = S.step(qv, qa, vmask, amask)
        assert rec[1]["path"] == "audio_riders" and rec[1]["n_splits"] == 0, rec
        np.testing.assert_array_equal(fv, S.separate_video(qv, vmask))
        assert_gates(bf16_f64(fa), S.oracle(qa, amask), label="riders", bound=S.bound(qa, amask))
        assert_gates(bf16_f64(fv), S.oracle(qv, vmask), label="video rows")
    finally:
        S.close()
