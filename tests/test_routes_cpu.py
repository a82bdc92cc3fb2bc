"""Which Sinkhorn kernel takes which image, without a GPU: every image that a call can hold has a kernel
that the call launches, on chip where one fits, and is held in as many bits as it ever was."""
import numpy as np
import pytest

from paper_2605_00392_amd import rtprune as rt

LENGTHS = (513, 640, 1083, 1156, 1441, 1500, 1900, 2137, 2900, 3584, 3586, 4512, 7779, 8192)
FIXED = (0.12, 0.3, 0.45, 0.517, 0.5793, 0.617, 0.7, 0.84, 0.9, 0.93, 0.95, 0.97, 1.0)
CLAMPS = (0.4, 0.6, 0.84, 0.9)


def kept_count(ratio, n):
    return np.minimum(np.maximum(np.ceil(np.float64(np.float32(ratio)) * n - 1e-3), 1), n).astype(np.int64)


def routes(max_tokens, m, r, own=0, batch=64, **params):
    rc, route = rt.rtprune_sinkhorn_routes(batch, max_tokens, rt.make_params(**params), own, m, r)
    assert rc == rt.RTP_OK
    return route & 15, (route & rt.RTP_ROUTE_F32) != 0


def cluster_shape(m, r):
    """Workgroups of 224, 448, 144 and 80 rows for images of up to 1792 x 128, 3584 x 128, 1152 x 576 and
    1280 x 960, the first that holds one; 0: beyond all."""
    g = lambda rows: -(-m // rows)
    return np.select([(m <= 1792) & (r <= 128), (m <= 3584) & (r <= 128), (m <= 1152) & (r <= 576), (m <= 1280) & (r <= 960)],
                     [g(224), g(448), g(144), g(80)], 0)


def on_chip_f32(max_tokens, m, r, params):
    """The images (beyond the one-workgroup shapes) that may be held as fp32: (on chip, or if streamed).  The
    longest page of a fixed retention says how many workgroups an image may take, eight under a
    dynamic one; a page beyond all shapes has the streaming kernels launched, which hold fp32."""
    g = cluster_shape(m, r)
    if params.get("dynamic"):
        return (g > 0) & (g <= 8), max_tokens - 1 > 3584
    m_top = int(kept_count(params["ratio"], max_tokens))
    top = int(cluster_shape(np.int64(m_top), np.int64(max_tokens - m_top)))
    return (g > 0) & (g <= (top if top else 8)), top == 0


def all_calls():
    for n in LENGTHS:
        for ratio in FIXED:
            yield n, dict(ratio=ratio)
        for clamp in CLAMPS:
            yield n, dict(dynamic=1, ratio_min=clamp)


def images(max_tokens, params, rng, own, count=4000):
    """Kept and pruned counts that such a call can hold."""
    n = np.concatenate([rng.integers(2, max_tokens + 1, count), np.full(count // 4, max_tokens)])
    if own:
        m = np.where(rng.random(len(n)) < 0.5, rng.integers(1, n), n - np.minimum(n - 1, rng.integers(1, 1400, len(n))))
    elif params.get("dynamic"):
        m = rng.integers(kept_count(params["ratio_min"], n), n + 1)
    else:
        m = kept_count(params["ratio"], n)
    m, r = m[m < n], (n - m)[m < n]
    return m, r


def one_workgroup(m, r):
    """The shapes of one workgroup that come first: up to 7 x 64 rows and 7 pruned tokens, 512 x 15, 511 x 31,
    1535 x 15, 1216 x 64."""
    return ((m + 1 <= 448) & (r + 1 <= 8)) | ((m + 1 <= 512) & (r + 1 <= 32)) | ((m + 1 <= 1536) & (r + 1 <= 16)) | (
        (m <= 1216) & (r <= 64))


@pytest.mark.parametrize("own", [0, 1])
def test_every_image_has_a_kernel_that_the_call_launches(own):
    rng = np.random.default_rng(1)
    for n, params in all_calls():
        for batch in (1, 64, 1024):
            m, r = images(n, params, rng, own, 1000)
            to, _ = routes(n, m, r, own, batch, **params)
            bad = (to == rt.RTP_ROUTE_UNSERVED) | (to == rt.RTP_ROUTE_NONE)
            assert not bad.any(), (n, params, batch, m[bad][:4], r[bad][:4])


@pytest.mark.parametrize("own", [0, 1])
def test_no_image_is_held_in_fewer_bits(own):
    rng = np.random.default_rng(2)
    for n, params in all_calls():
        for batch in (1, 64, 1024):
            m, r = images(n, params, rng, own)
            to, f32 = routes(n, m, r, own, batch, **params)
            chip, streamed = on_chip_f32(n, m, r, params)
            several = ~one_workgroup(m, r)
            # fp64 stays fp64 ...
            bad = several & f32 & ~chip & (not streamed) & (to != rt.RTP_ROUTE_ONE_WORKGROUP)
            assert not bad.any(), (n, params, batch, m[bad][:4], r[bad][:4])
            # ... and what was rounded once from an fp64 exponential on chip does not go through the streaming
            # kernels' fp32 one
            bad = several & chip & (to == rt.RTP_ROUTE_STREAMED)
            assert not bad.any(), (n, params, batch, m[bad][:4], r[bad][:4])


def test_counts_of_the_callers_own_get_no_slower_kernel():
    """The staged calls take any kept counts, whatever the parameters expect: an image that some launch of
    several workgroups holds or streams under these parameters does not end up with the one-workgroup kernel."""
    rng = np.random.default_rng(3)
    for n, params in all_calls():
        for batch in (1, 64, 1024):
            m, r = images(n, params, rng, 1)
            to, _ = routes(n, m, r, 1, batch, **params)
            chip, streamed = on_chip_f32(n, m, r, params)
            bad = (to == rt.RTP_ROUTE_GENERAL) & (chip | (streamed & (r <= 2048)))
            assert not bad.any(), (n, params, batch, m[bad][:4], r[bad][:4])
    for n, params, image in [(2137, dict(ratio=0.84), (1238, 899)), (4512, dict(ratio=0.84), (2783, 1729)),
                             (4512, dict(ratio=0.7), (2783, 1729)), (1083, dict(ratio=0.9), (560, 523)),
                             (1083, dict(ratio=1.0), (560, 523)), (1083, dict(dynamic=1, ratio_min=0.9), (560, 523))]:
        to, _ = routes(n, [image[0]], [image[1]], 1, 64, **params)
        assert to[0] in (rt.RTP_ROUTE_STRIPS, rt.RTP_ROUTE_STREAMED), (n, params, image, to)


def test_staged_calls_of_a_pipeline_take_the_fused_calls_kernels():
    rng = np.random.default_rng(4)
    for n, params in all_calls():
        for batch in (1, 64, 1024):
            m, r = images(n, params, rng, 0)
            fused, staged = routes(n, m, r, 0, batch, **params), routes(n, m, r, 1, batch, **params)
            differ = (fused[0] != staged[0]) | (fused[1] != staged[1])
            assert not differ.any(), (n, params, batch, m[differ][:4], r[differ][:4], fused[0][differ][:4], staged[0][differ][:4])
