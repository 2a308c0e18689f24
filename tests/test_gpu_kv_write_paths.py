"""GPU: both mappings of the paged writers (whole pages of a few heads per
workgroup; single tokens), at head counts that leave waves without work, more
requests than a wave has lanes, empty requests and pages entered midway.  Bit
for bit against a plain index map."""
import numpy as np
import pytest

import oracle
from paper_2511_20982_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu(require_gpu):
    pass


from tests import gpu_util as G  # noqa: E402


def lengths(rng, nreq, tokens):
    """New tokens per request: `tokens` on average, empty ones among them."""
    n = rng.integers(0, 2 * tokens + 1, nreq)
    n[-1] = max(1, n[-1])
    return n.astype(np.int32)


# (requests, mean new tokens): one token each, either side of the mapping's
# line at two per request, whole prompts; 65 and 130 pass one wave's lanes
@pytest.mark.parametrize("nreq,tokens", [(1, 1), (65, 1), (130, 2), (66, 3), (3, 40)])
@pytest.mark.parametrize("hkv,d", [(1, 64), (3, 64), (5, 128), (8, 128)])
@pytest.mark.parametrize("dtype", ["bf16", "fp32", "fp8"])
def test_paged_write(dtype, hkv, d, nreq, tokens):
    rng = np.random.default_rng(nreq + 7 * tokens + 31 * hkv + d)
    fresh = "fp32" if dtype == "fp32" else "bf16"
    n = lengths(rng, nreq, tokens)
    start = rng.integers(0, 40, nreq).astype(np.int32)
    pt, num_pages = I.allocate_pages(rng, n + start)
    cu = I.cu_from_lens(n)
    total = int(cu[-1])
    k, v = I.normal(rng, (total, hkv, d), fresh), I.normal(rng, (total, hkv, d), fresh)
    shape = G.A.make_shape(hkv, hkv, d, dtype)
    kp, vp = I.empty_pools(num_pages, hkv, d, fresh)
    if dtype == "fp8":
        kp = rng.integers(0, 255, kp.shape, dtype=np.uint8)
        vp = rng.integers(0, 255, vp.shape, dtype=np.uint8)
        ks = (0.005 + 0.01 * rng.random(hkv)).astype(np.float32)
        vs = (0.005 + 0.01 * rng.random(hkv)).astype(np.float32)
        kw, vw = oracle.e4m3_quantize(k, ks), oracle.e4m3_quantize(v, vs)
        gk, gv = G.gpu_kv_write_fp8(shape, k, v, ks, vs, kp, vp, pt, cu, start)
    else:
        kw, vw = k, v
        gk, gv = G.gpu_kv_write(shape, k, v, kp, vp, pt, cu, start)
    ek, ev = kp.copy(), vp.copy()
    for r in range(nreq):
        for i in range(int(n[r])):
            p = int(start[r]) + i
            page = pt[r, p // 16]
            ek[page, :, p % 16, :] = kw[cu[r] + i]
            ev[page, :, :, p % 16] = vw[cu[r] + i]
    bits = {"bf16": np.uint16, "fp32": np.uint32, "fp8": np.uint8}[dtype]
    assert np.array_equal(gk.view(bits), ek.view(bits))
    assert np.array_equal(gv.view(bits), ev.view(bits))


# Rows in front of the first request's belong to nobody and go nowhere, whichever
# mapping the total (which counts them) chooses.
@pytest.mark.parametrize("nreq,before", [(2, 1), (70, 5), (3, 9)])
def test_rows_before_the_first_request(nreq, before):
    hkv, d = 3, 64
    rng = np.random.default_rng(nreq + before)
    start = rng.integers(0, 40, nreq).astype(np.int32)
    pt, num_pages = I.allocate_pages(rng, start + 1)
    cu = (before + np.arange(nreq + 1)).astype(np.int32)
    k, v = (I.normal(rng, (before + nreq, hkv, d), "bf16") for _ in range(2))
    kp, vp = I.empty_pools(num_pages, hkv, d, "bf16")
    gk, gv = G.gpu_kv_write(G.A.make_shape(hkv, hkv, d, "bf16"), k, v, kp, vp, pt, cu, start)
    ek, ev = kp.copy(), vp.copy()
    for r in range(nreq):
        page, slot = pt[r, start[r] // 16], start[r] % 16
        ek[page, :, slot, :] = k[before + r]
        ev[page, :, :, slot] = v[before + r]
    assert np.array_equal(gk.view(np.uint16), ek.view(np.uint16))
    assert np.array_equal(gv.view(np.uint16), ev.view(np.uint16))


# One long request among empty or single-token ones: at most two tokens per request
# on average, so its whole pages are written token by token too.  17 heads of 64
# are two waves of a row and a part of a third.
@pytest.mark.parametrize("hkv,d", [(1, 64), (17, 64), (8, 128)])
@pytest.mark.parametrize("others", [0, 1])
@pytest.mark.parametrize("dtype", ["bf16", "fp32", "fp8"])
def test_one_long_request_among_many(dtype, others, hkv, d):
    rng = np.random.default_rng(5 * hkv + d + others)
    n = np.full(70, others, np.int32)
    n[41] = 69
    start = rng.integers(0, 40, 70).astype(np.int32)
    pt, num_pages = I.allocate_pages(rng, n + start)
    cu = I.cu_from_lens(n)
    fresh = "fp32" if dtype == "fp32" else "bf16"
    k, v = (I.normal(rng, (int(cu[-1]), hkv, d), fresh) for _ in range(2))
    shape = G.A.make_shape(hkv, hkv, d, dtype)
    if dtype == "fp8":
        kp, vp = (rng.integers(0, 255, s, dtype=np.uint8) for s in ((num_pages, hkv, 16, d), (num_pages, hkv, d, 16)))
        scale = (0.005 + 0.01 * rng.random(hkv)).astype(np.float32)
        got = G.gpu_kv_write_fp8(shape, k, v, scale, scale, kp, vp, pt, cu, start)
        k, v = oracle.e4m3_quantize(k, scale), oracle.e4m3_quantize(v, scale)
    else:
        kp, vp = I.empty_pools(num_pages, hkv, d, fresh)
        got = G.gpu_kv_write(shape, k, v, kp, vp, pt, cu, start)
    for g, e in zip(got, oracle.kv_write(k, v, kp, vp, pt, cu, start)):
        assert np.array_equal(g.view(np.uint8), e.view(np.uint8))


# Every range of slots of a page, each the one touched page of a request: the slots
# of a dim row leave in pieces of 1 to 16, and none outside the range is touched.
@pytest.mark.parametrize("hkv,d", [(3, 64), (2, 128)])
@pytest.mark.parametrize("dtype", ["bf16", "fp32", "fp8"])
def test_every_range_of_a_page(dtype, hkv, d):
    rng = np.random.default_rng(hkv + d)
    start, end = np.array([(a, b) for a in range(16) for b in range(a + 1, 17)], np.int32).T
    n = end - start
    pt, num_pages = I.allocate_pages(rng, end)
    cu = I.cu_from_lens(n)
    fresh = "fp32" if dtype == "fp32" else "bf16"
    k, v = (I.normal(rng, (int(cu[-1]), hkv, d), fresh) for _ in range(2))
    shape = G.A.make_shape(hkv, hkv, d, dtype)
    if dtype == "fp8":
        kp, vp = (rng.integers(0, 255, s, dtype=np.uint8) for s in ((num_pages, hkv, 16, d), (num_pages, hkv, d, 16)))
        scale = (0.005 + 0.01 * rng.random(hkv)).astype(np.float32)
        got = G.gpu_kv_write_fp8(shape, k, v, scale, scale, kp, vp, pt, cu, start)
        k, v = oracle.e4m3_quantize(k, scale), oracle.e4m3_quantize(v, scale)
    else:
        kp, vp = I.empty_pools(num_pages, hkv, d, fresh)
        got = G.gpu_kv_write(shape, k, v, kp, vp, pt, cu, start)
    for g, e in zip(got, oracle.kv_write(k, v, kp, vp, pt, cu, start)):
        assert np.array_equal(g.view(np.uint8), e.view(np.uint8))
