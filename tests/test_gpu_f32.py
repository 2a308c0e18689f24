"""GPU: the fp32 attention kernel at the edges of its tiles (16 columns of
(row, head) pairs, 16 keys, waves without keys), against the fp64 oracle, and
values no row may take from keys it does not see."""
import numpy as np
import pytest

import oracle
from paper_2511_20982_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu(require_gpu):
    pass


from tests import gpu_util as G  # noqa: E402
from tests.test_gpu_prefill_paged import paged_case  # noqa: E402

# g = 1, 4, 7, 20: columns that fill tiles evenly, unevenly and more than one
HEADS = [(2, 2), (8, 2), (7, 1), (20, 1)]


@pytest.mark.parametrize("hq,hkv", HEADS)
@pytest.mark.parametrize("d", [64, 128])
def test_f32_prefill_and_decode(hq, hkv, d):
    rng = np.random.default_rng(90 + hq + d)
    lens = np.array([1, 2, 15, 16, 17, 0, 33, 64, 129, 200], np.int32)
    q, k, v = I.prefill_batch(rng, lens, hq, hkv, d, "fp32")
    cu = I.cu_from_lens(lens)
    shape = G.A.make_shape(hq, hkv, d, "fp32")
    ref, ref_lse = oracle.prefill(q, k, v, cu, shape.softmax_scale)
    out, lse = G.gpu_prefill(shape, q, k, v, cu)
    G.assert_attention_close(out, ref, "fp32", "fp32 prefill")
    assert np.max(np.abs(lse - ref_lse)) < 1e-5

    w = I.decode_workload("f32", 91 + hq, [1, 16, 17, 127, 128, 129, 500], hq, hkv, d, "fp32")
    ref, ref_lse = oracle.decode(w.q_dec, w.k_pool, w.v_pool, w.page_table, w.context_lens, w.scale)
    out, lse = G.gpu_decode(G.shape_of(w), w.q_dec, w.k_pool, w.v_pool, w.page_table, w.context_lens)
    G.assert_attention_close(out, ref, "fp32", "fp32 decode")
    assert np.max(np.abs(lse - ref_lse)) < 1e-5

    q, kp, vp, pt, cu, pre = paged_case(92 + hq, [0, 1, 15, 16, 130, 0], [5, 17, 1, 40, 33, 0], hq, hkv, d, "fp32")
    ref, ref_lse = oracle.prefill_paged(q, kp, vp, pt, cu, pre, shape.softmax_scale)
    out, lse = G.gpu_prefill_paged(shape, q, kp, vp, pt, cu, pre)
    G.assert_attention_close(out, ref, "fp32", "fp32 chunk prefill")
    assert np.max(np.abs(lse - ref_lse)) < 1e-5


@pytest.mark.parametrize("scale", [0.0, -0.3, 4.0])
def test_f32_scales(scale):
    rng = np.random.default_rng(93)
    lens = np.array([40, 130], np.int32)
    q, k, v = I.prefill_batch(rng, lens, 8, 2, 64, "fp32")
    cu = I.cu_from_lens(lens)
    ref, _ = oracle.prefill(q, k, v, cu, scale)
    out, _ = G.gpu_prefill(G.A.make_shape(8, 2, 64, "fp32", scale), q, k, v, cu)
    # scores up to 4 * 8 sqrt(64) round to 2^-24 of their size each way: at scale 4 that
    # moves a weight by up to 4e-5 of itself (64 terms), the bar at scale <= 1 otherwise
    assert np.max(np.abs(out - ref)) < (1e-5 if abs(scale) <= 1 else 1e-4)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_f32_unseen_keys_never_reach_a_row(d, bad):
    """A V (or K) row that is not finite reaches the rows that see it and no other."""
    rng = np.random.default_rng(94)
    lens = np.array([70], np.int32)
    q, k, v = I.prefill_batch(rng, lens, 8, 2, d, "fp32")
    cu = I.cu_from_lens(lens)
    shape = G.A.make_shape(8, 2, d, "fp32")
    ref, _ = oracle.prefill(q, k, v, cu, shape.softmax_scale)
    for which in (v, k):
        t = 37
        x = which.copy()
        x[t] = bad
        kk, vv = (k, x) if which is v else (x, v)
        out, _ = G.gpu_prefill(shape, q, kk, vv, cu)
        assert np.max(np.abs(out[:t] - ref[:t])) < 1e-5
        if which is v:
            assert not np.isfinite(out[t:]).any()


def plain_f32(q, k, v, cu, scale):
    """Prefill in fp32 with nothing reordered for speed: a score's products added
    pair by pair, the keys one after the other with an online softmax, the
    exponentials rounded correctly."""
    f, (_, hq, d) = np.float32, q.shape
    out, g = np.zeros(q.shape, f), hq // k.shape[1]
    exp = lambda x: np.exp(x.astype(np.float64)).astype(f)  # noqa: E731
    for a, b in zip(cu[:-1], cu[1:]):
        kk, vv = np.repeat(k[a:b], g, 1), np.repeat(v[a:b], g, 1)
        m, l = np.full((b - a, hq), -np.inf, f), np.zeros((b - a, hq), f)
        o = np.zeros((b - a, hq, d), f)
        for j in range(b - a):
            x = q[a + j:b] * kk[j]
            while x.shape[-1] > 1:
                x = x[..., : x.shape[-1] // 2] + x[..., x.shape[-1] // 2:]
            s = x[..., 0] * f(scale)
            top = np.maximum(m[j:], s)
            alpha, p = exp(m[j:] - top), exp(s - top)
            l[j:] = l[j:] * alpha + p
            o[j:] = o[j:] * alpha[..., None] + p[..., None] * vv[j]
            m[j:] = top
        out[a:b] = o * (f(1) / l)[..., None]
    return out


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("longest", [16, 50, 120])
def test_f32_error_is_no_larger_than_plain_fp32(d, longest):
    """In the 2-norm over some thousand outputs, which one seed in the next moves by 2 %."""
    rng = np.random.default_rng(95)
    lens = rng.integers(longest // 2, longest + 1, 6).astype(np.int32)
    q, k, v = I.prefill_batch(rng, lens, 8, 2, d, "fp32")
    cu = I.cu_from_lens(lens)
    shape = G.A.make_shape(8, 2, d, "fp32")
    ref, _ = oracle.prefill(q, k, v, cu, shape.softmax_scale)
    plain = np.linalg.norm(plain_f32(q, k, v, cu, shape.softmax_scale) - ref)
    fresh, _ = G.gpu_prefill(shape, q, k, v, cu)
    # the same prompts as chunks over pages
    pt, num_pages = I.allocate_pages(rng, lens)
    kp, vp = oracle.kv_write(k, v, *I.empty_pools(num_pages, 2, d, "fp32"), pt, cu, np.zeros(6, np.int32))
    paged, _ = G.gpu_prefill_paged(shape, q, kp, vp, pt, cu, np.zeros(6, np.int32))
    for what, out in (("fresh rows", fresh), ("pages", paged)):
        ratio = float(np.linalg.norm(out - ref) / plain)
        assert ratio <= 1, f"{what}: {ratio:.3f} of plain fp32"


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_f32_one_tile(d, bad):
    """A single tile is stored without the merge: values that are not finite, and
    scores that are all minus infinity, come out as the merge would have them."""
    rng = np.random.default_rng(96)
    lens = np.array([12, 3], np.int32)
    q, k, v = I.prefill_batch(rng, lens, 3, 1, d, "fp32")
    cu = I.cu_from_lens(lens)
    shape = G.A.make_shape(3, 1, d, "fp32")
    v[5] = bad
    with np.errstate(invalid="ignore"):
        ref, ref_lse = oracle.prefill(q, k, v, cu, shape.softmax_scale)
    out, lse = G.gpu_prefill(shape, q, k, v, cu)
    np.testing.assert_allclose(out, ref, rtol=0, atol=1e-5)
    np.testing.assert_allclose(lse, ref_lse, rtol=0, atol=1e-5)
    q[:] = 1
    k[:] = -np.inf
    out, lse = G.gpu_prefill(shape, q, k, v, cu)
    assert np.isnan(out).all() and np.isnan(lse).all()


def test_f32_decode_of_more_workgroups_than_a_grid_dimension_takes():
    """8.4 million (request, KV head) pairs of one key each, whose V they return."""
    import torch

    n, hkv, d = 1 << 16, 129, 64
    shape = G.A.make_shape(hkv, hkv, d, "fp32")
    gen = torch.Generator(device="cuda").manual_seed(9)
    kp, vp = (torch.randn(s, device="cuda", generator=gen) for s in ((5, hkv, 16, d), (5, hkv, d, 16)))
    page = torch.arange(n, device="cuda", dtype=torch.int32).remainder(5).view(n, 1).contiguous()
    ctx = np.ones(n, np.int32)
    q = torch.randn(n, hkv, d, device="cuda", generator=gen)
    out = torch.full_like(q, float("nan"))
    G.A.dopd_decode_attn(shape, q, kp, vp, 5, page, 1, torch.from_numpy(ctx).cuda(), ctx, n, 0, out, None,
                         G.A.decode_workspace(shape, ctx, n))
    assert torch.equal(out, vp[page.view(-1).long(), :, :, 0])
