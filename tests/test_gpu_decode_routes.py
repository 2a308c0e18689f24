"""GPU: the decode's two routes (one workgroup per whole (request, KV head);
slices of a partition with merged partials) at the sizes where waves, pairs of
pages and page-id chunks end, against the fp64 oracle and each other."""
import numpy as np
import pytest

import oracle
from paper_2511_20982_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu(require_gpu):
    pass


from tests import gpu_util as G  # noqa: E402

SCALES = lambda hkv: (np.linspace(0.01, 0.02, hkv, dtype=np.float32),  # noqa: E731
                      np.linspace(0.012, 0.022, hkv, dtype=np.float32))


def both_routes(w, dtype):
    """(reference, automatic, 64-token slices): out and lse of each."""
    if dtype == "fp8":
        ks, vs = SCALES(w.hkv)
        kq, vq = G.quantize_pools(w.k_pool, w.v_pool, ks, vs)
        ref = oracle.decode_e4m3(w.q_dec, kq, vq, ks, vs, w.page_table, w.context_lens, w.scale)
        shape = G.A.make_shape(w.hq, w.hkv, w.d, "fp8", w.scale)
        return ref, *(G.gpu_decode_fp8(shape, w.q_dec, kq, vq, ks, vs, w.page_table, w.context_lens, split=s)
                      for s in (0, 64))
    ref = oracle.decode(w.q_dec, w.k_pool, w.v_pool, w.page_table, w.context_lens, w.scale)
    return ref, *(G.gpu_decode(G.shape_of(w), w.q_dec, w.k_pool, w.v_pool, w.page_table, w.context_lens, split=s)
                  for s in (0, 64))


def check(w, dtype):
    (ref, ref_lse), *got = both_routes(w, dtype)
    for name, (out, lse) in zip(("automatic", "slices of 64"), got):
        G.assert_attention_close(out, ref, "bf16", f"{w.name} {dtype} {name}")
        assert np.max(np.abs(lse - ref_lse)) < 2e-2, name


@pytest.mark.parametrize("hq,hkv,d", [(8, 8, 128), (28, 4, 128), (16, 1, 64), (10, 5, 64)])
@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
def test_direct_route_edges(dtype, hq, hkv, d):
    """Every wave empty but one, a ragged pair, the eighth wave's first pair, its second."""
    ctx = [1, 16, 17, 31, 32, 33, 64, 225, 255, 256]
    check(I.decode_workload("edges", 70 + hq + d, ctx, hq, hkv, d), dtype)


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
def test_direct_route_long(dtype):
    """Equal contexts past the 256 pairs whose page ids eight waves hold at
    once (the requests share their pages)."""
    w = I.decode_workload("long", 71, [8193 + 40], 16, 8, 64)
    n = 32
    rng = np.random.default_rng(72)
    w.page_table = np.repeat(w.page_table, n, axis=0)
    w.context_lens = np.full(n, w.context_lens[0], np.int32)
    w.context_lens[::5] -= 17
    w.q_dec = I.normal(rng, (n, w.hq, w.d), "bf16")
    check(w, dtype)


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("n,lo,hi", [(1, 3000, 3000), (80, 1, 900), (40, 100, 4000)])
def test_partition_route(dtype, n, lo, hi):
    """One long context; more (request, KV head) than CUs; uneven contexts."""
    rng = np.random.default_rng(73 + n)
    check(I.decode_workload("partition", 74 + n, rng.integers(lo, hi + 1, n), 28, 4, 128), dtype)
