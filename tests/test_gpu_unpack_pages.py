"""GPU: the E4M3 unpack (a wave per page and heads) at head counts that leave
waves and lanes without work, ragged lengths and offsets that are aligned to
one byte only, bit for bit against a plain index map."""
import numpy as np
import pytest

import oracle
from paper_2511_20982_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu(require_gpu):
    pass


from tests import gpu_util as G  # noqa: E402


@pytest.mark.parametrize("hkv,d,layers", [(1, 64, 3), (3, 64, 1), (6, 64, 2), (1, 128, 2), (9, 128, 1)])
@pytest.mark.parametrize("shift", [0, 3])
def test_unpack_e4m3(hkv, d, layers, shift):
    rng = np.random.default_rng(hkv + d + shift)
    lens = np.array([1, 16, 0, 17, 100, 31, 64], np.int32)
    pt, num_pages = I.allocate_pages(rng, np.maximum(lens[::-1], 1))
    offs = I.handoff_offsets(lens, layers, hkv, d) + shift * np.arange(len(lens) + 1)
    buf = rng.integers(0, 256, int(offs[-1]), dtype=np.uint8)
    kp = rng.integers(0, 256, (layers, num_pages, hkv, 16, d), dtype=np.uint8)
    vp = rng.integers(0, 256, (layers, num_pages, hkv, d, 16), dtype=np.uint8)
    req = np.arange(len(lens), dtype=np.int32)[::-1].copy()
    ek, ev = kp.copy(), vp.copy()
    for n, r in enumerate(req):
        x = buf[offs[n]:offs[n] + layers * 2 * hkv * lens[n] * d].reshape(layers, 2, hkv, lens[n], d)
        for t in range(int(lens[n])):
            page = pt[r, t // 16]
            ek[:, page, :, t % 16, :] = x[:, 0, :, t]
            ev[:, page, :, :, t % 16] = x[:, 1, :, t]
    shape = G.A.make_shape(hkv, hkv, d, "fp8")
    gk, gv = G.gpu_unpack(shape, buf, offs[:-1].copy(), req, lens, kp, vp, layers, pt)
    assert np.array_equal(gk, ek) and np.array_equal(gv, ev)


@pytest.mark.parametrize("hkv,d", [(5, 64), (3, 128)])
def test_unpack_e4m3_last_pages(hkv, d):
    """Last pages of 1 to 16 tokens."""
    rng = np.random.default_rng(hkv + d)
    lens = np.arange(1, 34, dtype=np.int32)
    pt, num_pages = I.allocate_pages(rng, lens)
    offs = I.handoff_offsets(lens, 2, hkv, d)
    buf = rng.integers(0, 256, int(offs[-1]), dtype=np.uint8)
    kp = rng.integers(0, 256, (2, num_pages, hkv, 16, d), dtype=np.uint8)
    vp = rng.integers(0, 256, (2, num_pages, hkv, d, 16), dtype=np.uint8)
    req = np.arange(len(lens), dtype=np.int32)
    got = G.gpu_unpack(G.A.make_shape(hkv, hkv, d, "fp8"), buf, offs[:-1].copy(), req, lens, kp, vp, 2, pt)
    for g, e in zip(got, oracle.unpack(buf, offs, req, lens, kp, vp, 2, pt)):
        assert np.array_equal(g, e)


@pytest.mark.parametrize("dtype,hkv,d,shift", [("bf16", 8, 128, 0), ("bf16", 8, 128, 3), ("fp32", 8, 64, 0)])
def test_unpack_of_a_large_buffer(dtype, hkv, d, shift):
    """Buffers above 128 MiB are read with other loads; compared on the GPU."""
    import torch

    gen = torch.Generator(device="cuda").manual_seed(7)
    size, t = (2, torch.int16) if dtype == "bf16" else (4, torch.int32)
    layers = 9
    lens = np.array([1, 2049, 0, 2100], np.int32)
    offs = I.handoff_offsets(lens, layers, hkv, d) + shift
    assert (offs[-1] - shift) * size > 128 << 20
    pt, num_pages = I.allocate_pages(np.random.default_rng(8), np.maximum(lens, 1))
    rand = lambda *s: torch.randint(-2 ** 15, 2 ** 15, s, dtype=t, device="cuda", generator=gen)  # noqa: E731
    buf = rand(int(offs[-1]))
    kp, vp = rand(layers, num_pages, hkv, 16, d), rand(layers, num_pages, hkv, d, 16)
    ek, ev = kp.clone(), vp.clone()
    for r, n in enumerate(lens):
        x = buf[offs[r]:offs[r] + layers * 2 * hkv * int(n) * d].view(layers, 2, hkv, int(n), d)
        for i in range((int(n) + 15) // 16):
            rows = x[:, :, :, 16 * i:16 * (i + 1)]
            ek[:, pt[r, i], :, :rows.shape[3]] = rows[:, 0]
            ev[:, pt[r, i], :, :, :rows.shape[3]] = rows[:, 1].transpose(-1, -2)
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    G.A.dopd_kv_unpack_from_handoff(G.A.make_shape(hkv, hkv, d, dtype), layers, buf, dev(offs[:-1].copy()),
                                    dev(np.arange(4, dtype=np.int32)), dev(lens), lens, 4, kp, vp, num_pages,
                                    dev(pt), pt.shape[1])
    assert torch.equal(kp, ek) and torch.equal(vp, ev)


@pytest.mark.parametrize("dtype,hkv,d,shift", [("bf16", 8, 128, 0), ("bf16", 8, 64, 3), ("fp32", 4, 128, 0),
                                               ("fp32", 8, 64, 1), ("fp8", 16, 128, 0), ("fp8", 16, 64, 5)])
def test_pack_of_a_large_buffer(dtype, hkv, d, shift):
    """Buffers above 128 MiB are packed with other loads; compared on the GPU."""
    import torch

    gen = torch.Generator(device="cuda").manual_seed(9)
    t = {"bf16": torch.int16, "fp32": torch.int32, "fp8": torch.uint8}[dtype]
    layers = 9 * 128 // d
    lens = np.array([1, 2049, 0, 2100], np.int32)
    offs = I.handoff_offsets(lens, layers, hkv, d) + shift
    assert (offs[-1] - shift) * t.itemsize > 128 << 20
    pt, num_pages = I.allocate_pages(np.random.default_rng(10), np.maximum(lens, 1))
    lo, hi = (0, 256) if dtype == "fp8" else (-2 ** 15, 2 ** 15)
    rand = lambda *s: torch.randint(lo, hi, s, dtype=t, device="cuda", generator=gen)  # noqa: E731
    buf = rand(int(offs[-1]))
    kp, vp = rand(layers, num_pages, hkv, 16, d), rand(layers, num_pages, hkv, d, 16)
    want = buf.clone()
    for r, n in enumerate(lens):
        x = want[offs[r]:offs[r] + layers * 2 * hkv * int(n) * d].view(layers, 2, hkv, int(n), d)
        for i in range((int(n) + 15) // 16):
            rows = x[:, :, :, 16 * i:16 * (i + 1)]
            rows[:, 0] = kp[:, pt[r, i], :, :rows.shape[3]]
            rows[:, 1] = vp[:, pt[r, i], :, :, :rows.shape[3]].transpose(-1, -2)
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    G.A.dopd_kv_pack_for_handoff(G.A.make_shape(hkv, hkv, d, dtype), layers, kp, vp, num_pages, dev(pt), pt.shape[1],
                                 dev(np.arange(4, dtype=np.int32)), dev(lens), lens, dev(offs[:-1].copy()), 4, buf)
    assert torch.equal(buf, want)
