"""GPU load-time transcoder (format-v1 codes -> Planes14 stream) through the C
ABI: on small shapes the codes come from the oracle's index and the stream
decodes (with the GEMV's own decoder) to the oracle's points; on every shape
the stream equals the host expansion byte for byte and its GEMV equals the
host-expanded matrix's bit for bit; invalid codes are counted."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2609_02652_amd as P  # noqa: E402
from paper_2609_02652_amd import _lib, synth  # noqa: E402
from oracle import index as I  # noqa: E402

pytestmark = pytest.mark.gpu


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    return torch.device("cuda:0")


@pytest.fixture(scope="module")
def dcb(dev):
    return P.DeviceCodebook(P.Codebook(12), dev)


def transcode_and_compare(dev, dcb, inp, codes, oracle_rows=None):
    M, nb = inp.M, inp.nb
    cls, sm, lv = dcb.cb.fields_from_points(inp.z)
    ref = P.LeechMatrix.from_fields(dcb, P.PLANES14, cls, inp.gain, sm, lv, inp.scale, dev)
    mat = P.LeechMatrix.from_codes(dcb, torch.from_numpy(codes.view(np.int64)).to(dev), inp.scale)
    assert mat.desc.as_dict() == ref.desc.as_dict()
    assert torch.equal(mat.main, ref.main), "transcoded stream differs from the host expansion"
    z, c, g = mat.decode()
    zc = z.cpu().numpy()
    if oracle_rows is None:
        assert np.array_equal(zc, inp.z)
    else:
        r, j = oracle_rows
        want = np.array([I.point_of_index(int(codes[a, b]) & ((1 << 47) - 1))
                         for a, b in zip(r, j)], dtype=np.int8)
        assert np.array_equal(zc[r, j], want)
    assert np.array_equal(g.cpu().numpy(), inp.gain)
    x = torch.from_numpy(inp.x).to(dev)
    y0 = ref.gemv(x, centroids=(0.75, 1.25)).cpu().numpy()
    y1 = mat.gemv(x, centroids=(0.75, 1.25)).cpu().numpy()
    assert np.array_equal(y0.view(np.uint32), y1.view(np.uint32))


@pytest.mark.parametrize("M,K", [(1, 24), (65, 408), (257, 792)])
def test_transcode_oracle_codes(dev, dcb, M, K):
    say(f"[transcode] oracle codes {M}x{K}")
    inp = synth.make_gemv_inputs(M, K, seed=M, name="transcode")
    codes = np.array([[I.code_of(I.index_of_point(inp.z[r, j]), int(inp.gain[r, j]))
                       for j in range(inp.nb)] for r in range(M)], dtype=np.uint64)
    transcode_and_compare(dev, dcb, inp, codes)


@pytest.mark.parametrize("M,K", [(14337, 120), (4096, 4096), (17408, 5120), (1024, 17408)])
def test_transcode_full_shapes(dev, dcb, M, K):
    """Tall odd-tile (lane_cols 1), the 8B q/o shape, the 14B gate/up shape
    and a wide one; codes from the host encoder, 512 blocks against the oracle."""
    say(f"[transcode] host codes {M}x{K}")
    inp = synth.make_gemv_inputs(M, K, seed=7, name="transcode-full")
    cls, sm, lv = dcb.cb.fields_from_points(inp.z)
    codes = P.index_encode(dcb.cb, cls, inp.gain, sm, lv)
    rng = np.random.default_rng(M)
    rows = (rng.integers(0, M, 512), rng.integers(0, inp.nb, 512))
    transcode_and_compare(dev, dcb, inp, codes, oracle_rows=rows)


def test_invalid_codes_are_counted_and_zeroed(dev, dcb):
    inp = synth.make_gemv_inputs(65, 408, seed=9, name="transcode-bad")
    cls, sm, lv = dcb.cb.fields_from_points(inp.z)
    codes = P.index_encode(dcb.cb, cls, inp.gain, sm, lv)
    N = I.class_offsets()[-1]
    planted = {(0, 0): 1 << 48, (10, 5): N, (64, 16): (1 << 47) - 1}
    for (r, j), v in planted.items():
        codes[r, j] = v
    with pytest.raises(P.LeechError, match="3 of"):
        P.LeechMatrix.from_codes(dcb, torch.from_numpy(codes.view(np.int64)).to(dev), inp.scale)
    desc = P.planes14_desc(65, 408)
    d_codes = torch.from_numpy(codes.view(np.int64)).to(dev)
    main = torch.full((desc.main_bytes,), 0xAB, dtype=torch.uint8, device=dev)
    bad = torch.full((1,), 77, dtype=torch.int32, device=dev)
    _lib.transcode_planes14(desc, dcb.index.data_ptr(), d_codes.data_ptr(), main.data_ptr(),
                            bad.data_ptr())
    torch.cuda.synchronize()
    assert int(bad.item()) == 3
    ref = P.LeechMatrix.from_fields(dcb, P.PLANES14, cls, inp.gain, sm, lv, inp.scale, dev)
    got, want = main.cpu().numpy(), ref.main.cpu().numpy()
    geo_index = host_storage_index(desc)
    for (r, j) in planted:
        s = geo_index(r, j)
        assert np.all(got[14 * s:14 * s + 14] == 0)
        want[14 * s:14 * s + 14] = 0
    assert np.array_equal(got, want)


@pytest.mark.parametrize("M,nb,geo", [(1, 1, (1, 4)), (1, 1, (16, 4)), (5, 3, (2, 32)), (63, 5, (3, 20)),
                                      (65, 2, (1, 64)), (4, 67, (8, 8)), (130, 19, (4, 16)),
                                      (37, 33, (16, 4)), (9, 4, (1, 4))])
def test_transcode_geometries(dev, dcb, M, nb, geo):
    """Runs of 64 slots that cross tiles and units, ragged last tiles and
    groups, units of one block: every slot's record is its block's."""
    say(f"[transcode] geometry {geo} {M}x{nb}")
    inp = synth.make_gemv_inputs(M, 24 * nb, seed=M + nb, name="transcode-geo")
    cls, sm, lv = dcb.cb.fields_from_points(inp.z)
    codes = P.index_encode(dcb.cb, cls, inp.gain, sm, lv)
    desc, main, _, _ = P.expand_layout(dcb.cb, P.PLANES14, cls, inp.gain, sm, lv, geo)
    d_codes = torch.from_numpy(codes.view(np.int64)).to(dev)
    got = torch.full((desc.main_bytes,), 0xAB, dtype=torch.uint8, device=dev)
    bad = torch.full((1,), 77, dtype=torch.int32, device=dev)
    _lib.transcode_planes14(desc, dcb.index.data_ptr(), d_codes.data_ptr(), got.data_ptr(),
                            bad.data_ptr())
    assert int(bad.item()) == 0
    assert np.array_equal(got.cpu().numpy(), main)
    # the scales' order on the device is the host's
    rows = torch.from_numpy(inp.scale.reshape(-1).view(np.int16)).to(dev)
    order = torch.zeros(M * nb + 1, dtype=torch.int16, device=dev)
    _lib.layout_scales_device(desc, rows.data_ptr(), order.data_ptr())
    want = P.layout_scales(desc, inp.scale).view(np.int16)
    assert np.array_equal(order.cpu().numpy(), np.append(want, np.int16(0)))


def test_transcode_tile_past_32_bits(dev, dcb):
    """One row of 2^29 + 3 blocks in tiles of 4: a tile of more than 2^31 slots
    takes the 64-bit slot arithmetic.  With one row the stream is in block
    order, so it must be the records of the repeated pool of codes."""
    nb, pool = (1 << 29) + 3, 4099
    if torch.cuda.mem_get_info(dev)[0] < 24 << 30:
        pytest.skip("needs 24 GB of device memory")
    say("[transcode] one row past 32-bit tiles")
    inp = synth.make_gemv_inputs(1, 24 * pool, seed=3, name="transcode-long")
    cls, sm, lv = dcb.cb.fields_from_points(inp.z)
    codes = torch.from_numpy(P.index_encode(dcb.cb, cls, inp.gain, sm, lv).view(np.int64)).to(dev)
    _, main, _, _ = P.expand_layout(dcb.cb, P.PLANES14, cls, inp.gain, sm, lv, (16, 4))
    recs = torch.from_numpy(main[:14 * pool].reshape(pool, 14)).to(dev)
    desc = P.planes14_desc(1, 24 * nb, (16, 4))
    reps = -(-nb // pool)
    d_codes = codes.reshape(-1).repeat(reps)[:nb].contiguous()
    got = torch.empty(desc.main_bytes, dtype=torch.uint8, device=dev)
    bad = torch.full((1,), 77, dtype=torch.int32, device=dev)
    _lib.transcode_planes14(desc, dcb.index.data_ptr(), d_codes.data_ptr(), got.data_ptr(),
                            bad.data_ptr())
    assert int(bad.item()) == 0
    whole = nb // pool
    body = got[:14 * pool * whole].view(whole, pool, 14)
    for i in range(0, whole, 8192):
        assert bool((body[i:i + 8192] == recs).all())
    rest = nb - whole * pool
    tail = got[14 * pool * whole:]
    assert torch.equal(tail[:14 * rest].view(rest, 14), recs[:rest])
    assert bool((tail[14 * rest:] == 0).all())


def test_scales_past_one_launch(dev):
    """65,541 rows of 65,536 blocks, more than 2^32: the storage order takes two
    launches.  Each tile's slots hold its rows' scales by column group, row and
    column."""
    M, nb, (C, R) = 65541, 65536, (16, 4)
    if torch.cuda.mem_get_info(dev)[0] < 40 << 30:
        pytest.skip("needs 40 GB of device memory")
    say(f"[scales] {M}x{24 * nb}")
    desc = P.planes14_desc(M, 24 * nb, (C, R))
    col = torch.arange(nb, device=dev, dtype=torch.int32)
    rows = torch.empty((M, nb), dtype=torch.int16, device=dev)
    for r0 in range(0, M, 4096):
        r = torch.arange(r0, min(M, r0 + 4096), device=dev, dtype=torch.int32)
        rows[r0:r0 + 4096] = (r[:, None] * 40503 + col * 30011 + (col >> 8)).to(torch.int16)
    out = torch.full((M * nb + 1,), 77, dtype=torch.int16, device=dev)
    _lib.layout_scales_device(desc, rows.data_ptr(), out.data_ptr())
    full = M // R * R
    got = out[:full * nb].view(full // R, nb // C, R, C)
    want = rows[:full].view(full // R, R, nb // C, C)
    for t in range(0, full // R, 1024):
        assert torch.equal(got[t:t + 1024], want[t:t + 1024].transpose(1, 2)), t
    assert torch.equal(out[full * nb:-1].view(nb // C, M - full, C),
                       rows[full:].view(M - full, nb // C, C).transpose(0, 1))
    assert int(out[-1]) == 77


@pytest.mark.parametrize("kind", ["stream", "handle", "default"])
def test_from_codes_on_another_stream(dev, dcb, kind):
    """With stream= other than the current one, and work ahead of the transcoder
    on both: the codes are read after the current stream has written them,
    invalid ones are counted, and the matrix is whole on return.  A stale or
    early count would fail the valid matrix or pass the invalid one."""
    say(f"[transcode] caller's stream: {kind}")
    M, K = 1024, 24 * 64
    inp = synth.make_gemv_inputs(M, K, seed=9, name="transcode-stream")
    cls, sm, lv = dcb.cb.fields_from_points(inp.z)
    codes = P.index_encode(dcb.cb, cls, inp.gain, sm, lv).view(np.int64)
    ref = P.LeechMatrix.from_fields(dcb, P.PLANES14, cls, inp.gain, sm, lv, inp.scale, dev)
    good = torch.from_numpy(codes).to(dev)
    wrong = good.clone()
    wrong[5, 7] = wrong[M - 1, 3] = 1 << 50
    work = torch.randn(4096, 4096, device=dev)
    side, outer = torch.cuda.Stream(dev), torch.cuda.Stream(dev)
    torch.cuda.synchronize()
    # "default": the current stream is another one, the caller's the default
    given = {"stream": side, "handle": side.cuda_stream, "default": torch.cuda.default_stream(dev)}
    with torch.cuda.stream(outer if kind == "default" else torch.cuda.current_stream(dev)):
        for turn in range(4):
            with torch.cuda.stream(torch.cuda.default_stream(dev) if kind == "default" else side):
                (work @ work).sum()
            live = torch.zeros_like(good)       # not codes of these points until the copy
            (work @ work).sum()
            live.copy_(wrong if turn % 2 else good)
            if turn % 2:
                with pytest.raises(P.LeechError, match="2 of"):
                    P.LeechMatrix.from_codes(dcb, live, inp.scale, stream=given[kind])
            else:
                mat = P.LeechMatrix.from_codes(dcb, live, inp.scale, stream=given[kind])
                assert torch.equal(mat.main, ref.main) and torch.equal(mat.scale, ref.scale)


def host_storage_index(desc):
    """Storage slot of block (r, j) in the wave-tile order (rows grouped in
    tiles of tile_rows, units of lane_cols columns, stored row by row)."""
    C = desc.lane_cols
    R = desc.tile_rows
    M, nb = desc.M, desc.nb

    def index(r, j):
        t, g = r // R, j // C
        rows = min(R, M - t * R)
        cols = min(C, nb - g * C)
        return t * R * nb + g * rows * C + (r % R) * cols + (j % C)
    return index
