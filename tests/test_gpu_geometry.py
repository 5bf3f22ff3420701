"""GPU parity across tile geometries (lane_cols × tile_rows) and row groups
that share a tile, through the C ABI.

* Geometries of every lane_cols the kernels serve, the library's choices on
  the workload shapes among them (3 × 20, 4 × 16, 2 × 32, 1 × 64, 8 × 8, ...),
  plus small ones, on a matrix with a ragged last tile and a ragged last column group:
  each layout decodes bit-exactly to the drawn points, all four layouts (and
  both exception decoders) give bit-identical y, and y is within the GEMV
  tolerance of the oracle's f64 matvec on every row.
* The batched and rotated entry points on 3 × 20, 2 × 24 and 1 × 60 give
  the single GEMV's bits (batches: in the v_dot2 mode; on the matrix cores,
  within the dot units' rounding) and the two-call bits.
* Row groups whose boundaries fall inside tiles (each such tile holds rows of
  two groups, every lane reading its own row's centroids): every row matches
  the oracle with its own group's centroids, in every layout, bit-identical
  across layouts; the same launch rotated in the prologue gives the two-call
  bits.
"""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2609_02652_amd as P  # noqa: E402
from paper_2609_02652_amd import _lib, synth  # noqa: E402
from oracle import decode as D  # noqa: E402

pytestmark = pytest.mark.gpu

TOL_NORM = 2e-3
TOL_PAPER = 1e-5
CEN = (0.75, 1.25)
# (lane_cols, tile_rows)
GEOMETRIES = [(3, 20), (3, 12), (3, 4), (2, 28), (2, 24), (2, 12), (1, 60), (1, 56), (1, 44),
              (1, 4), (4, 12), (8, 8), (16, 4), (4, 16)]


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


@pytest.fixture(scope="module")
def ragged():
    """203 rows (ragged last tile in every geometry here) × 37 blocks (ragged
    last column group for lane_cols 2, 3, 4, 8, 16)."""
    return synth.make_gemv_inputs(203, 24 * 37 - 5, seed=31, name="geometry")


@pytest.mark.parametrize("geo", GEOMETRIES, ids=[f"{c}x{r}" for c, r in GEOMETRIES])
def test_geometry_all_layouts(dev, dcb, ragged, geo):
    inp = ragged
    say(f"[geometry] {geo} {inp.M}x{inp.K}")
    cls, sm, lv = dcb.cb.fields_from_points(inp.z)
    x = torch.from_numpy(inp.x).to(dev)
    W = D.weights64_from_points(inp.z, inp.gain, inp.scale, CEN)
    y64 = D.gemv64(W, inp.x)
    ys = {}
    for name, layout in P.LAYOUTS.items():
        mat = P.LeechMatrix.from_fields(dcb, layout, cls, inp.gain, sm, lv, inp.scale, dev,
                                        geometry=geo)
        assert (mat.desc.lane_cols, mat.desc.tile_rows) == geo
        z, c, g = mat.decode()
        assert np.array_equal(z.cpu().numpy(), inp.z), name
        assert np.array_equal(c.cpu().numpy().astype(np.uint16), cls), name
        assert np.array_equal(g.cpu().numpy(), inp.gain), name
        modes = (P.EXC_HOISTED, P.EXC_INLINE) if name in ("planes12x", "golay70") else (None,)
        for mode in modes:
            if mode is not None:
                P.set_exception_mode(mode)
            try:
                ys[(name, mode)] = mat.gemv(x, centroids=CEN).cpu().numpy()
            finally:
                P.set_exception_mode(P.EXC_HOISTED)
    ref = ys[("planes14", None)]
    for key, y in ys.items():
        assert np.array_equal(y.view(np.uint32), ref.view(np.uint32)), key
    e = D.errors(ref, y64, W, inp.x)
    say(f"    errors {e}")
    assert e["max_norm_err"] <= TOL_NORM and e["max_abs_err"] <= TOL_PAPER, e


@pytest.mark.parametrize("geo", [(3, 20), (2, 24), (1, 60)], ids=["3x20", "2x24", "1x60"])
def test_geometry_batched_and_rotated(dev, dcb, geo):
    M, K = 301, 24 * 50
    inp = synth.make_gemv_inputs(M, K, seed=32, name="geometry-batch")
    cls, sm, lv = dcb.cb.fields_from_points(inp.z)
    mat = P.LeechMatrix.from_fields(dcb, P.PLANES14, cls, inp.gain, sm, lv, inp.scale, dev,
                                    geometry=geo)
    X = np.stack([synth.make_activation(K, seed=40 + b, name="geometry-batch") for b in range(5)])
    Xt = torch.from_numpy(X).to(dev)
    Y = mat.gemv_batch(Xt, centroids=CEN).cpu().numpy()
    P.set_batch_mode(P.BATCH_DOT2)
    try:
        Yd = mat.gemv_batch(Xt, centroids=CEN).cpu().numpy()
    finally:
        P.set_batch_mode(P.BATCH_AUTO)
    W = D.weights64_from_points(inp.z, inp.gain, inp.scale, CEN)
    for b in range(5):
        y1 = mat.gemv(Xt[b].contiguous(), centroids=CEN).cpu().numpy()
        assert np.array_equal(Yd[b].view(np.uint32), y1.view(np.uint32)), b
        # matrix-core products: within the dot units' rounding (2^-15 · Σ|w x|)
        bound = 2.0 ** -15 * (np.abs(W) @ np.abs(X[b].astype(np.float64)))
        assert (np.abs(Y[b].astype(np.float64) - y1) <= bound).all(), b
    raw = Xt[0, :K].contiguous()
    s = torch.from_numpy(synth.make_signs(K, seed=3, name="geometry-batch")).to(dev)
    y_rot = mat.gemv_rotated(raw, s, group_centroids=(CEN,)).cpu().numpy()
    y_two = mat.gemv(P.rotate_x(raw, s, inp.Kpad), centroids=CEN).cpu().numpy()
    assert np.array_equal(y_rot.view(np.uint32), y_two.view(np.uint32))


# (group rows, geometry): boundaries inside tiles, on tile starts, and a group
# shorter than a tile that starts on a tile boundary
STRADDLE = [([100, 37, 90], (3, 20)), ([4096 - 8, 8 + 1024, 1024], (2, 24)),
            ([13, 51, 64, 7], (1, 64)), ([24, 10, 30], (4, 12))]


@pytest.mark.parametrize("case", range(len(STRADDLE)))
def test_groups_sharing_tiles(dev, dcb, case):
    parts, geo = STRADDLE[case]
    K = 24 * 23
    ins = [synth.make_gemv_inputs(M, K, seed=600 + 10 * case + i, name=f"straddle{i}")
           for i, M in enumerate(parts)]
    cens = [(0.75, 1.25), (0.9, 1.1), (1.3, 0.6), (1.05, 0.85)][:len(parts)]
    z = np.concatenate([i.z for i in ins])
    gain = np.concatenate([i.gain for i in ins])
    scale = np.concatenate([i.scale for i in ins])
    x = ins[0].x
    cls, sm, lv = dcb.cb.fields_from_points(z)
    xt = torch.from_numpy(x).to(dev)
    ref = None
    for name, layout in P.LAYOUTS.items():
        say(f"[groups] {parts} geometry {geo} {name}")
        mat = P.LeechMatrix.from_fields(dcb, layout, cls, gain, sm, lv, scale, dev, geometry=geo)
        y = mat.gemv_grouped(xt, parts, cens).cpu().numpy()
        r0 = 0
        for inp, c in zip(ins, cens):
            W = D.weights64_from_points(inp.z, inp.gain, inp.scale, c)
            e = D.errors(y[r0:r0 + inp.M], D.gemv64(W, x), W, x)
            assert e["max_norm_err"] <= TOL_NORM and e["max_abs_err"] <= TOL_PAPER, (name, e)
            r0 += inp.M
        if ref is None:
            ref = y
        if name == "planes14":
            raw = xt[:K].contiguous()
            y_rot = mat.gemv_rotated(raw, None, parts, cens).cpu().numpy()
            y_two = mat.gemv_grouped(P.rotate_x(raw, None, mat.Kpad), parts, cens).cpu().numpy()
            assert np.array_equal(y_rot.view(np.uint32), y_two.view(np.uint32))
        assert np.array_equal(y.view(np.uint32), ref.view(np.uint32)), name


@pytest.mark.parametrize("step", [-1, 0, 1])
@pytest.mark.parametrize("geo", [(1, 64), (3, 20), (16, 4)], ids=["1x64", "3x20", "16x4"])
def test_decode_runs(dev, dcb, geo, step):
    """Whole-matrix decode where a row has one block fewer than a workgroup's
    eight units, just as many, and one more; z at an address that is a multiple
    of 4 only, and each output on its own.  Nothing past an output is written."""
    C, R = geo
    M, nb = R + 3, 8 * C + step
    say(f"[decode runs] {geo} {M}x{24 * nb}")
    inp = synth.make_gemv_inputs(M, 24 * nb, seed=33, name="decode-runs")
    cls, sm, lv = dcb.cb.fields_from_points(inp.z)
    mat = P.LeechMatrix.from_fields(dcb, P.PLANES14, cls, inp.gain, sm, lv, inp.scale, dev,
                                    geometry=geo)
    n = M * nb
    z = torch.full((24 * n + 8,), 99, dtype=torch.int8, device=dev)
    c = torch.full((n + 1,), 999, dtype=torch.int16, device=dev)
    g = torch.full((n + 1,), 9, dtype=torch.uint8, device=dev)
    for zp, cp, gp in ((z.data_ptr() + 4, 0, 0), (0, c.data_ptr(), 0), (0, 0, g.data_ptr())):
        _lib.decode_blocks(mat.desc, mat.main.data_ptr(), 0, 0, dcb.table.data_ptr(), 0, zp, cp, gp,
                           torch.cuda.current_stream().cuda_stream)
    z, c, g = z.cpu().numpy(), c.cpu().numpy(), g.cpu().numpy()
    assert np.array_equal(z[4:-4].reshape(M, nb, 24), inp.z)
    assert (z[:4] == 99).all() and (z[-4:] == 99).all()
    assert np.array_equal(c[:-1].reshape(M, nb), cls) and c[-1] == 999
    assert np.array_equal(g[:-1].reshape(M, nb), inp.gain) and g[-1] == 9


@pytest.mark.parametrize("geo,step", [((1, 64), -1), ((1, 64), 1), ((3, 20), -1), ((3, 20), 1),
                                      ((4, 16), 0), ((16, 4), -1), ((16, 4), 1)])
@pytest.mark.parametrize("layout", [P.SLOT32, P.PLANES14, P.PLANES12X, P.GOLAY70])
def test_decode_both_kernels(dev, dcb, layout, geo, step):
    """Decode on both sides of the block count that chooses the kernel:
    rows of one block fewer than a workgroup's eight units, as many and one more,
    a ragged last tile, z at an address that is a multiple of 4 only, nothing
    written past an output."""
    (C, R), pool = geo, 4099
    nb = 8 * C + step
    inp = synth.make_gemv_inputs(pool, 24, seed=3, name="decode-both")
    cls, sm, lv = dcb.cb.fields_from_points(inp.z[:, 0])
    line = {1: 1200, 16: 768}.get(C, 640) * 1024
    over = -(-line // nb)
    for M in ((line - 1) // nb, over + (over % R == 0)):
        say(f"[decode both] layout {layout} {geo} {M}x{24 * nb}")
        at = np.random.default_rng(nb).integers(0, pool, (M, nb))
        gain = inp.gain[at, 0]
        mat = P.LeechMatrix.from_fields(dcb, layout, cls[at], gain, sm[at], lv[at],
                                        np.ones((M, nb), np.float16), dev, geometry=geo)
        n = M * nb
        z = torch.full((24 * n + 8,), 99, dtype=torch.int8, device=dev)
        c = torch.full((n + 1,), 999, dtype=torch.int16, device=dev)
        g = torch.full((n + 1,), 9, dtype=torch.uint8, device=dev)
        m, s0, s1 = mat._ptrs()
        _lib.decode_blocks(mat.desc, m, s0, s1, dcb.table.data_ptr(), dcb.golay_gen.data_ptr(),
                           z.data_ptr() + 4, c.data_ptr(), g.data_ptr(),
                           torch.cuda.current_stream().cuda_stream)
        where = torch.from_numpy(at.reshape(-1)).to(dev)
        assert torch.equal(z[4:-4].view(n, 24), torch.from_numpy(inp.z[:, 0]).to(dev)[where])
        assert torch.equal(c[:-1], torch.from_numpy(cls.astype(np.int16)).to(dev)[where])
        assert torch.equal(g[:-1], torch.from_numpy(inp.gain[:, 0].copy()).to(dev)[where])
        assert bool((z[:4] == 99).all()) and bool((z[-4:] == 99).all())
        assert int(c[-1]) == 999 and int(g[-1]) == 9


def test_decode_past_one_launch(dev, dcb):
    """2^26 + 5 rows of one block in tiles of four: 2^24 + 2 workgroups of 256
    threads, more than the 2^32 threads of a launch, so the decode takes two.
    With one column the stream is in row order: the records of a repeated pool."""
    M, pool = (1 << 26) + 5, 4099
    say(f"[decode] {M}x24")
    inp = synth.make_gemv_inputs(pool, 24, seed=3, name="decode-long")
    cls, sm, lv = dcb.cb.fields_from_points(inp.z)
    _, main, _, _ = P.expand_layout(dcb.cb, P.PLANES14, cls, inp.gain, sm, lv, (16, 4))
    desc = P.planes14_desc(M, 24, (16, 4))
    rows = torch.arange(M, device=dev) % pool
    recs = torch.from_numpy(main[:14 * pool].reshape(pool, 14)).to(dev)
    stream = torch.zeros(desc.main_bytes, dtype=torch.uint8, device=dev)
    stream[:14 * M].view(M, 14).copy_(recs[rows])
    empty = torch.empty(0, dtype=torch.uint8, device=dev)
    z, c, g = P.LeechMatrix(desc, stream, empty, empty, None, dcb).decode()
    for got, want in ((z[:, 0], inp.z[:, 0]), (c[:, 0], cls[:, 0].astype(np.int16)),
                      (g[:, 0], inp.gain[:, 0])):
        assert torch.equal(got, torch.from_numpy(np.ascontiguousarray(want)).to(dev)[rows])
