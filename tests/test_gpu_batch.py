"""Batched GEMV (Planes14) through the C ABI.  With v_dot2 products
(BATCH_DOT2) every output vector is bit-identical to the single GEMV of its
activation; with the matrix-core products (BATCH_AUTO, every geometry) each
vector is within tolerance of the oracle's f64 product and of its single
GEMV, and bit-identical whatever the batch size and its position in the
batch.  Batches not a power of two, above 16, wide K (narrower chunks), every
geometry the matrix-core path takes (ragged tiles, lanes without a column),
strided activations and outputs."""
import os
import re
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2609_02652_amd as P  # noqa: E402
from paper_2609_02652_amd import synth  # noqa: E402
from oracle import decode as D  # noqa: E402

pytestmark = pytest.mark.gpu
CEN = (0.75, 1.25)


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


def activations(K, B, seed):
    return np.stack([synth.make_activation(K, seed=seed + b, name="batch") for b in range(B)])


def oracle_check(inp, rows, X, Y, bs):
    sub = synth.GemvInputs(len(rows), inp.K, inp.Kpad, inp.nb, inp.z[rows], inp.gain[rows],
                           inp.scale[rows], inp.x, inp.seed, inp.name)
    W = D.weights64_from_points(sub.z, sub.gain, sub.scale, CEN)
    for b in bs:
        e = D.errors(Y[b][rows], D.gemv64(W, X[b]), W, X[b])
        assert e["max_norm_err"] <= 2e-3 and e["max_abs_err"] <= 1e-5, (b, e)
    return W


def sample_rows(M):
    return np.arange(M) if M <= 1024 else np.sort(np.random.default_rng(M).choice(M, 256, False))


def build(dev, dcb, M, K, seed, geometry=None):
    inp = synth.make_gemv_inputs(M, K, seed=seed, name="batch")
    cls, sm, lv = dcb.cb.fields_from_points(inp.z)
    mat = P.LeechMatrix.from_fields(dcb, P.PLANES14, cls, inp.gain, sm, lv, inp.scale, dev,
                                    geometry=geometry)
    return inp, mat


def matrix_cores(mat, B):
    return B > 1


@pytest.fixture
def dot2_mode():
    P.set_batch_mode(P.BATCH_DOT2)
    yield
    P.set_batch_mode(P.BATCH_AUTO)


SHAPES = [(1, 24, 2), (65, 408, 3), (257, 792, 8), (768, 1536, 5), (4096, 4096, 11),
          (14337, 120, 4), (1024, 17408, 8), (300, 24 * 30, 1), (768, 1536, 21), (257, 792, 16)]


@pytest.mark.parametrize("M,K,B", SHAPES)
def test_dot2_batch_bit_identical_to_single(dev, dcb, dot2_mode, M, K, B):
    say(f"[batch dot2] {M}x{K} B={B}")
    inp, mat = build(dev, dcb, M, K, M + B)
    X = activations(K, B, seed=K)
    Xd = torch.from_numpy(X).to(dev)
    Y = mat.gemv_batch(Xd, centroids=CEN).cpu().numpy()
    for b in range(B):
        y1 = mat.gemv(Xd[b].contiguous(), centroids=CEN).cpu().numpy()
        assert np.array_equal(Y[b].view(np.uint32), y1.view(np.uint32)), f"vector {b}"
    oracle_check(inp, sample_rows(M), X, Y, (0, B - 1))


def check_auto(dev, mat, inp, X, Y):
    """Y from BATCH_AUTO: bit-identical to single GEMVs where the products are
    v_dot2; on the matrix cores within tolerance of the oracle and, row by
    row, within 2^-15 · Σ|w x| of the single GEMV.  The bound: a block's
    24-product dot of the decoded (subnormal) weights with an N(0,1) binary16
    activation errs by at most 119 (v_dot2) and 155 (matrix core) units of
    2^-24 · Σ|h x| over 512,000 measured dot products, so two paths differ by
    under 2^-15 · Σ|h x| a block; the blocks' f32 accumulation adds a few
    more units."""
    B = X.shape[0]
    Xd = torch.from_numpy(X).to(dev)
    rows = sample_rows(inp.M)
    if not matrix_cores(mat, B):
        for b in range(B):
            y1 = mat.gemv(Xd[b].contiguous(), centroids=CEN).cpu().numpy()
            assert np.array_equal(Y[b].view(np.uint32), y1.view(np.uint32)), f"vector {b}"
        oracle_check(inp, rows, X, Y, (0, B - 1))
        return
    W = oracle_check(inp, rows, X, Y, range(B))
    for b in (0, B - 1):
        y1 = mat.gemv(Xd[b].contiguous(), centroids=CEN).cpu().numpy()
        bound = 2.0 ** -15 * (np.abs(W) @ np.abs(X[b].astype(np.float64)))
        diff = np.abs(Y[b][rows].astype(np.float64) - y1[rows])
        assert (diff <= bound).all(), (b, float((diff / np.maximum(bound, 1e-300)).max()))


@pytest.mark.parametrize("M,K,B", SHAPES)
def test_batch_matches_oracle_and_single(dev, dcb, M, K, B):
    say(f"[batch] {M}x{K} B={B}")
    inp, mat = build(dev, dcb, M, K, M + B)
    say(f"[batch] geometry {mat.desc.lane_cols}x{mat.desc.tile_rows}, "
        f"matrix cores {matrix_cores(mat, B)}")
    X = activations(K, B, seed=K)
    Y = mat.gemv_batch(torch.from_numpy(X).to(dev), centroids=CEN).cpu().numpy()
    check_auto(dev, mat, inp, X, Y)


# lane placements of the matrix-core path: every lane_cols (1, 2, 3, 4, 8, 16),
# tile_rows from 4 to 64, lanes past the last column (R · C < 64), ragged last
# tiles (rows of a 4-lane block partly past the matrix) and last column groups
MX_GEOMETRIES = [((1, 64), 1000, 24 * 37), ((2, 32), 777, 24 * 41), ((4, 16), 301, 24 * 43),
                 ((3, 16), 333, 24 * 29), ((1, 16), 70, 24 * 11), ((1, 48), 100, 24 * 7),
                 ((2, 16), 50, 24 * 9), ((1, 32), 33, 24), ((4, 16), 4096, 4104),
                 ((2, 28), 1000, 24 * 45), ((2, 24), 301, 24 * 50), ((1, 20), 333, 24 * 13),
                 ((4, 12), 100, 24 * 23), ((1, 60), 777, 24 * 17), ((3, 12), 200, 24 * 31),
                 ((4, 4), 37, 24 * 9), ((3, 20), 301, 24 * 50), ((8, 8), 100, 24 * 37),
                 ((16, 4), 30, 24 * 70), ((8, 4), 66, 24 * 20), ((3, 20), 5120, 5136)]


@pytest.mark.parametrize("geo,M,K", MX_GEOMETRIES)
def test_matrix_core_geometries(dev, dcb, geo, M, K):
    inp, mat = build(dev, dcb, M, K, M + K, geometry=geo)
    assert (mat.desc.lane_cols, mat.desc.tile_rows) == geo
    for B in (2, 3, 5, 16, 17):
        say(f"[batch mx] {geo} {M}x{K} B={B}")
        X = activations(K, B, seed=K + B)
        Y = mat.gemv_batch(torch.from_numpy(X).to(dev), centroids=CEN).cpu().numpy()
        check_auto(dev, mat, inp, X, Y)


@pytest.mark.parametrize("geo,M,K", [((4, 16), 301, 24 * 43), ((2, 32), 777, 24 * 41),
                                     ((1, 64), 1000, 24 * 37), ((2, 28), 1000, 24 * 45),
                                     ((3, 20), 301, 24 * 50), ((8, 8), 100, 24 * 37)])
def test_matrix_core_bits_independent_of_batch(dev, dcb, geo, M, K):
    """One activation's y is the same bits alone in a 2-wide launch, in
    every position of 4-, 8- and 16-wide launches and in a trailing chunk."""
    inp, mat = build(dev, dcb, M, K, 3 * M + K, geometry=geo)
    X = activations(K, 17, seed=K)
    Xd = torch.from_numpy(X).to(dev)
    ref = mat.gemv_batch(Xd[:2], centroids=CEN).cpu().numpy()
    for B in (3, 4, 8, 16, 17):
        say(f"[batch bits] {geo} B={B}")
        Y = mat.gemv_batch(Xd[:B], centroids=CEN).cpu().numpy()
        assert np.array_equal(Y[:2].view(np.uint32), ref.view(np.uint32)), B
    full = mat.gemv_batch(Xd, centroids=CEN).cpu().numpy()
    for shift in (1, 5, 13, 16):
        say(f"[batch bits] {geo} shift {shift}")
        Y = mat.gemv_batch(torch.roll(Xd, shift, 0).contiguous(), centroids=CEN).cpu().numpy()
        assert np.array_equal(Y.view(np.uint32), np.roll(full, shift, 0).view(np.uint32)), shift


# the wide kernel's tiles of every lane_cols (by the batch, which sets the
# number of workgroups), with ragged tiles, row blocks and last column groups
TILE_CASES = [((1, 64), 333, 24 * 21, 1700), ((1, 64), 333, 24 * 21, 850), ((1, 48), 333, 24 * 9, 424),
              ((1, 64), 70, 24 * 3, 5), ((2, 32), 333, 24 * 23, 856), ((2, 28), 100, 24 * 17, 1300),
              ((2, 24), 100, 24 * 40, 9), ((3, 20), 333, 24 * 50, 860), ((3, 12), 70, 24 * 26, 1701),
              ((3, 20), 70, 24 * 49, 17), ((4, 16), 333, 24 * 39, 857), ((4, 16), 100, 24 * 33, 1281),
              ((4, 4), 333, 24 * 5, 240), ((4, 12), 17, 24 * 70, 33), ((8, 8), 333, 24 * 67, 465),
              ((8, 4), 100, 24 * 41, 641), ((8, 8), 9, 24 * 9, 6), ((16, 4), 333, 24 * 131, 240),
              ((16, 4), 30, 24 * 18, 19)]


@pytest.mark.parametrize("geo,M,K,B", TILE_CASES)
def test_wide_batch_tiles(dev, dcb, geo, M, K, B):
    """Every tile of the wide kernel, strided activations and outputs: the bits
    of the four-activation launches (which the tests above hold to the oracle
    and the single GEMV)."""
    say(f"[batch tiles] {geo} {M}x{K} B={B}")
    inp, mat = build(dev, dcb, M, K, M + B, geometry=geo)
    g = torch.Generator().manual_seed(B)
    X = torch.randn(B, inp.Kpad + 8, generator=g).half().to(dev)
    Y = torch.full((B, M + 1), -3.0, dtype=torch.float32, device=dev)
    mat.gemv_batch(X[:, :inp.Kpad], Y[:, :M], centroids=CEN)
    ref = torch.empty((B, M), dtype=torch.float32, device=dev)
    for b in range(0, B, 4):
        n = min(4, B - b)
        x = X[b:b + n, :inp.Kpad] if n > 1 else X[b - 1:b + 1, :inp.Kpad]
        ref[b:b + n] = mat.gemv_batch(x, centroids=CEN)[-n:]
    assert torch.equal(Y[:, :M].view(torch.int32), ref.view(torch.int32))
    assert torch.all(Y[:, M] == -3.0)


# (rows, activations, ring depth) of the wide kernel's tiles by lane_cols, widest
# first, as batch.hip's kTiles and its launch table
WIDE_TILES = {1: [(64, 64, 4), (64, 32, 4), (64, 16, 4), (32, 16, 4)],
              2: [(64, 32, 4), (32, 32, 4), (32, 16, 4)],
              3: [(64, 32, 3), (32, 32, 3), (32, 16, 3)],
              4: [(64, 32, 4), (32, 32, 4), (32, 16, 4), (16, 16, 4)],
              8: [(32, 32, 4), (32, 16, 4), (16, 16, 4)],
              16: [(32, 16, 8), (16, 16, 4)]}


def wide_tile(C, M, B):
    """batch.hip's choose_tile."""
    for tile in WIDE_TILES[C]:
        rw, nb = tile[:2]
        if (nb == 16 or 2 * B > nb) and -(-M // rw) * -(-B // nb) >= 160:
            break
    return tile


def plain_waves(geo, M, nb, tile):
    """(row block, wave) pairs whose steps take the steady loop of constant
    addresses (batch.hip's `plain` with two rings of steps and more), of all."""
    (C, R), (rw, _, D) = geo, tile
    sc, groups, plain, pairs = 64 // rw, -(-nb // C), 0, 0
    for row0 in range(0, M, rw):
        tile0 = row0 // R
        t_last = (min(row0 + rw, M) - 1 - tile0 * R) // R
        for wave in range(min(8, groups)):
            units = (groups - 1 - wave) // 8 + 1
            steps = -(-units * C // sc)
            assert steps >= 3 * D + 1, (geo, tile, wave, steps)
            pairs += 1
            plain += ((C % sc == 0 or sc % C == 0) and units * C % sc == 0
                      and (t_last == 0 or (tile0 + t_last + 1) * R <= M)
                      and (nb % C == 0 or (groups - 1) % 8 != wave))
    return plain, pairs


def test_wide_tiles_are_the_sources():
    """WIDE_TILES is what the library compiles."""
    with open(os.path.join(os.path.dirname(P.__file__), "csrc", "batch.hip")) as f:
        src = f.read()
    built = {tuple(map(int, t)) for t in re.findall(r"launch_tile<(\d+), (\d+), (\d+), (\d+), \d+>", src)}
    assert built == {(C, *t) for C, tiles in WIDE_TILES.items() for t in tiles}
    for C, tiles in re.findall(r"\{(\d+), \{([\d, ]+)\}\}", src[src.index("kTiles[] ="):]):
        order = [divmod(int(t), 100) for t in tiles.split(",") if int(t)]
        assert order == [t[:2] for t in WIDE_TILES[int(C)]], C


# per tile: geometry, blocks a row (three rings of steps and more on every
# wave), rows (full tiles and a ragged last one of an odd number of rows)
STEADY_CASES = [((1, 64), 107, 353, 0), ((1, 64), 107, 353, 1), ((1, 64), 107, 353, 2),
                ((1, 48), 211, 203, 3), ((2, 32), 117, 353, 0), ((2, 28), 117, 333, 0),
                ((2, 32), 213, 353, 1), ((2, 24), 214, 203, 2), ((3, 20), 104, 353, 0),
                ((3, 16), 104, 331, 0), ((3, 20), 176, 353, 1), ((3, 12), 176, 203, 2),
                ((4, 16), 139, 353, 0), ((4, 16), 235, 353, 1), ((4, 12), 236, 203, 2),
                ((4, 16), 427, 203, 3), ((8, 8), 279, 203, 0), ((8, 8), 280, 203, 1),
                ((8, 4), 471, 107, 2), ((16, 4), 559, 203, 0), ((16, 4), 560, 107, 1)]


@pytest.mark.parametrize("geo,nb,M,which", STEADY_CASES)
def test_wide_batch_steady_loop(dev, dcb, geo, nb, M, which):
    """Every tile of the wide kernel over rows long enough that each wave refills
    its ring of records at least twice: the steady loop of constant addresses
    (record parity included: odd units of one and three columns in the ragged
    tile), its hand-over to the general one, row blocks and waves that take the
    general one alone.  The bits of the four-activation launches."""
    tile = WIDE_TILES[geo[0]][which]
    B = next(b for b in range(9, 6000) if b % 16 in (3, 11) and wide_tile(geo[0], M, b) == tile)
    plain, pairs = plain_waves(geo, M, nb, tile)
    say(f"[batch steady] {geo} {M}x{24 * nb} B={B} tile {tile} plain {plain}/{pairs}")
    sc = 64 // tile[0]
    if geo[0] % sc == 0 or sc % geo[0] == 0:
        assert 0 < plain
    else:
        assert plain == 0
    inp, mat = build(dev, dcb, M, 24 * nb, nb, geometry=geo)
    g = torch.Generator().manual_seed(B)
    X = torch.randn(B, inp.Kpad, generator=g).half().to(dev)
    Y = torch.full((B, M + 1), -3.0, dtype=torch.float32, device=dev)
    mat.gemv_batch(X, Y[:, :M], centroids=CEN)
    ref = torch.empty((B, M), dtype=torch.float32, device=dev)
    for b in range(0, B, 4):
        b = min(b, B - 4)
        ref[b:b + 4] = mat.gemv_batch(X[b:b + 4], centroids=CEN)
    assert torch.equal(Y[:, :M].view(torch.int32), ref.view(torch.int32))
    assert torch.all(Y[:, M] == -3.0)


# both sides of the lines between narrow launches and the wide kernel: one launch
# of 8, two of 4, three of 2, single ones, by lane_cols
NARROW_CASES = [((16, 4), 199, (5, 8)), ((16, 4), 200, (5, 8)), ((16, 4), 699, (5, 8)),
                ((16, 4), 700, (5, 7, 8)), ((16, 4), 1001, (3, 4)), ((16, 4), 1399, (5, 6)),
                ((16, 4), 1400, (5, 6)), ((16, 4), 1536, (2, 4)), ((16, 4), 1537, (2, 3, 4, 5)),
                ((16, 4), 3019, (2, 4)), ((8, 8), 319, (6,)), ((8, 8), 320, (5, 6, 8)),
                ((8, 8), 869, (3,)), ((8, 8), 870, (3, 4)), ((8, 8), 1601, (2, 3)),
                ((3, 20), 119, (7,)), ((3, 20), 120, (5, 7, 8)), ((3, 20), 384, (8,)),
                ((3, 20), 386, (8,)), ((1, 64), 400, (5, 8)), ((4, 16), 385, (5, 8))]


@pytest.mark.parametrize("geo,nb,batches", NARROW_CASES)
def test_narrow_and_wide_batches(dev, dcb, geo, nb, batches):
    """A batch's bits do not depend on the kernel: those of a batch of 16, which
    is always the wide one's, with a ragged last tile, strided activations and
    outputs, and nothing written past an output row."""
    M = geo[1] + 5
    say(f"[narrow] {geo} {M}x{24 * nb} B={batches}")
    inp, mat = build(dev, dcb, M, 24 * nb, nb, geometry=geo)
    g = torch.Generator().manual_seed(nb)
    X = torch.randn(16, inp.Kpad + 8, generator=g).half().to(dev)[:, :inp.Kpad]
    want = mat.gemv_batch(X, centroids=CEN)
    for B in batches:
        Y = torch.full((B + 1, M + 3), -3.0, dtype=torch.float32, device=dev)
        mat.gemv_batch(X[:B], Y[:B, :M], centroids=CEN)
        assert torch.equal(Y[:B, :M].view(torch.int32), want[:B].view(torch.int32)), B
        assert bool((Y[:, M:] == -3.0).all()) and bool((Y[B] == -3.0).all())


@pytest.mark.parametrize("geo", [(1, 64), (2, 32), (3, 20), (4, 16), (8, 8), (16, 4)])
def test_batch_unused_centroid(dev, dcb, geo):
    """No block has gain bit 0, so its centroid does not matter, NaN included:
    batches of every kernel give the bits of a finite one, with columns to spare
    in the last group and waves without a unit."""
    C, R = geo
    M, nb = R + 5, 9 * C + max(1, C - 1)
    say(f"[batch centroid] {geo} {M}x{24 * nb}")
    inp = synth.make_gemv_inputs(M, 24 * nb, seed=5, name="batch-centroid")
    cls, sm, lv = dcb.cb.fields_from_points(inp.z)
    mat = P.LeechMatrix.from_fields(dcb, P.PLANES14, cls, np.ones_like(inp.gain), sm, lv,
                                    inp.scale, dev, geometry=geo)
    X = torch.from_numpy(activations(24 * nb, 33, seed=nb)).to(dev)
    for B in (2, 4, 5, 16, 33):
        want = mat.gemv_batch(X[:B], centroids=(1.0, 1.25))
        for unused in (float("nan"), float("inf"), 3e38):
            got = mat.gemv_batch(X[:B], centroids=(unused, 1.25))
            assert torch.equal(got.view(torch.int32), want.view(torch.int32)), (B, unused)


def test_batch_past_one_launch(dev, dcb):
    """One row and 2^24 + 37 activations: 8 · (2^20 + 3) workgroups of 512
    threads, more than the 2^32 threads of a launch, so the batch takes two.
    The same bits as in calls of 2^20 activations."""
    B = (1 << 24) + 37
    say(f"[batch] 1x24 B={B}")
    inp, mat = build(dev, dcb, 1, 24, 7, geometry=(16, 4))
    g = torch.Generator(device=dev).manual_seed(1)
    X = torch.randn(B, 24, generator=g, device=dev, dtype=torch.float16)
    Y = torch.full((B + 1, 1), -3.0, dtype=torch.float32, device=dev)
    mat.gemv_batch(X, Y[:B], centroids=CEN)
    for b0 in range(0, B, 1 << 20):
        part = mat.gemv_batch(X[b0:b0 + (1 << 20)], centroids=CEN)
        assert torch.equal(Y[b0:b0 + part.shape[0]].view(torch.int32), part.view(torch.int32)), b0
    assert float(Y[B]) == -3.0


def test_batch_mode_rejects_unknown(dev):
    with pytest.raises(P.LeechError):
        P.set_batch_mode(7)
    P.set_batch_mode(P.BATCH_AUTO)


def test_strided_activations_and_outputs(dev, dcb):
    M, K, B = 257, 792, 6
    inp = synth.make_gemv_inputs(M, K, seed=5, name="batch-stride")
    cls, sm, lv = dcb.cb.fields_from_points(inp.z)
    mat = P.LeechMatrix.from_fields(dcb, P.PLANES14, cls, inp.gain, sm, lv, inp.scale, dev)
    X = activations(K, B, seed=9)
    big = torch.zeros((B, inp.Kpad + 40), dtype=torch.float16, device=dev)
    big[:, :inp.Kpad] = torch.from_numpy(X).to(dev)
    Ybig = torch.full((B, M + 3), 123.0, dtype=torch.float32, device=dev)
    mat.gemv_batch(big[:, :inp.Kpad], Ybig[:, :M], centroids=CEN)
    Yc = mat.gemv_batch(torch.from_numpy(X).to(dev), centroids=CEN)
    assert torch.equal(Ybig[:, :M], Yc)
    assert torch.all(Ybig[:, M:] == 123.0)
