"""MEAN9 and the mean filter on the matrix-core tiles, at the sizes where they
can go wrong: rows of every alignment (nx mod 4, and volumes that start at
every byte of a word), volumes narrower and lower than a block of 16 and a
window of 32, one more and one less than a tile, both faces in one window, and
values whose digits reach both ends of their range.  Integer work: every byte
equals the oracle's."""
import numpy as np
import pytest

import oracle
from oracle import compare as ocmp
from paper_1807_03119_amd import _lib

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DTYPES = {"u8": (torch.uint8, np.uint8), "u16": (torch.uint16, np.uint16)}
# nx around 8, 16, 32, 64, 128 and 144 with every remainder mod 4; ny around 16 and 32
DIMS = [(1, 1, 3), (5, 2, 4), (7, 17, 3), (8, 15, 9), (15, 33, 5), (16, 16, 16), (17, 31, 6),
        (30, 9, 11), (33, 32, 5), (63, 18, 4), (64, 47, 3), (66, 16, 7), (127, 34, 3),
        (128, 33, 4), (131, 20, 5), (145, 49, 3), (270, 17, 2)]


def _values(dims, dtype, kind, seed):
    nx, ny, nz = dims
    rng = np.random.default_rng(seed)
    top = np.iinfo(dtype).max
    if kind == "uniform":
        return rng.integers(0, top + 1, (nz, ny, nx)).astype(dtype)
    if kind == "max":
        return np.full((nz, ny, nx), top, dtype)
    # only bytes 0x00, 0x7f, 0x80 and 0xff: the extremes of each biased digit
    b = np.array([0x00, 0x7F, 0x80, 0xFF])
    v = b[rng.integers(0, 4, (nz, ny, nx))]
    if dtype == np.uint16:
        v = v + 256 * b[rng.integers(0, 4, (nz, ny, nx))]
    return v.astype(dtype)


def _at_offset(vol, torch_dtype, lead):
    """The volume on the device, starting `lead` elements into an allocation."""
    n = vol.size
    buf = torch.zeros(n + lead + 64, dtype=torch_dtype, device="cuda")
    t = buf[lead:lead + n].view(vol.shape)
    t.copy_(torch.from_numpy(vol).cuda())
    return t


@pytest.mark.parametrize("r", [1, 2, 3, 4])
@pytest.mark.parametrize("dt", ["u8", "u16"])
def test_tile_edges_every_variant_and_alignment(dt, r):
    from paper_1807_03119_amd.api import Filter
    tdt, ndt = DTYPES[dt]
    code = _lib.LNF_U8 if dt == "u8" else _lib.LNF_U16
    f = Filter(_lib.LNF_MEAN9, 0)
    kinds = ["uniform", "digits", "max"]
    for i, dims in enumerate(DIMS):
        vol = _values(dims, ndt, kinds[i % 3], 7000 + i)
        want = oracle.filter_volume(vol, r)
        want_mean = ocmp.mean_filter(vol, r)
        for lead in range(4 // ndt().itemsize):
            dev = _at_offset(vol, tdt, lead)
            out = _at_offset(np.zeros_like(vol), tdt, (lead + i) % 3)
            for variant in range(-1, _lib.lnf_tile_variants(_lib.LNF_MEAN9, code, r)):
                for zs in (0, 3):
                    got = f(dev, r, out=out, variant=variant, zs=zs).cpu().numpy()
                    assert np.array_equal(got, want), (dims, lead, variant, zs)
            got = f.mean(dev, r, out=out).cpu().numpy()
            assert np.array_equal(got, want_mean), (dims, lead, "mean")
    f.close()


@pytest.mark.parametrize("nx", [2, 4, 6, 30, 34, 62, 66, 126, 130, 134, 258])
@pytest.mark.parametrize("r", [1, 3, 4])
def test_even_rows_of_uint16_start_at_words(r, nx):
    """nx mod 4 == 2: the last four outputs of a row overlap the ones before
    them, a tile with two columns left goes the other way; guard bytes stay."""
    from paper_1807_03119_amd.api import Filter
    f = Filter(_lib.LNF_MEAN9, 0)
    vol = _values((nx, 18, 5), np.uint16, "uniform", 40 + nx)
    want = oracle.filter_volume(vol, r)
    dev = _at_offset(vol, torch.uint16, 2)
    buf = torch.full((vol.size + 128,), 0xA5A5 - 65536, dtype=torch.int16, device="cuda")
    out = buf[64:64 + vol.size].view(torch.uint16).view(vol.shape)
    for variant in range(-1, _lib.lnf_tile_variants(_lib.LNF_MEAN9, _lib.LNF_U16, r)):
        f(dev, r, out=out, variant=variant)
        assert np.array_equal(out.cpu().numpy(), want), variant
    guard = torch.cat([buf[:64], buf[64 + vol.size:]]).cpu()
    assert bool((guard == 0xA5A5 - 65536).all())
    f.close()


def test_stores_stay_inside_the_volume():
    """No byte before or after an output of odd rows changes."""
    from paper_1807_03119_amd.api import Filter
    f = Filter(_lib.LNF_MEAN9, 0)
    for nx, ny, nz in ((67, 19, 5), (68, 33, 4), (3, 2, 2)):
        vol = torch.full((nz, ny, nx), 500, dtype=torch.uint16, device="cuda")
        buf = torch.full((nx * ny * nz + 512,), 7, dtype=torch.uint16, device="cuda")
        for lead in (255, 256):
            f(vol, 3, out=buf[lead:lead + vol.numel()].view(vol.shape))
            host = buf.cpu().numpy()
            assert (host[:lead] == 7).all() and (host[lead + vol.numel():] == 7).all()
            assert (host[lead:lead + vol.numel()] == 500).all()
            buf.view(torch.int16).fill_(7)
    f.close()


@pytest.mark.parametrize("r", [1, 2, 3, 4])
@pytest.mark.parametrize("dt", ["u8", "u16"])
def test_points_at_faces_and_alignments(dt, r):
    """Listed points on rows of every alignment: voxels whose rows end at a
    face, touch it, or leave the volume, points outside it, and lists that do
    not fill a group of sixteen points."""
    from paper_1807_03119_amd.api import Filter
    tdt, ndt = DTYPES[dt]
    for i, dims in enumerate([(4 * r + 1, 3, 2), (4 * r + 2, 9, 7), (4 * r + 7, 19, 5), (64, 11, 6), (3, 4, 5)]):
        nx, ny, nz = dims
        vol = _values(dims, ndt, "digits" if i % 2 else "uniform", 7100 + i)
        rng = np.random.default_rng(i)
        pts = [(x, int(rng.integers(0, ny)), int(rng.integers(0, nz))) for x in range(nx)]
        pts += [(x, y, z) for x in (0, nx - 1) for y in (0, ny - 1) for z in (0, nz - 1)]
        ok = np.array(pts)
        out = np.array([(-1, 0, 0), (0, ny, 0), (0, 0, -1), (nx, 0, 0)])
        for rule, orule in ((_lib.LNF_MEAN9, oracle.MEAN9), (_lib.LNF_MINVAR9, oracle.MINVAR9)):
            want = np.concatenate([oracle.filter_points(vol, r, ok, orule), np.full(4, 0xFFFFFFFF, np.uint32)])
            f = Filter(rule, 0)
            for lead in range(4 // ndt().itemsize):
                dev = _at_offset(vol, tdt, lead)
                for n in (len(want), 1, 17):
                    sel = np.random.default_rng(n).permutation(len(want))[:n]
                    xyz = torch.from_numpy(np.concatenate([ok, out])[sel].astype(np.int32)).cuda()
                    got = f.points(dev, r, xyz).cpu().numpy().view(np.uint32)
                    assert np.array_equal(got, want[sel]), (dims, rule, lead, n)
            f.close()


@pytest.mark.parametrize("r", [1, 2, 3, 4])
@pytest.mark.parametrize("dt", ["u8", "u16"])
def test_points_lists_of_every_lane_split(dt, r):
    """Lists around two points a SIMD, where a point's rows go from sixty-four
    lanes to sixteen, and one that does not fill its last wavefront."""
    from paper_1807_03119_amd.api import Filter
    tdt, ndt = DTYPES[dt]
    vol = _values((37, 21, 13), ndt, "uniform", 7300 + r)
    nz, ny, nx = vol.shape
    edge = 8 * torch.cuda.get_device_properties(0).multi_processor_count
    rng = np.random.default_rng(r)
    pts = np.stack([rng.integers(0, m, edge + 70) for m in (nx, ny, nz)], 1)
    pts[::97] = [nx, 0, 0]
    inside = pts[:, 0] < nx
    for rule, orule in ((_lib.LNF_MEAN9, oracle.MEAN9), (_lib.LNF_MINVAR9, oracle.MINVAR9)):
        want = np.full(len(pts), 0xFFFFFFFF, np.uint32)
        want[inside] = oracle.filter_points(vol, r, pts[inside], orule)
        with Filter(rule, 0) as f:
            for lead in range(4 // ndt().itemsize):
                dev = _at_offset(vol, tdt, lead)
                for n in (3, edge - 1, edge, edge + 1, edge + 70):
                    xyz = torch.from_numpy(pts[:n].astype(np.int32)).cuda()
                    got = f.points(dev, r, xyz).cpu().numpy().view(np.uint32)
                    assert np.array_equal(got, want[:n]), (rule, lead, n)


@pytest.mark.parametrize("r", [1, 2, 3, 4])
def test_points_of_a_uint16_volume_at_an_odd_address(r):
    """The C interface takes any byte address; a row's last voxel may then end
    past the words that hold a row of an even address."""
    vol = _values((4 * r + 9, 7, 6), np.uint16, "uniform", 7200 + r)
    nz, ny, nx = vol.shape
    pts = np.stack(np.meshgrid(np.arange(nx), [0, 3, ny - 1], [0, 2, nz - 1], indexing="ij"), -1).reshape(-1, 3)
    xyz = torch.from_numpy(pts.astype(np.int32)).cuda()
    out = torch.empty(len(pts), dtype=torch.int32, device="cuda")
    buf = torch.zeros(2 * vol.size + 64, dtype=torch.uint8, device="cuda")
    for rule, orule in ((_lib.LNF_MEAN9, oracle.MEAN9), (_lib.LNF_MINVAR9, oracle.MINVAR9)):
        want = oracle.filter_points(vol, r, pts, orule)
        h = _lib.lnf_create(rule, 0, 0)
        for lead in (1, 3):
            buf[lead:lead + 2 * vol.size].copy_(torch.from_numpy(vol.reshape(-1).view(np.uint8)).cuda())
            rc = _lib.lnf_filter_points(h, buf.data_ptr() + lead, (nx, ny, nz), _lib.LNF_U16, r, xyz,
                                        len(pts), out, None)
            assert rc == _lib.LNF_OK
            assert np.array_equal(out.cpu().numpy().view(np.uint32), want), (rule, lead)
        _lib.lnf_destroy(h)


# ---- Otsu's threshold and 2 sigma, found on the device ------------------------

def _levels(dt, kind):
    top = int(np.iinfo(dt).max)
    rng = np.random.default_rng(99)
    if kind == "one":
        v = np.full(60, top)
    elif kind == "two":
        v = np.array([0, top] * 30)
    elif kind == "ties":   # symmetric: several thresholds with the same criterion
        v = np.array([0, 1, top - 1, top] * 15)
    elif kind == "every":  # every level once
        v = np.arange(top + 1)
    elif kind == "chunks":  # at the edges of groups of 64 levels
        v = rng.choice(np.array([0, 63, 64, 65, 127, 128, 191, 192, top - 63, top]), 4096)
    else:                  # few levels, uneven counts
        v = rng.choice(rng.integers(0, top + 1, 7), 1001, p=[.5, .2, .1, .1, .05, .04, .01])
    return v.astype(dt)


@pytest.mark.parametrize("kind", ["one", "two", "ties", "every", "chunks", "few"])
@pytest.mark.parametrize("dt", [np.uint8, np.uint16])
def test_threshold_and_half_width_on_the_device(dt, kind):
    from oracle import otsu as ootsu
    from paper_1807_03119_amd.api import Filter
    v = _levels(dt, kind)
    vol = np.ascontiguousarray(v.reshape(1, 1, -1) if v.size % 4 else v.reshape(2, 2, -1))
    dev = torch.from_numpy(vol).cuda()
    counts = np.bincount(v, minlength=int(np.iinfo(dt).max) + 1)
    want_t = ootsu.otsu_threshold(counts)
    want_w = ocmp.sigma_half_width(vol)
    for rule, orule in ((_lib.LNF_MEAN9, oracle.MEAN9), (_lib.LNF_MINVAR9, oracle.MINVAR9)):
        f = Filter(rule, 0)
        out, t = f.filter_otsu(dev, 1)
        assert t == want_t
        assert np.array_equal(out.cpu().numpy(), oracle.filter_volume(vol, 1, orule, t))
        out, w = f.sigma(dev, 1)
        assert w == want_w
        assert np.array_equal(out.cpu().numpy(), ocmp.sigma_filter(vol, 1))
        f.close()


def test_otsu_calls_in_flight_on_several_streams():
    """More calls in flight than the context keeps threshold slots: each filter
    is gated at its own volume's threshold."""
    from oracle import otsu as ootsu
    from paper_1807_03119_amd.api import Filter
    f = Filter(_lib.LNF_MEAN9, 0)
    rng = np.random.default_rng(5)
    vols = [(rng.integers(0, 2, (24, 40, 50)) * (k + 1) * 900 + 100 * k).astype(np.uint16) for k in range(24)]
    devs = [torch.from_numpy(v).cuda() for v in vols]
    outs = [torch.empty_like(d) for d in devs]
    streams = [torch.cuda.Stream() for _ in range(3)]
    torch.cuda.synchronize()
    ts = []
    for k, d in enumerate(devs):
        with torch.cuda.stream(streams[k % 3]):
            ts.append(f.filter_otsu(d, 2, out=outs[k])[1])
    torch.cuda.synchronize()
    for v, o, t in zip(vols, outs, ts):
        assert t == ootsu.otsu_threshold(np.bincount(v.ravel(), minlength=65536))
        assert np.array_equal(o.cpu().numpy(), oracle.filter_volume(v, 2, oracle.MEAN9, t))
    f.close()


@pytest.mark.parametrize("lead", range(8))
@pytest.mark.parametrize("n", [1, 7, 8, 15, 16385, 65537])
def test_histogram_of_volumes_that_start_anywhere(n, lead):
    """Voxels before the first 16-byte vector, the vectors, and what is left."""
    from paper_1807_03119_amd.api import Filter
    vol = _values((n, 1, 1), np.uint16, "uniform", 60 + n)
    with Filter(_lib.LNF_MEAN9, 0) as f:
        got = f.histogram(_at_offset(vol, torch.uint16, lead)).cpu().numpy()
    assert np.array_equal(got, np.bincount(vol.ravel(), minlength=65536))


@pytest.mark.parametrize("value", [0, 1, 65534, 65535])
def test_histogram_counts_do_not_carry_between_the_halves_of_a_word(value):
    """One value over several chunks of every workgroup, ends on both sides."""
    from paper_1807_03119_amd.api import Filter
    n = 40_000_013
    buf = torch.zeros(n + 16, dtype=torch.int16, device="cuda")
    buf.fill_(value if value < 32768 else value - 65536)
    vol = buf[3:3 + n].view(torch.uint16).view(1, 1, n)
    with Filter(_lib.LNF_MEAN9, 0) as f:
        got = f.histogram(vol).cpu()
    want = torch.zeros(65536, dtype=torch.int64)
    want[value] = n
    assert torch.equal(got, want)


@pytest.mark.parametrize("rule", [_lib.LNF_MEAN9, _lib.LNF_MINVAR9])
def test_strips_deeper_than_the_volume(rule):
    """Any depth is accepted; one beyond the volume is one strip."""
    from paper_1807_03119_amd.api import Filter
    vol = _values((1024, 520, 2), np.uint8, "uniform", 77)
    dev = torch.from_numpy(vol).cuda()
    with Filter(rule, 0) as f:
        want = f(dev, 1, zs=2).cpu().numpy()
        for zs in (3, 2 ** 31 - 2, 2 ** 31 - 1):
            for variant in (-1, 0, 1):
                out = torch.zeros_like(dev)
                assert np.array_equal(f(dev, 1, out=out, variant=variant, zs=zs).cpu().numpy(), want), (zs, variant)


# ---- planes just below 4 GiB ---------------------------------------------------

def _mean_at(vol, r, pts):
    """The mean filter at listed voxels, from its definition."""
    nz, ny, nx = vol.shape
    off = np.arange(-r, r + 1)
    x, y, z = (np.clip(pts[:, k, None] + off, 0, n - 1) for k, n in enumerate((nx, ny, nz)))
    cube = vol[z[:, :, None, None], y[:, None, :, None], x[:, None, None, :]].astype(np.int64)
    n = (2 * r + 1) ** 3
    return ((2 * cube.sum((1, 2, 3)) + n) // (2 * n)).astype(np.uint32)


@pytest.mark.parametrize("dims,r", [((65534, 32769, 1), 1),     # 2^32 - 4 bytes, rows are whole words
                                    ((42966, 49981, 1), 3),     # 2^32 - 4 bytes, nx mod 4 == 2
                                    ((2699, 795659, 1), 4),     # 2^32 - 14 bytes, odd rows
                                    ((22605091, 95, 1), 2)])    # 2^32 - 6 bytes, few long rows
def test_uint16_planes_up_to_four_gigabytes(dims, r):
    """Planes whose last voxels lie within a few bytes of 4 GiB: the values at
    random voxels, at all four edges and in the last voxels of the plane, for
    MEAN9 alone and in a batch and for the mean filter."""
    from paper_1807_03119_amd.api import Filter
    nx, ny, nz = dims
    gen = torch.Generator(device="cuda").manual_seed(31)
    dev = torch.empty((nz, ny, nx), dtype=torch.int16, device="cuda").random_(-32768, 32768, generator=gen)
    host = dev.cpu().numpy().view(np.uint16)
    rng = np.random.default_rng(17)
    ex = np.array([0, 1, nx // 2, nx - 2, nx - 1])
    ey = np.array([0, 1, ny // 2, ny - 2, ny - 1])
    last = np.arange(nx * ny - 600, nx * ny)
    pts = np.concatenate([
        np.stack([rng.integers(0, nx, 2000), rng.integers(0, ny, 2000)], 1),
        np.stack([ex[rng.integers(0, 5, 600)], rng.integers(0, ny, 600)], 1),
        np.stack([rng.integers(0, nx, 600), ey[rng.integers(0, 5, 600)]], 1),
        np.stack([last % nx, last // nx], 1)])
    pts = np.concatenate([pts, np.zeros((len(pts), 1), pts.dtype)], 1)
    at = torch.from_numpy(pts[:, 1].astype(np.int64) * nx + pts[:, 0]).cuda()
    out = torch.empty_like(dev)

    def taken():
        return out.view(-1)[at].cpu().numpy().view(np.uint16).astype(np.uint32)
    vol, res = dev.view(torch.uint16), out.view(torch.uint16)
    want, want_mean = oracle.filter_points(host, r, pts, oracle.MEAN9), _mean_at(host, r, pts)
    with Filter(_lib.LNF_MEAN9, 0) as f:
        for name, call, w in (("filter", lambda: f(vol, r, out=res), want),
                              ("batch", lambda: f.batch([(vol, res, r)]), want),
                              ("mean", lambda: f.mean(vol, r, out=res), want_mean)):
            out.fill_(0)
            call()
            assert np.array_equal(taken(), w), (dims, r, name)
