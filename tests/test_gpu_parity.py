"""Parity of the HIP path (through the C ABI) with the FP64 CPU oracle.

Bars: Morton codes, level sizes, occupancy bytes, header fields and decoded positions
bit-exact; FP32 coefficients within 1e-5 of the per-channel maximum of the FP64 ones; quantized
coefficients equal to the oracle's except at rounding ties (at most 1e-4 of them, off by one,
each within the FP32 error of a decision boundary), and equal to the decision rule applied to
the GPU's own coefficients; attributes decoded by the GPU from the oracle's stream within 1e-5
of the per-channel maximum of the oracle's FP64 decode of the same stream.
"""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2606_05650_amd import gsc, synth
from gpucheck import REL_TOL, _dev, gpu_encode, roundtrip

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


GROUPED = synth.quant_steps(synth.STEPS_GROUPED)
UNIFORM = synth.quant_steps(synth.STEPS_UNIFORM_64)


@pytest.mark.parametrize("n,J,seed", [
    (100_000, 10, 1),      # the 100K-Gaussian depth-10 workload
    (20_000, 8, 2),
    (5_000, 12, 3),
    (700, 21, 4),          # deepest octree: 63-bit codes, level 63
    (4097, 9, 5),          # one past a sort tile
    (2049, 7, 6),          # one past an occupancy tile
    (513, 11, 7),          # one past a transform tile
    (1, 5, 8),
    (2, 1, 9),
])
def test_frame_roundtrip(n, J, seed):
    pos, attr = synth.make_frame(n, seed=seed)
    roundtrip(pos, attr, J, UNIFORM if J == 10 else GROUPED)


@pytest.mark.parametrize("n,J", [
    (16 * 2048, 12),        # 16 sort tiles of 2048 keys: exactly one look-back group
    (16 * 2048 + 1, 10),    # 17 tiles: a second group of one tile (8-bit digits)
    (33 * 2048 + 5, 12),    # 34 tiles: two full groups and a partial one
    (1 << 18, 11),          # 128 tiles: the largest frame on 2048-key tiles, eight groups
    ((1 << 18) + 1, 12),    # 65 tiles of 4096 keys: four groups and one tile
])
def test_sort_lookback_groups(n, J):
    """The sort's two-level look-back (groups of 16 tiles, group totals summed at publication)
    at group boundaries: the sorted order bit-exact against the oracle's stable sort, and the
    whole round trip."""
    assert gsc.tune_get(J, n) == gsc.sort_default_variant(n)
    pos, attr = synth.make_frame(n, seed=n % 97)
    roundtrip(pos, attr, J, GROUPED)


def test_deep_uniform_frame_many_levels():
    """Uniform points at depth 21 (63-bit codes): every 512-entry tile leaves entries open, and
    two upper tiling levels carry entries (about 3600 and 90 at 200K), which the persistent
    upper-level launches take in order through their phase flags."""
    rng = np.random.default_rng(21)
    n = 200_000
    pos = rng.random((n, 3), dtype=np.float32)
    attr = synth.sample_attributes(rng, n)
    roundtrip(pos, attr, 21, GROUPED)


@pytest.mark.parametrize("C", [1, 3, 5, 64])
def test_channel_counts(C):
    pos, _ = synth.make_frame(3000, seed=10 + C)
    rng = np.random.default_rng(C)
    attr = rng.normal(0, 1, size=(3000, C)).astype(np.float32)
    roundtrip(pos, attr, 8, np.full(C, 1 / 32, np.float32))


def test_duplicates_merge():
    pos, attr = synth.make_duplicates_frame(30_000, seed=11, grid=16)
    roundtrip(pos, attr, 6, GROUPED)   # 4096 sites: ~7 Gaussians per voxel
    roundtrip(pos, attr, 3, GROUPED)   # 512 voxels hold everything


def test_degenerate_frames():
    C = 56
    rng = np.random.default_rng(12)
    attr = synth.sample_attributes(rng, 100)
    roundtrip(np.full((100, 3), 0.25, np.float32), attr, 9, GROUPED)   # zero extent
    roundtrip(np.zeros((0, 3), np.float32), np.zeros((0, C), np.float32), 9, GROUPED)
    pos, attr = synth.make_frame(5000, seed=13)
    roundtrip(pos * 2 - 0.5, attr, 9, GROUPED, bbox=(np.zeros(3), 1 / 512))  # clamped points


def test_quantizer_variants():
    pos, attr = synth.make_frame(20_000, seed=14)
    odd = np.linspace(0.011, 0.3, 56).astype(np.float32)   # steps that are not powers of two
    roundtrip(pos, attr, 9, odd, tau=0.5)
    roundtrip(pos, attr, 9, GROUPED, tau=0.25)
    roundtrip(pos, attr, 9, GROUPED, tau=0.0)


@pytest.mark.slow
def test_frame_1M_depth12_full():
    pos, attr = synth.make_frame(1_000_000, seed=2)
    roundtrip(pos, attr, 12, GROUPED)


@pytest.mark.slow
@pytest.mark.parametrize("flags", [0, gsc.FLAG_FP64_WEIGHTS])
def test_frame_4M_depth14(flags):
    """The 4M-Gaussian frame at depth 14 (42-bit codes): codes, the sorted order, the voxel
    map, every occupancy byte, positions and coefficients against the oracle, with the FP32 and
    the FP64 computation of the butterfly rotations. Prints the tiling levels used."""
    pos, attr = synth.make_frame(4_000_000, seed=5)
    g, ref = roundtrip(pos, attr, 14, GROUPED, flags=flags)
    info = g["enc"].host_info()
    scale = np.abs(ref["Y"]).max(axis=0)
    rel = (np.abs(g["Y"] - ref["Y"]).max(axis=0) / scale).max()
    print(f"4M/J14 flags={flags}: Nv={g['nv']} tiling levels={int(info[4])} "
          f"max relative coefficient error {rel:.3g}", flush=True)
    assert int(info[4]) >= 2


def test_fp64_rotation_flag():
    """GSC_FLAG_FP64_WEIGHTS: recorded in the header, followed by the decoder, same bars."""
    pos, attr = synth.make_frame(30_000, seed=31)
    roundtrip(pos, attr, 11, GROUPED, flags=gsc.FLAG_FP64_WEIGHTS)


def test_corrupt_streams_are_rejected():
    dev = _dev()
    pos, attr = synth.make_frame(3000, seed=15)
    g = gpu_encode(pos, attr, 7, GROUPED)
    nv = g["nv"]

    def dec(blob, J=7):
        t = torch.from_numpy(blob.copy()).to(dev)
        d = gsc.decode_frame(t, J, 56, nv)
        torch.cuda.synchronize()
        return int(d.info[0].item())

    assert dec(g["blob"]) == 0
    bad = g["blob"].copy()
    bad[1024 + 5] = 0                       # a node without children
    assert dec(bad) == 5
    bad = g["blob"].copy()
    bad[1024 + 1] = 0xFF if bad[1024 + 1] != 0xFF else 0x01   # child count changes
    assert dec(bad) == 5
    bad = g["blob"].copy()
    bad[:4] = 0                             # magic
    assert dec(bad) == 5
    assert dec(g["blob"], J=8) == 5         # depth mismatch
    assert dec(g["blob"][:2000]) == 5       # truncated
    assert dec(g["blob"][:600]) == 5        # shorter than the header
    assert dec(g["blob"][:16]) == 5         # shorter than the header's counts


def test_nonfinite_positions_are_rejected():
    """A position that is not finite makes an encode that finds the bounding cube fail with
    GSC_ERR_INVALID_ARG (device status), whether it lies in the float4 batches or in the last
    coordinates that do not fill one (3n mod 4 of them); a finite frame then encodes as usual."""
    dev = _dev()
    for n, row, axis in [(5000, 1234, 1), (5001, 5000, 2)]:
        pos, attr = synth.make_frame(n, seed=21)
        p = gsc.make_params(10, attr.shape[1], GROUPED)
        for bad_val in (np.nan, np.inf, -np.inf):
            bad = pos.copy()
            bad[row, axis] = bad_val
            e = gsc.encode_frame(torch.from_numpy(bad).to(dev), torch.from_numpy(attr).to(dev), p)
            torch.cuda.synchronize()
            assert int(e.host_info()[0]) == 1, (n, bad_val)
    roundtrip(*synth.make_frame(5001, seed=21), 10, GROUPED)


def test_transform_entry_points():
    dev = _dev()
    rng = np.random.default_rng(16)
    for n, J in [(3000, 7), (50_000, 12)]:
        pos, _ = synth.make_frame(n, seed=17)
        vox, _, _ = orc.voxelize(pos, J)
        codes = np.unique(orc.morton_encode_array(vox, J))
        A = rng.normal(-1, 2, size=(codes.size, 6))
        Y = orc.raht_forward(codes, J, A)
        tc = torch.from_numpy(codes.view(np.int64)).to(dev)
        out, info = gsc.raht_forward(tc, torch.from_numpy(A.astype(np.float32)).to(dev), J)
        back, info2 = gsc.raht_adjoint(tc, out, J)
        torch.cuda.synchronize()
        assert int(info[0]) == 0 and int(info2[0]) == 0
        scale = np.abs(Y).max(axis=0)
        assert (np.abs(out.cpu().numpy() - Y).max(axis=0) / scale).max() <= REL_TOL
        assert np.abs(back.cpu().numpy() - A).max() <= 1e-5 * np.abs(A).max()


def test_batch_equals_per_frame():
    dev = _dev()
    frames = [synth.make_frame(n, seed=20 + i) for i, n in enumerate([3000, 17_000, 1, 0, 9000])]
    p = gsc.make_params(9, 56, GROUPED)
    tens = [(torch.from_numpy(a).to(dev), torch.from_numpy(b).to(dev)) for a, b in frames]
    outs = gsc.encode_batch(tens, p)
    torch.cuda.synchronize()
    singles = []
    for a, b in tens:
        e = gsc.encode_frame(a, b, p)
        torch.cuda.synchronize()
        singles.append(e)
    for e, s in zip(outs, singles):
        e.check()
        assert e.to_bytes() == s.to_bytes()
    decs = gsc.decode_batch(outs, [max(f[0].shape[0], 1) for f in frames])
    torch.cuda.synchronize()
    for d, e in zip(decs, outs):
        d.check()
        nv = e.n_vox()
        ref = gsc.decode_frame(e.stream, 9, 56, max(nv, 1))
        torch.cuda.synchronize()
        assert torch.equal(d.attr[:nv], ref.attr[:nv]) and torch.equal(d.pos[:nv], ref.pos[:nv])


def test_deterministic_bytes():
    dev = _dev()
    pos, attr = synth.make_frame(200_000, seed=30)
    p = gsc.make_params(12, 56, GROUPED)
    tp, ta = torch.from_numpy(pos).to(dev), torch.from_numpy(attr).to(dev)
    a = gsc.encode_frame(tp, ta, p)
    b = gsc.encode_frame(tp, ta, p)
    torch.cuda.synchronize()
    assert a.to_bytes() == b.to_bytes()


@pytest.mark.parametrize("nv,C", [
    (500, 4),           # one tile: no upper level
    (513, 64),          # two tiles, three channel slices above them
    (400_000, 64),      # an upper item per workgroup
    (6_200_000, 32),    # an upper tile per workgroup, its two slices one after the other
    (14_000_000, 4),    # more upper tiles than workgroups: all schedules first
])
def test_adjoint_inverts_the_forward_over_the_upper_level_paths(nv, C):
    """A = T^T (T A) on float rows, one size for each way the inverse launch deals its upper tiles. Each of
    the at most 3J butterflies a value passes, in each direction, is off by a few FP32 roundings (about
    1.5e-7): 1e-5 of the largest value bounds their sum."""
    print(f"case nv={nv} C={C} transform and adjoint", flush=True)
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(nv)
    J = 12
    gaps = torch.randint(1, max(2, (1 << (3 * J)) // nv), (nv,), generator=g, device=dev)
    codes = torch.cumsum(gaps, 0) - 1
    assert int(codes[-1]) < 1 << (3 * J)
    A = torch.randn(nv, C, generator=g, device=dev)
    ws = gsc.Workspace(nv, J, C, dev)
    Y, info = gsc.raht_forward(codes, A, J, ws=ws)
    B, info2 = gsc.raht_adjoint(codes, Y, J, ws=ws)
    torch.cuda.synchronize()
    assert int(info[0]) == 0 and int(info2[0]) == 0
    assert (B - A).abs().max().item() <= 1e-5 * A.abs().max().item()
    # (orthonormal: the energy is kept)
    e = (Y.double().square().sum() / A.double().square().sum()).item()
    assert abs(e - 1.0) <= 1e-5


@pytest.mark.parametrize("J", [1, 9])
def test_decoding_at_the_capacity_where_the_octree_tiles_change(J):
    """Capacities of up to 2^19 voxels expand the octree with 1024 threads a tile, larger ones with 256:
    the same stream decodes to the same frame, bit for bit."""
    dev = torch.device("cuda:0")
    pos, attr = synth.make_frame(9000, seed=J)
    C = 5
    print(f"case J={J} decode capacities", flush=True)
    e = gsc.encode_frame(torch.from_numpy(pos).to(dev), torch.from_numpy(np.ascontiguousarray(attr[:, :C])).to(dev),
                         gsc.make_params(J, C, synth.quant_steps(synth.STEPS_GROUPED)[:C])).check()
    nv = e.n_vox()
    got = []
    for cap in (nv, 1 << 19, (1 << 19) + 1):
        d = gsc.decode_frame(e.stream, J, C, cap, want_vox=True)
        torch.cuda.synchronize()
        assert int(d.info[0].item()) == 0 and int(d.info[1].item()) == nv
        got.append([t[:nv].clone() for t in (d.pos, d.attr, d.vox)])
    for other in got[1:]:
        assert all(torch.equal(x, y) for x, y in zip(got[0], other))
