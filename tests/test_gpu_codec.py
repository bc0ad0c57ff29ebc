"""Arc codec on the GPU against the FP64 reference codec: the same fallback
decisions and codes (both quantise in FP64; a code may differ only where a
field sits within rounding of a tie), decoding within FP32 rounding of the
reference's decoding of the same codes, the Eq. 5 bound on the decoded
arcs, and fallback arcs returned whole."""

import numpy as np
import pytest

import latgen
from oracle import codec

pytestmark = pytest.mark.gpu


def _line(msg):
    print(msg, flush=True)


CASES = [
    ("cfg2_bcc5", lambda: latgen.config(2, scale=5), 16),
    ("cfg4_octet3", lambda: latgen.config(4, scale=3), 12),
    ("cubic_cones", lambda: latgen.cubic(5, radius=("uniform", 0.05, 0.15), jitter=0.04, seed=5), 8),
]


@pytest.mark.parametrize("name,make,k", CASES, ids=[c[0] for c in CASES])
def test_codec_matches_reference(name, make, k):
    import torch

    from paper_2405_15197_amd import Mesher

    lat = make()
    M = Mesher(lat)
    try:
        r = M.run(k)
        enc = M.encode_arcs(r)
        dec = M.decode_arcs(enc, r)
        torch.cuda.synchronize()
        arcs = r.arc_f32.cpu().numpy().T.astype(np.float64)
        u32 = r.arc_u32.cpu().numpy().view(np.uint32).T
        codes = enc["codes"].cpu().numpy().view(np.uint32)
        mask = enc["mask"].cpu().numpy().view(np.uint32)
        dec = dec.cpu().numpy().T.astype(np.float64)
        r_min, r_max = enc["r_min"], enc["r_max"]
    finally:
        M.close()
    E = arcs.shape[0]
    fb_gpu = ((mask[np.arange(E) >> 5] >> (np.arange(E) & 31)) & 1).astype(bool)
    p, q, node = u32[:, 0] & 0xFF, (u32[:, 0] >> 8) & 0xFF, u32[:, 2]
    d = codec.reference_dirs(lat, node, p, q)
    qo, fb_o, raw = codec.encode(arcs, d, r_min, r_max)
    _line(f"codec {name}: {E} arcs, {fb_gpu.sum()} kept whole ({enc['n_fallback']})")
    assert enc["n_fallback"] == int(fb_gpu.sum())
    assert np.array_equal(fb_gpu, fb_o)
    ok = ~fb_o
    ref_codes = codec.pack(qo)
    diff = np.any(codes != ref_codes, axis=1) & ok
    if diff.any():
        # allowed only where a field's scaled value is within rounding of a
        # tie between two levels
        near = np.zeros(E, bool)
        for name_f, _ in codec.FIELDS:
            f = np.asarray(raw[name_f])
            near |= np.abs(f - np.floor(f) - 0.5) < 1e-9
        assert not (diff & ~near).any(), int((diff & ~near).sum())
    _line(f"  codes differing from the reference: {int(diff.sum())}")
    # decoding: the reference's decoding of the GPU's own codes
    ref_dec = codec.decode(codec.unpack(codes[ok]), d[ok], r_min, r_max)
    tol = 2.5e-7 * np.abs(ref_dec) + 1e-9
    assert (np.abs(dec[ok] - ref_dec) <= tol).all(), float(np.max(np.abs(dec[ok] - ref_dec) / tol))
    # arcs kept whole come back bit for bit
    assert np.array_equal(dec[fb_o].astype(np.float32), arcs[fb_o].astype(np.float32))
    # Eq. 5 on the decoded arcs (FP32 rounding of the output aside)
    err = codec.arc_error(arcs[ok], dec[ok])
    _line(f"  max error {err.max() / r_max:.3e} r_max (bound {codec.eq5_bound():.3e})")
    assert err.max() <= codec.eq5_bound() * r_max + 4e-7 * r_max


def test_codec_fallback_capacity():
    import torch

    from paper_2405_15197_amd import Mesher
    from paper_2405_15197_amd.latmesh import LM_ERR_CAPACITY, LatmeshError

    lat = latgen.cubic(4, radius=("uniform", 0.05, 0.15), jitter=0.04, seed=5)
    M = Mesher(lat)
    try:
        r = M.run(8)
        # a radius range that leaves every arc outside the format
        with pytest.raises(LatmeshError) as e:
            M.encode_arcs(r, r_min=10.0, r_max=10.0, cap_fallback=4)
        assert e.value.code == LM_ERR_CAPACITY
        enc = M.encode_arcs(r, r_min=10.0, r_max=10.0, cap_fallback=r.arc_f32.shape[1])
        dec = M.decode_arcs(enc, r)
        torch.cuda.synchronize()
        assert enc["n_fallback"] == r.arc_f32.shape[1]
        assert torch.equal(dec, r.arc_f32)
    finally:
        M.close()


def test_decode_every_angle_code():
    """Every code of an azimuth and of a polar angle, for both vectors: FP64
    to a few rounding steps, then one rounding to FP32.  b's direction
    a x d / |a x d| magnifies them by 1 / |a x d|."""
    import types

    import torch

    from paper_2405_15197_amd import Mesher

    lat = latgen.config(4, scale=2)
    rng = np.random.default_rng(4)
    n = 1 << 16
    i = np.arange(n)
    q = {name: rng.integers(0, 1 << bits, n) for name, bits in codec.FIELDS}
    q["pha"], q["tha"] = i, i % (1 << codec.M_TH)
    q["phc"], q["thc"] = (i * 40503 + 7) % n, (i // 2) ^ 1
    codes = codec.pack(q)
    M = Mesher(lat)
    try:
        r = M.run(8)
        sel = torch.from_numpy(rng.integers(0, r.arc_u32.shape[1], n)).cuda()
        u32 = r.arc_u32[:, sel].contiguous()
        lo, hi = M.radius_range()
        enc = {"codes": torch.from_numpy(codes.view(np.int32)).cuda(), "r_min": lo, "r_max": hi, "cap_fallback": 0,
               "mask": torch.zeros(n // 32, dtype=torch.int32, device="cuda"), "_fb_full": torch.empty((1, 11), device="cuda")}
        dec = M.decode_arcs(enc, types.SimpleNamespace(arc_u32=u32)).cpu().numpy().T.astype(np.float64)
        u = u32.cpu().numpy().view(np.uint32)
    finally:
        M.close()
    d = codec.reference_dirs(lat, u[2], u[0] & 0xFF, (u[0] >> 8) & 0xFF)
    want = codec.decode(q, d, lo, hi)
    ah = want[:, 3:6] / np.linalg.norm(want[:, 3:6], axis=1)[:, None]
    x = np.linalg.norm(np.cross(ah, d), axis=1)
    tol = 2.0**-24 * np.abs(want) + 16 * 2.0**-52 * 4 * hi
    tol[:, 6:9] += 16 * 2.0**-52 * hi / np.maximum(x, 1e-12)[:, None]
    assert (np.abs(dec - want) <= tol * (1 + 1e-6)).all(), float(np.max(np.abs(dec - want) / tol))


@pytest.mark.parametrize("quantile", [0.001, 0.3, 0.97])
def test_arcs_kept_whole_between_coded_ones(quantile):
    """Few, some and most arcs of a wave out of the radius range: every one
    has a slot of its own and comes back bit for bit; a ragged last wave."""
    from paper_2405_15197_amd import Mesher

    M = Mesher(latgen.cubic(5, radius=("uniform", 0.05, 0.15), jitter=0.04, seed=5))
    try:
        r = M.run(8)
        E = r.arc_f32.shape[1] - 37
        r.arc_f32, r.arc_u32 = r.arc_f32[:, :E], r.arc_u32[:, :E]
        arcs = r.arc_f32.cpu().numpy()
        ra = np.linalg.norm(arcs[3:6].astype(np.float64), axis=0)
        lo = float(np.quantile(ra, quantile))
        hi = max(lo, M.radius_range()[1])
        enc = M.encode_arcs(r, r_min=lo, r_max=hi, cap_fallback=E)
        dec = M.decode_arcs(enc, r).cpu().numpy()
        mask = enc["mask"].cpu().numpy().view(np.uint32)
        codes = enc["codes"].cpu().numpy()
    finally:
        M.close()
    i = np.arange(E)
    fb = ((mask[i >> 5] >> (i & 31)) & 1).astype(bool)
    assert fb[ra < np.float32(lo) * (1 - 1e-6)].all() and 0 < fb.sum() == enc["n_fallback"]
    assert np.array_equal(np.sort(codes[fb, 0]), np.arange(fb.sum()))
    assert np.array_equal(dec[:, fb], arcs[:, fb])
    assert not np.array_equal(dec[:, ~fb], arcs[:, ~fb])
