"""GPU parity of the batched form: many independent complex64 1D transforms
of mixed lengths plus 2D transforms, as one launch per (length, pass) group
(mode 0), as a single persistent launch for the whole batch (mode 1) or as
one persistent launch per phase (mode 2), against the oracle transform by
transform (rel L2 <= 1e-5 each, on the complex64-rounded inputs); the three
modes run the same tile code and must agree bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2004_09883_amd import fb, inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOL = 1e-5


def rel_l2(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def packed_input(batch, seed):
    x = inputs.uniform_grid((batch.elements,), seed)
    return inputs.round_c64(x)


def ref_transform(batch, x, i, sign):
    o = batch.offsets[i]
    if i < len(batch.lens):
        seg = x[o:o + batch.lens[i]].astype(np.complex128)
        return oracle.fft1d_many(seg[None, :], sign)[0]
    s = batch.side2d
    seg = x[o:o + s * s].astype(np.complex128).reshape(s, s)
    return oracle.fft2d(seg, sign).reshape(-1)


def run(batch, x, direction, persistent, in_place):
    xin = torch.from_numpy(x).cuda()
    out = xin if in_place else torch.empty_like(xin)
    ws = torch.zeros(batch.workspace_bytes(in_place) + 256, dtype=torch.uint8, device="cuda")
    wsp = ws.data_ptr()
    wsp = (wsp + 255) // 256 * 256
    fb.fb_batch_exec(batch, xin, out, wsp, direction, persistent)
    torch.cuda.synchronize()
    return out.cpu().numpy()


MIXED = [256, 768, 4096, 3072, 6144, 8192, 24576, 65536, 196608, 12, 2, 3, 48, 512, 98304, 256, 12288, 16384,
         32768, 49152, 1536, 2048]


MODES = (0, 1, 2)


@pytest.mark.parametrize("persistent", MODES)
@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("direction", [fb.FB_FORWARD, fb.FB_INVERSE])
def test_mixed_batch(persistent, in_place, direction):
    print(f"batch persistent={persistent} in_place={in_place} dir={direction}", flush=True)
    batch = fb.Batch(MIXED, n2d=3, side2d=64)
    x = packed_input(batch, 3)
    got = run(batch, x, direction, persistent, in_place)
    for i in range(len(MIXED) + 3):
        o = batch.offsets[i]
        n = MIXED[i] if i < len(MIXED) else 64 * 64
        e = rel_l2(got[o:o + n].astype(np.complex128), ref_transform(batch, x, i, direction))
        assert e < TOL, (i, n, e)


def test_persistent_equals_per_group_bitwise():
    batch = fb.Batch(MIXED, n2d=2, side2d=512)
    assert "onelaunch=1" in batch.description, batch.description
    x = packed_input(batch, 5)
    for in_place in (False, True):
        for direction in (fb.FB_FORWARD, fb.FB_INVERSE):
            a = run(batch, x, direction, 0, in_place)
            b = run(batch, x, direction, 1, in_place)
            assert np.array_equal(a, b), (in_place, direction)
            c = run(batch, x, direction, 2, in_place)
            assert np.array_equal(a, c), (in_place, direction)
    d = run(batch, x, fb.FB_FORWARD, 1, False)   # a second single launch on the same plan
    assert np.array_equal(d, run(batch, x, fb.FB_FORWARD, 0, False))


def test_batch_workload_4096_plus_64x512x512():
    """4096 1D lengths drawn from {2^k, 3*2^k : 8 <= k <= 16} (seed 3) plus
    64 2D 512 x 512 transforms; uniform inputs.  Checks a sample of
    transforms of every length (the smallest and the largest index of each)
    and two 2D transforms, in both execution modes."""
    lens = inputs.batch_lengths(4096, 3).tolist()
    batch = fb.Batch(lens, n2d=64, side2d=512)
    print("batch plan:", batch.description, flush=True)
    assert "onelaunch=1" in batch.description   # the workload runs in one launch
    x = packed_input(batch, 3)
    first = {}
    last = {}
    for i, n in enumerate(lens):
        first.setdefault(n, i)
        last[n] = i
    sample = sorted(set(first.values()) | set(last.values())) + [4096, 4096 + 63]
    outs = []
    for persistent in MODES:
        got = run(batch, x, fb.FB_FORWARD, persistent, False)
        outs.append(got)
        worst = 0.0
        for i in sample:
            o = batch.offsets[i]
            n = lens[i] if i < 4096 else 512 * 512
            e = rel_l2(got[o:o + n].astype(np.complex128), ref_transform(batch, x, i, fb.FB_FORWARD))
            worst = max(worst, e)
            assert e < TOL, (persistent, i, n, e)
        print(f"batch workload persistent={persistent}: {len(sample)} transforms checked, worst rel L2 {worst:.2e}",
              flush=True)
    assert np.array_equal(outs[0], outs[1]) and np.array_equal(outs[0], outs[2]) and np.array_equal(outs[0], outs[2])


@pytest.mark.parametrize("lens,n2d,side", [([], 2, 64), ([196608], 0, 0), ([2], 0, 0), ([3] * 5, 0, 0),
                                           ([24576, 24576], 1, 512), ([4096] * 3 + [8], 0, 0)])
def test_batch_edge_shapes(lens, n2d, side):
    """Only 2D transforms, a single transform of the largest length, a single
    length-2 transform, several tiny transforms, one long length plus one 2D
    transform: both modes against the oracle, and equal to each other."""
    print(f"batch edge lens={lens[:4]} n2d={n2d} side={side}", flush=True)
    batch = fb.Batch(lens, n2d=n2d, side2d=side)
    x = packed_input(batch, 11)
    outs = []
    for persistent in MODES:
        got = run(batch, x, fb.FB_FORWARD, persistent, False)
        for i in range(len(lens) + n2d):
            o = batch.offsets[i]
            n = lens[i] if i < len(lens) else side * side
            e = rel_l2(got[o:o + n].astype(np.complex128), ref_transform(batch, x, i, fb.FB_FORWARD))
            assert e < TOL, (persistent, i, n, e)
        outs.append(got)
    assert np.array_equal(outs[0], outs[1]) and np.array_equal(outs[0], outs[2])


@pytest.mark.parametrize("lens,n2d,side", [([196608], 0, 0), ([256] * 7 + [98304], 2, 64), ([4096] * 3, 0, 0)])
def test_unbalanced_batch_equals_per_group_bitwise(lens, n2d, side):
    """Batches whose longest transform outweighs an even share of the device
    run mode 1 phase by phase: the bits of the other modes, in and out of
    place, both directions."""
    batch = fb.Batch(lens, n2d=n2d, side2d=side)
    balance = float(batch.description.split("balance=")[1].split()[0])
    assert balance > 1.25, batch.description
    x = packed_input(batch, 9)
    for in_place in (False, True):
        for direction in (fb.FB_FORWARD, fb.FB_INVERSE):
            a = run(batch, x, direction, 0, in_place)
            assert np.array_equal(a, run(batch, x, direction, 1, in_place)), (in_place, direction)
    i = len(lens) - 1
    o = batch.offsets[i]
    assert rel_l2(a[o:o + lens[i]].astype(np.complex128), ref_transform(batch, x, i, fb.FB_INVERSE)) < TOL


@pytest.mark.parametrize("lens,n2d,side", [([6144] * 2048 + [256] * 8191, 0, 0), ([8192] * 1024 + [48] * 3000, 512, 64),
                                           ([4096] * 2045, 0, 0)])
def test_balanced_batch_in_one_launch_equals_per_group_bitwise(lens, n2d, side):
    """Batches that mode 1 runs in one launch (their description's balance is
    at most 1.25): the bits of the per-group mode, in and out of place, both
    directions, and again on the same plan; 6144 points are split so that an
    item holds two transforms."""
    batch = fb.Batch(lens, n2d=n2d, side2d=side)
    print("balanced batch:", batch.description, flush=True)
    assert "onelaunch=1" in batch.description
    assert float(batch.description.split("balance=")[1].split()[0]) <= 1.25, batch.description
    x = packed_input(batch, 17)
    for in_place in (False, True):
        for direction in (fb.FB_FORWARD, fb.FB_INVERSE):
            a = run(batch, x, direction, 0, in_place)
            for _ in range(2):
                assert np.array_equal(a, run(batch, x, direction, 1, in_place)), (in_place, direction)
    for i in (0, 1, len(lens) // 2, len(lens) - 1, len(lens) + n2d - 1):
        o = batch.offsets[i]
        n = lens[i] if i < len(lens) else side * side
        assert rel_l2(a[o:o + n].astype(np.complex128), ref_transform(batch, x, i, fb.FB_INVERSE)) < TOL, i


def test_balanced_batch_is_one_launch():
    """The launches that mode 1 makes, by the profile: one where the balance is
    at most 1.25, one per phase above it."""
    for lens, names in (([8192] * 1024, ["batch_onelaunch<c64>"]),
                        ([8192] * 3, ["batch_persistent<c64,phase0>", "batch_persistent<c64,phase1>"])):
        batch = fb.Batch(lens)
        x = torch.zeros(batch.elements, dtype=torch.complex64, device="cuda")
        y = torch.empty_like(x)
        ws = torch.empty(256, dtype=torch.uint8, device="cuda")
        fb.fb_profile_enable(True)
        fb.fb_batch_exec(batch, x, y, ws, fb.FB_FORWARD, 1)
        report = fb.fb_profile_report()
        fb.fb_profile_enable(False)
        assert [r["kernel"] for r in report] == names, batch.description


@pytest.mark.parametrize("lens,n2d", [([], 1), ([], 2), ([3], 5), ([48, 3, 256], 301), ([2] * 7, 4000), ([], 65536)])
def test_images_of_odd_side(lens, n2d):
    """3 x 3 images, whose columns do not pair up: every mode, in and out of
    place, both directions, against the oracle; nothing past the data is
    written."""
    batch = fb.Batch(lens, n2d=n2d, side2d=3)
    x = packed_input(batch, 23)
    e = batch.elements
    ws = torch.zeros(8 * e + 512, dtype=torch.uint8, device="cuda")
    wsp = (ws.data_ptr() + 255) // 256 * 256
    for direction in (fb.FB_FORWARD, fb.FB_INVERSE):
        ref = np.concatenate([ref_transform(batch, x, i, direction) for i in range(len(lens) + n2d)])
        for in_place in (False, True):
            for persistent in MODES:
                print(f"odd side lens={len(lens)} n2d={n2d} dir={direction} in_place={in_place} mode={persistent}",
                      flush=True)
                buf = torch.full((e + 64,), 7.0, dtype=torch.complex64, device="cuda")
                buf[:e] = torch.from_numpy(x)
                src = buf[:e]
                dst = src if in_place else torch.full((e + 64,), 7.0, dtype=torch.complex64, device="cuda")[:e]
                fb.fb_batch_exec(batch, src, dst, wsp, direction, persistent)
                assert rel_l2(dst.cpu().numpy().astype(np.complex128), ref) < TOL
                whole = torch.as_strided(dst, (e + 64,), (1,))
                assert torch.all(whole[e:] == 7.0)
