"""GPU parity of the band-decomposition kernels (csrc/bands.hip) against the
oracle's numpy FFTs (oracle/bands.py), through the C ABI's component op."""
import math

import numpy as np
import pytest

from oracle import bands, dit
from paper_2609_30096_amd import synth

from gpu_helpers import dev, normal, say

pytestmark = pytest.mark.gpu


def _guided(v, B, w):
    return v[1] + w * (v[0] - v[1]) if B == 2 else v[0]


@pytest.mark.parametrize("C,F,H,W,patch,B", [
    (4, 5, 12, 20, (1, 2, 2), 2),
    (3, 7, 6, 10, (1, 2, 2), 1),
    (2, 6, 8, 8, (2, 2, 2), 2),
    (1, 1, 2, 2, (1, 2, 2), 2),
    (2, 3, 34, 38, (1, 2, 2), 2),      # W > 32: two column blocks, the second ragged
    (16, 21, 60, 104, (1, 2, 2), 2),   # the Wan 81 x 480 x 832 latent
])
def test_band_energy_matches_oracle(C, F, H, W, patch, B):
    import torch
    from paper_2609_30096_amd import track
    say(f"band energy C={C} F={F} H={H} W={W} patch={patch} B={B}")
    shape = synth.LatentShape(C, F, H, W, 16)
    L = shape.tokens(patch)
    P = C * math.prod(patch)
    key = 7000 + C + F + H + W + B
    vL = normal((key, 1), (B, L, P))
    vS = vL + 0.3 * normal((key, 2), (B, L, P))
    w = 5.0
    ws = torch.empty(track.band_workspace_bytes(shape, patch), dtype=torch.uint8, device="cuda")
    got = track.op_band_energy(shape, B, w, dev(vL), dev(vS), ws, patch)
    d_tok = _guided(vS.astype(np.float64), B, w) - _guided(vL.astype(np.float64), B, w)
    sp, tp = bands.band_energies(dit.unpatchify(d_tok, C, F, H, W, patch))
    ref = np.concatenate([sp, tp])
    tot = float(sp.sum())
    say(f"  got {np.round(got, 3)}\n  ref {np.round(ref, 3)}")
    assert np.all(np.abs(got - ref) <= 2e-5 * tot + 2e-5 * np.abs(ref)), (got, ref)
    # Parseval on the device: both triples sum to ||d||^2
    assert got[:3].sum() == pytest.approx(tot, rel=1e-5)
    assert got[3:].sum() == pytest.approx(tot, rel=1e-5)
    # a second call on the same workspace gives the same bits
    again = track.op_band_energy(shape, B, w, dev(vL), dev(vS), ws, patch)
    np.testing.assert_array_equal(got, again)


@pytest.mark.parametrize("C,F,H,W,patch,offset", [
    (1, 1, 1, 1, (1, 1, 1), 0),
    (2, 3, 34, 258, (1, 2, 2), 0),    # three column groups, three staged chunks
    (1, 33, 98, 6, (1, 2, 2), 0),     # k_f beyond one block of 16, k_h beyond 48
    (1, 64, 256, 4, (1, 2, 2), 0),    # the largest F and H
    (1, 2, 2, 1024, (1, 2, 2), 0),    # the largest W
    (1, 1, 2, 840, (1, 2, 2), 0),     # the W with the most divisors
    (3, 5, 17, 33, (1, 1, 1), 0),     # odd sizes, element-wise staging
    (4, 5, 12, 20, (1, 2, 2), 1),     # velocities that are not 16-byte aligned
])
def test_band_energy_block_edges(C, F, H, W, patch, offset):
    """Tolerance: float32 DFT sums of up to 1024 terms and the float32 table entries, a few 1e-7 of the energy,
    and the float32 guided predictions, each off by at most 2^-23 of itself and its inputs (summed by
    Cauchy-Schwarz)."""
    import torch
    from paper_2609_30096_amd import track
    say(f"band energy edges C={C} F={F} H={H} W={W} patch={patch} offset={offset}")
    shape = synth.LatentShape(C, F, H, W, 16)
    L, P, B, w = shape.tokens(patch), C * math.prod(patch), 2, 5.0
    key = 7100 + C + F + H + W
    vL = normal((key, 1), (B, L, P))
    vS = vL + 0.3 * normal((key, 2), (B, L, P))

    def shifted(v):
        t = torch.empty(v.size + offset, device="cuda")
        t[offset:] = dev(v).reshape(-1)
        return t[offset:]

    ws = torch.empty(track.band_workspace_bytes(shape, patch), dtype=torch.uint8, device="cuda")
    got = track.op_band_energy(shape, B, w, shifted(vL), shifted(vS), ws, patch)
    d_tok = _guided(vS.astype(np.float64), B, w) - _guided(vL.astype(np.float64), B, w)
    sp, tp = bands.band_energies(dit.unpatchify(d_tok, C, F, H, W, patch))
    ref = np.concatenate([sp, tp])
    tot = float(sp.sum())
    size = (2 * w + 1) * (np.linalg.norm(vL) + np.linalg.norm(vS))
    assert np.all(np.abs(got - ref) <= 2e-6 * tot + 2 * np.sqrt(tot) * 2.0 ** -23 * size), (got, ref)


@pytest.mark.parametrize("C,F,H,W,patch,offset", [(2, 21, 60, 104, (1, 2, 2), 0), (1, 5, 12, 20, (1, 2, 2), 0),
                                                  (2, 5, 12, 20, (1, 2, 2), 1), (2, 6, 10, 6, (2, 1, 1), 0)])
def test_band_energy_of_a_constant_is_exact(C, F, H, W, patch, offset):
    """A constant difference of 3 on integer velocities: its transforms at frequency 0 are sums of integers below 2^24,
    through table entries that are exactly 1, so both low bands hold 9 C F H W but for float64 roundings and the
    squares of the other frequencies' rounding (below 1e-13 of it).  The rounding of the table's other entries (1e-8
    and more of an energy) must not reach them."""
    import torch
    from paper_2609_30096_amd import track
    say(f"band energy constant C={C} F={F} H={H} W={W} patch={patch} offset={offset}")
    shape = synth.LatentShape(C, F, H, W, 16)
    n = C * F * H * W
    vL = np.rint(100 * normal((7200, F, H), (n + offset,))).astype(np.float32)
    ws = torch.empty(track.band_workspace_bytes(shape, patch), dtype=torch.uint8, device="cuda")
    got = track.op_band_energy(shape, 1, 1.0, dev(vL)[offset:], dev(vL + 3)[offset:], ws, patch)
    want = np.array([9.0 * n, 0, 0] * 2)
    assert np.all(np.abs(got - want) <= 1e-12 * 9.0 * n), got / (9.0 * n) - [1, 0, 0] * 2


def test_band_energy_argument_checks():
    import torch
    from paper_2609_30096_amd import track
    shape = synth.LatentShape(2, 3, 4, 4, 16)
    v = torch.zeros(2 * 2 * 3 * 4 * 4, device="cuda")
    ws = torch.empty(track.band_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    with pytest.raises(track.TrackError):  # workspace too small
        track.op_band_energy(shape, 2, 1.0, v, v, ws[:256])
    with pytest.raises(track.TrackError):  # batch 3
        track.op_band_energy(shape, 3, 1.0, v, v, ws)
    with pytest.raises(track.TrackError):  # latent not divisible by the patch
        track.op_band_energy(synth.LatentShape(2, 3, 5, 4, 16), 2, 1.0, v, v, ws)
    assert track.band_workspace_bytes(synth.LatentShape(2, 3, 300, 4, 16)) == 0  # H beyond the kernels' bound
