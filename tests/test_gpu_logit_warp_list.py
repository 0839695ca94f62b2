"""Every variant of the front end gives the same bits: aligned rows in registers, unaligned ones, and for rows too long for
registers the list of tokens with mass and the streaming passes where the list does not apply.  A short row spread over a
long one, in order, with tokens without mass in between, has the short row's probabilities."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHORT = 20000


def rows(rng):
    z = rng.standard_normal((8, SHORT)).astype(np.float32) * 3
    z[1] = np.sort(z[1])                       # the maximum grows to the end: more and more tokens are listed
    z[2] = 1.5                                 # all tokens tie
    z[3] = np.round(z[3])                      # ties at the threshold
    z[4, ::7] = np.nan
    z[5, 17] = z[5, 19990] = np.inf
    z[6, 4000:] = -np.inf
    z[7] *= 0.01                               # flat
    return z


@pytest.mark.parametrize("V", [20003, 32769, 53247, 53251, 65540, 70001, 131072, 262145])
@pytest.mark.parametrize("temperature,top_p", [(0.05, 0.95), (0.2, 0.95), (0.35, 0.5), (0.5, 0.9), (1.0, 0.95), (0.2, 1.0)])
def test_long_rows_have_the_bits_of_short_ones(V, temperature, top_p):
    import torch
    import paper_2404_15778_amd as bass
    rng = np.random.default_rng(V)
    short = rows(rng)
    at = np.sort(rng.choice(V, SHORT, replace=False))
    filler = np.where(np.isfinite(short), short, -1e3).max(-1, keepdims=True) - np.float32(1000.0)
    long = np.broadcast_to(filler, (len(short), V)).copy()
    long[:, at] = short
    out = []
    for z in (short, long):
        z = torch.from_numpy(z).cuda()
        p = torch.full_like(z, 7.0)
        bass.bass_warp_probs(z, temperature, top_p, p)
        out.append(p.cpu().numpy())
    assert np.array_equal(out[1][:, at].view(np.uint32), out[0].view(np.uint32))
    rest = np.ones(V, bool)
    rest[at] = False
    assert not out[1][:, rest].any()


@pytest.mark.parametrize("V", [53251, 65540, 131072, 262145])
@pytest.mark.parametrize("flat_from", [0.3, 0.9])
def test_a_list_that_overflows_late_is_given_up(V, flat_from):
    """Peaked at first, flat in the rest: more tokens have mass than the list holds, which shows after the first batch only."""
    import torch
    import paper_2404_15778_amd as bass
    rng = np.random.default_rng(V)
    z = np.full((3, V), -60.0, np.float32)
    z[:, 7] = 0.0
    z[:2, int(flat_from * V):] = rng.standard_normal((2, V - int(flat_from * V))).astype(np.float32) * 0.01
    z[1, V - 1] = 30.0  # ... and a peak at the end, under which nothing of it has mass
    p = torch.full((3, V), 7.0, device="cuda:0")
    bass.bass_warp_probs(torch.from_numpy(z).cuda(), 1.0, 0.95, p)
    p = p.cpu().numpy().astype(np.float64)
    n = int((z[0] > -1).sum())
    assert abs((p[0] > 0).sum() - 0.95 * n) <= 0.01 * n and abs(p[0].sum() - 1.0) <= 1e-5
    kept = p[0] > 0
    assert z[0][kept].min() >= z[0][~kept].max()  # the most probable tokens
    assert p[1, V - 1] == 1.0 and p[1].sum() == 1.0
    assert p[2, 7] == 1.0 and p[2].sum() == 1.0
