"""GPU: the exhaustive search's bounded groups.  A dense set longer than one ring window skips groups of
64 widths that an upper bound shows cannot raise a best; the same widths given as a list are all
evaluated.  Both give the same planes and candidates bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def rows(kind, n, rng):
    x = rng.standard_normal((3, n)).astype(np.float32)
    t = np.arange(n)
    if kind == "pulses":
        for d, (s, w, a) in enumerate(((300, 700, 1.0), (0, 255, 2.0), (n - 400, 400, 1.5))):
            x[d, s:s + w] += np.float32(a)
    elif kind == "trend":                       # every group raises a best
        x += (t * 1e-2).astype(np.float32)
    elif kind == "offset":                      # large sums either way: slack against rounding
        x[0] += 1000.0
        x[1] -= 1000.0
    elif kind == "constant":                    # ties between widths
        x[:] = np.array([0.0, 1.0, -1.0], np.float32)[:, None]
    elif kind == "steps":                       # sums that rise and fall in steps of a group
        x = (np.where((t // 64) % 2 == 0, 1.0, -1.0) * np.ones((3, 1))).astype(np.float32)
    elif kind == "special":
        x[0, 900] = np.nan
        x[1, 1000] = np.inf
        x[2, 1100] = -np.inf
        x[2, 40] = 3e38
    return x


@pytest.mark.parametrize("kind", ["noise", "pulses", "trend", "offset", "constant", "steps", "special"])
@pytest.mark.parametrize("l_end,n", [(513, 2000), (576, 1111), (1000, 2049), (1600, 1500), (2305, 6001)])
def test_bounded_groups_equal_the_width_list(kind, l_end, n):
    from paper_1910_08324_amd import spd
    dev = torch.device("cuda:0")
    x = torch.from_numpy(rows(kind, n, np.random.default_rng(l_end))).to(dev)
    mu = torch.zeros(3, device=dev)
    sg = torch.full((3,), 1.25, device=dev)
    got = []
    for widths in (None, range(1, l_end + 1)):
        r = spd.search(x, mu, sg, spd.Config("exh", l_end, threshold=4.0, widths=widths), cand_cap=1 << 15)
        torch.cuda.synchronize()
        Y, W = r.level(0)
        got.append((Y.cpu().numpy().view(np.uint32), W.cpu().numpy(), r.candidates_host()))
    for a, b in zip(*got):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("l_end", [15, 16, 17, 255, 256, 257, 511, 512])
def test_short_sets_replay_every_position(l_end):
    """The argmax replay at every group of a short set and both item counts per wave, against the
    definition in 64 bits: the width attains the maximum (to the SNR's rounding) and fits."""
    from paper_1910_08324_amd import spd
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(l_end)
    n = 1500
    x = rng.standard_normal((4, n)).astype(np.float32)
    x[1, 700:700 + l_end] += 1.0
    t = torch.from_numpy(x).to(dev)
    mu, sg = torch.zeros(4, device=dev), torch.ones(4, device=dev)
    P = np.concatenate([np.zeros((4, 1)), np.cumsum(x.astype(np.float64), axis=1)], axis=1)
    first = None
    for segment in (256, 512, 1024):
        r = spd.search(t, mu, sg, spd.Config("exh", l_end, segment=segment, candidates=False))
        torch.cuda.synchronize()
        Y, W = (a.cpu().numpy() for a in r.level(0))
        W = W.view(np.uint16).astype(np.int64)
        s = np.arange(n)[None, :]
        assert (W >= 1).all() and (W <= l_end).all() and (s + W <= n).all()
        own = (np.take_along_axis(P, s + W, axis=1) - P[:, :n]) / np.sqrt(W)
        best = np.full((4, n), -np.inf)
        for L in range(1, l_end + 1):
            best[:, :n - L + 1] = np.maximum(best[:, :n - L + 1], (P[:, L:] - P[:, :n - L + 1]) / np.sqrt(L))
        tol = 1e-5 * np.maximum(1.0, np.abs(best))
        assert (np.abs(Y - best) <= tol).all() and (np.abs(own - best) <= 2 * tol).all()
        if first is None:
            first = (Y, W)
        assert np.array_equal(first[0], Y) and np.array_equal(first[1], W)
