"""GPU: the peak finder over chunks of 256 slots.  Candidate lists do not depend on how the tiles cut
the rows (several chunks per bit of a tile's word, chunks that a tile ends inside, peaks beside chunk
and tile edges), on where the values come from (planes, chunk records, slots formed again when the
records' room is used up), and follow the oracle's rules."""
import numpy as np
import pytest

import synth
from oracle import planes as oplanes, widths as ow
from tests import parity
from tests.test_gpu_parity import dev, make_input  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def lists(dev, x, mu, sg, segment, step_levels, **kw):
    from paper_1910_08324_amd import spd
    t = [torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(dev) for a in (x, mu, sg)]
    out = []
    for planes in (True, False):
        cfg = spd.Config(planes=planes, segment=segment, step_levels=step_levels, **kw)
        r = spd.search(*t, cfg, cand_cap=1 << 18)
        torch.cuda.synchronize()
        out.append((int(r.count.item()), r.candidates_host()))
    return out


@pytest.mark.parametrize("method,segment,step_levels", [
    ("ig1", 256, 1), ("ig1", 768, 2), ("ig1", 8192, 4), ("ig1", 8448, 1), ("ig1", 14848, 1),
    ("bd16", 256, 1), ("bd16", 768, 2), ("bd16", 7168, 3)])
@pytest.mark.parametrize("threshold", [4.5, 1.5])
def test_lists_do_not_depend_on_tiles(dev, method, segment, step_levels, threshold):
    """1.5 is far below the noise's own peaks: most slots are above it and few chunks get a record."""
    n_dm, n = 5, 2 * 32768 + 515
    # peaks on either side of chunk and tile edges, in rows that see each other
    edges = (255, 256, 767, 768, 8191, 8192, 8447, 8448, 14847, 14848, 65535, 65536)
    pulses = [synth.Pulse(i % n_dm, e, 1, 12.0 + i) for i, e in enumerate(edges)]
    pulses += [synth.Pulse(2, 30000, 6000, 60.0)]
    x, mu, sg = make_input(n_dm, n, 77, pulses=pulses)
    kw = dict(method=method, l_end=512, threshold=threshold)
    (n0, ref), (n1, rec) = lists(dev, x, mu, sg, 0, 0, **kw)
    assert n0 == n1 == len(ref) > 100 and np.array_equal(ref, rec)
    for got, c in lists(dev, x, mu, sg, segment, step_levels, **kw):
        assert got == n0 and np.array_equal(c, ref)
    if threshold > 4:
        R = oplanes.planes(x, mu, sg, ow.method_levels(method, 512))
        parity.check_candidates(ref, R, threshold, what=method)


@pytest.mark.parametrize("cap", [0, 1, 37])
def test_short_list_is_a_prefix(dev, cap):
    """A list with less room holds the first candidates; the count is the whole number."""
    from paper_1910_08324_amd import spd
    x, mu, sg = make_input(40, 20000, 78, pulses=[synth.Pulse(7, 9000, 30, 25.0)])
    t = [torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(dev) for a in (x, mu, sg)]
    for planes in (True, False):
        cfg = spd.Config("ig1", 512, threshold=3.0, planes=planes)
        whole = spd.search(*t, cfg)
        r = spd.Runner(*t, cfg, cand_cap=max(1, cap))
        r.cap = cap
        r.result.cand.fill_(0xA5)
        r.search()
        torch.cuda.synchronize()
        assert int(r.result.count.item()) == int(whole.count.item()) > 100
        got = r.result.cand.cpu().numpy().view(spd.CANDIDATE_DTYPE)[:cap]
        assert np.array_equal(got, whole.candidates_host()[:cap])
        if cap == 0:
            assert (r.result.cand.cpu().numpy() == 0xA5).all()
