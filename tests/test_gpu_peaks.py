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


@pytest.mark.parametrize("method", ["ig1", "exh"])
@pytest.mark.parametrize("n_out", [2301, 2302, 2303, 2304])
def test_last_slot_sees_the_evaluated_slot_after_it(dev, method, n_out):
    """With look-ahead samples the last slot of a row is held against the slot after it where the search
    evaluates that one with it (same group of 4, exhaustive: same 256); planes and candidates only."""
    from paper_1910_08324_amd import spd
    n_dm, n, l_end = 6, 2900, 200
    pulses = [synth.Pulse(0, n_out - 1, 3, 30.0), synth.Pulse(1, n_out, 1, 30.0), synth.Pulse(2, n_out - 20, 40, 40.0),
              synth.Pulse(3, n_out - 1, 1, 30.0), synth.Pulse(4, n_out - 100, 190, 40.0)]
    x, mu, sg = make_input(n_dm, n, 79, pulses=pulses)
    t = [torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(dev) for a in (x, mu, sg)]
    wide = spd.search(*t, spd.Config(method, l_end, threshold=6.0), n_out=n_out + 64 * 4)
    torch.cuda.synchronize()
    for planes in (True, False):
        r = spd.search(*t, spd.Config(method, l_end, threshold=6.0, planes=planes), n_out=n_out)
        torch.cuda.synchronize()
        got = {(int(c["level"]), int(c["dm"]), int(c["start"])) for c in r.candidates_host()}
        for i in range(r.info.n_levels):
            k, slots = int(r.info.level_shift[i]), int(r.info.plane_slots[i])
            Y = np.full((n_dm + 2, slots + 2), -np.inf, np.float32)
            Y[1:-1, 1:-1] = wide.level(i)[0][:, :slots].cpu().numpy()
            after = wide.level(i)[0][:, slots].cpu().numpy()
            for d in range(n_dm):
                c, m = Y[d + 1, slots], slots - 1
                ok = c > 6.0 and all(c > v for v in (*Y[d, slots - 1:slots + 2], Y[d + 1, slots - 1])) and \
                    all(c >= v for v in (Y[d + 1, slots + 1], *Y[d + 2, slots - 1:slots + 2]))
                seen = slots % (256 if method == "exh" else 4) != 0
                if ok and seen and not c >= after[d]:
                    ok = False
                assert ((i, d, m << k) in got) == ok, (method, planes, i, d)


@pytest.mark.parametrize("method,n_dm,n,l_end", [("bd32", 4, 4096, 1533), ("ig1", 1, 257, 64), ("bd16", 16, 16384, 512)])
def test_small_block_under_a_bright_pulse(dev, method, n_dm, n, l_end):
    """One pulse lifts nearly every slot of its row: full records, and in the largest block too many."""
    x, mu, sg = make_input(n_dm, n, 79, pulses=[synth.Pulse(0, n // 4, n // 2, 900.0)])
    if n_dm > 4:
        x[4:] += 6.0
    (n0, ref), (n1, rec) = lists(dev, x, mu, sg, 0, 0, method=method, l_end=l_end, threshold=5.0)
    assert n0 == n1 == len(ref) > 0 and np.array_equal(ref, rec)
    R = oplanes.planes(x, mu, sg, ow.method_levels(method, l_end))
    parity.check_candidates(ref, R, 5.0, what=method)


@pytest.mark.parametrize("planes", [True, False])
@pytest.mark.parametrize("method,l_end,segment,step_levels", [
    ("bd8", 500, 0, 0), ("bd16", 400, 512, 2), ("bd32", 700, 0, 0), ("bd32", 700, 0, 1), ("bd", 300, 256, 3)])
@pytest.mark.parametrize("n_out", [2290, 2301, 2306])
def test_last_slot_of_boxdit_levels(dev, planes, method, l_end, segment, step_levels, n_out):
    """BoxDIT: the slot after a level's last one is evaluated with the carried prefix that the search of a
    longer plane gives it, at every level (its prefix comes from slots past the lower levels' ends), for
    every remainder of the levels' slots and with steps that hand the prefixes on."""
    from paper_1910_08324_amd import spd
    n_dm, n, thr = 96, 4200, 6.0
    rng = np.random.default_rng(n_out)
    # pulses of any width that end near the planes' ends, so that the two slots are close
    pulses = [synth.Pulse(d, n_out - int(w * rng.uniform(0.0, 1.0)), int(w), 45.0)
              for d in range(n_dm) for w in (np.exp(rng.uniform(0, np.log(l_end))),)]
    x, mu, sg = make_input(n_dm, n, 80, pulses=pulses)
    t = [torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(dev) for a in (x, mu, sg)]
    kw = dict(boxdit_lmax=[6, 10]) if method == "bd" else {}
    wide = spd.search(*t, spd.Config(method, l_end, threshold=thr, **kw), n_out=n_out + 1024)
    r = spd.search(*t, spd.Config(method, l_end, threshold=thr, planes=planes, segment=segment,
                                  step_levels=step_levels, **kw), n_out=n_out)
    torch.cuda.synchronize()
    got = {(int(c["level"]), int(c["dm"]), int(c["start"])) for c in r.candidates_host()}
    barred = 0
    for i in range(r.info.n_levels):
        k, slots = int(r.info.level_shift[i]), int(r.info.plane_slots[i])
        Y = np.full((n_dm + 2, slots + 2), -np.inf, np.float32)
        Y[1:-1, 1:-1] = wide.level(i)[0][:, :slots].cpu().numpy()
        after = wide.level(i)[0][:, slots].cpu().numpy()
        for d in range(n_dm):
            c, m = Y[d + 1, slots], slots - 1
            ok = c > thr and all(c > v for v in (*Y[d, slots - 1:slots + 2], Y[d + 1, slots - 1])) and \
                all(c >= v for v in (Y[d + 1, slots + 1], *Y[d + 2, slots - 1:slots + 2]))
            if ok and slots % 4 != 0 and not c >= after[d]:
                barred += 1
                ok = False
            assert ((i, d, m << k) in got) == ok, (i, k, slots, d, c, after[d])
    assert barred > 3


@pytest.mark.parametrize("method,bound", [("ig1", 14.0), ("bd32", 45.0)])
def test_slots_formed_again_by_whole_waves(dev, method, bound):
    """At a threshold of 2 most chunks find no room for a record and their slots are formed again.  A wave
    that forms a chunk together costs the peak finder a few times what reading planes costs (6 and 16 times
    as measured); lanes that form their own slots one after another cost 23 and 136 times as much."""
    from paper_1910_08324_amd import spd
    g = torch.Generator(device=dev).manual_seed(5)
    x = torch.randn((128, 65536), generator=g, device=dev)
    mu, sg = torch.zeros(128, device=dev), torch.ones(128, device=dev)
    ms, lists = [], []
    for planes in (True, False):
        r = spd.Runner(x, mu, sg, spd.Config(method, 4096, threshold=2.0, planes=planes), cand_cap=1 << 21)
        r.search()
        best = np.inf
        for _ in range(5):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            r.peaks()
            e[1].record()
            torch.cuda.synchronize()
            best = min(best, e[0].elapsed_time(e[1]))
        ms.append(best)
        lists.append(r.result.candidates_host())
    assert np.array_equal(*lists) and len(lists[0]) > 100000
    assert ms[1] <= bound * ms[0], ms


def test_records_of_many_chunks(dev):
    """Candidates only: when nearly every chunk asks for a record's room (a threshold of 2.5) the cascade takes
    a few times as long as when none does, not as long as that many atomics on one counter (3.2
    times as measured, 39 with one counter)."""
    from paper_1910_08324_amd import spd
    g = torch.Generator(device=dev).manual_seed(6)
    x = torch.randn((256, 131072), generator=g, device=dev)
    mu, sg = torch.zeros(256, device=dev), torch.ones(256, device=dev)
    ms = []
    for threshold in (8.0, 2.5):
        r = spd.Runner(x, mu, sg, spd.Config("ig1", 512, threshold=threshold, planes=False))
        r.filter()
        best = np.inf
        for _ in range(5):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            r.filter()
            e[1].record()
            torch.cuda.synchronize()
            best = min(best, e[0].elapsed_time(e[1]))
        ms.append(best)
    assert ms[1] <= 8.0 * ms[0], ms


@pytest.mark.parametrize("slabs", [1, 189, 190, 191, 380, 381, 1023, 1025, 2049, 4099])
def test_lists_do_not_depend_on_groups(dev, slabs):
    """One level and tiles of 256 slots, so a row is a slab: at every step of the slabs a group takes (which
    differ with planes, candidates only and in a batch) the list is the same, and follows the rules."""
    from paper_1910_08324_amd import spd
    x, mu, sg = make_input(slabs, 256, 81, pulses=[synth.Pulse(slabs // 2, 120, 3, 20.0)])
    x[::5, 250:] += 3.0
    kw = dict(method="ig1", l_end=4, threshold=3.0)
    (n0, ref), (n1, rec) = lists(dev, x, mu, sg, 256, 1, **kw)
    assert n0 == n1 == len(ref) > 0 and np.array_equal(ref, rec)
    t = [torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(dev) for a in (x, mu, sg)]
    small = [a[:3] for a in t]
    for planes in (True, False):
        b = spd.Batch([small, t, small], spd.Config(segment=256, step_levels=1, planes=planes, **kw), cand_cap=1 << 16)
        b.search()
        torch.cuda.synchronize()
        assert np.array_equal(b.results[1].candidates_host(), ref)
        assert np.array_equal(b.results[0].candidates_host(), b.results[2].candidates_host())
    R = oplanes.planes(x, mu, sg, ow.method_levels("ig1", 4))
    parity.check_candidates(ref, R, 3.0, what="groups")


@pytest.mark.parametrize("method,l_end", [("bd32", 1024), ("ig3", 1024)])
def test_lookahead_costs_the_filter_nothing(dev, method, l_end):
    """A small block of a dense set, planes and candidates: with look-ahead samples (and fewer slots) the filter
    takes no longer than without, give or take a tenth (evaluating the chunks at the rows' ends again, one
    width after another, made it 1.9 times as long)."""
    from paper_1910_08324_amd import spd
    g = torch.Generator(device=dev).manual_seed(7)
    n_dm, n = 16, 16384
    x = torch.randn((n_dm, n), generator=g, device=dev)
    x[:, n - 3 * l_end:] += 0.5                      # chunks above the threshold at every level's end
    mu, sg = torch.zeros(n_dm, device=dev), torch.ones(n_dm, device=dev)
    runs = [spd.Runner(x, mu, sg, spd.Config(method, l_end, threshold=4.0), n_out=n_out) for n_out in (n, n - l_end + 1)]
    best = [np.inf, np.inf]
    for r in runs:
        r.filter()
    for _ in range(20):
        for i, r in enumerate(runs):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            for _ in range(10):
                r.filter()
            e[1].record()
            torch.cuda.synchronize()
            best[i] = min(best[i], e[0].elapsed_time(e[1]) / 10)
    assert best[1] <= 1.1 * best[0], best


@pytest.mark.parametrize("planes", [True, False])
@pytest.mark.parametrize("method,segment,limit,where", [
    ("ig1", 0, 64, 4096), ("ig1", 256, 64, 256), ("bd4", 1024, 64, 1024), ("exh", 0, 16, 256)])
def test_many_maxima_lift_the_bar_on_the_last_slot(dev, planes, method, segment, limit, where):
    """The last slot of a row, below the evaluated slot after it, is barred up to `limit` local maxima above the
    threshold in its tile (of `where` slots) and a candidate beyond, whatever lies in the other tiles."""
    from paper_1910_08324_amd import spd
    n_out, n = 3 * 1024 + 1021, 4200
    tile0 = (n_out - 1) // where * where
    spots = [s for s in range(4, n_out - 12, 4 if method == "exh" else 8)]   # one maximum each, clear of chunk edges
    inside = [s for s in spots if s >= tile0]
    for count in (0, limit, limit + 1):
        if count > len(inside):
            assert segment == 256                      # (a tile of 256 slots has no room for 65 spikes 8 apart)
            count = len(inside)
        x = np.zeros((3, n), np.float32)
        x[1, n_out] = 30.0                             # slots n_out - 1, n_out: 21 and 30
        x[1, inside[:count]] = 10.0
        x[1, [s for s in spots if s < tile0]] = 10.0   # (other tiles: as many as there are)
        t = [torch.from_numpy(a).to(dev) for a in (x, np.zeros(3, np.float32), np.ones(3, np.float32))]
        l_end = 2 if method == "exh" else 4
        r = spd.search(*t, spd.Config(method, l_end, threshold=9.0, planes=planes, segment=segment), n_out=n_out)
        torch.cuda.synchronize()
        got = {(int(c["level"]), int(c["dm"]), int(c["start"])) for c in r.candidates_host()}
        assert ((0, 1, n_out - 1) in got) == (count > limit), count
        assert {(0, 1, s) for s in inside[:count]} <= got
