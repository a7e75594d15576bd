"""Performance cases of the boxcar single-pulse search: what a user's program has this library do, through its public
entry points, from a few short rows to a whole beam.

A case is a dict of plain values; "kind" selects the path:
  search     the search of one block (spd.Runner / spd.search): IGRID, BoxDIT or exhaustive, planes and candidates or
             candidates alone, with or without a sigma table, with or without look-ahead samples
  batch      many beams of uneven shapes in one set of launches (spd.Batch)
  msd        noise statistics of every row (msd.msd)
  train      one training step of the tile proposal on given tiles (proposal.Labeller, proposal.Network)
  gated      the proposal-gated exhaustive search of a block (proposal.GatedSearch)

prepare() makes what the program has in hand (inputs on the GPU, plan, buffers, weights), run() is one pass, exact() the
same outputs in 64 bits from plain torch.
"""
import ctypes
import math

import numpy as np
import torch

from paper_1910_08324_amd import msd, proposal, spd

DEV = "cuda"
CAND_CAP = 1 << 17


# ------------------------------------------------------------------------------------------------------------------
# The cases
# ------------------------------------------------------------------------------------------------------------------
def search_case(name, method, n_dm, n, l_end, planes=True, rho=False, lookahead=False, runner=True):
    c = {"kind": "search", "method": method, "n_dm": n_dm, "n": n, "l_end": l_end, "planes": planes, "rho": rho,
         "lookahead": lookahead, "runner": runner}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: a few trials of a short block, where launches and host work are what counts
        search_case("ig1_small", "ig1", 8, 5003, 512, runner=False),
        # rows of a length as it comes (no multiple of anything, rows one after another), with the look-ahead samples
        # that a streaming caller gives
        search_case("ig1_ragged", "ig1", 500, 100003, 4096, lookahead=True),
        # the headline workload: a whole beam, planes and candidates
        search_case("ig1_beam", "ig1", 4096, 262144, 8192),
        # a finer width grid with measured (red) noise: the sigma table of every row
        search_case("ig2_rho", "ig2", 1024, 131072, 8192, rho=True),
        # the dense BoxDIT searches: the paper's performance shape, planes and candidates
        search_case("bd16", "bd16", 1024, 131072, 8192),
        # ... and the densest one when the program keeps only the candidates
        search_case("bd32_candidates", "bd32", 512, 131072, 8192, planes=False),
        # many beams of uneven shapes at once, candidates only (what the streaming server and a multi-beam run do)
        {"kind": "batch", "method": "ig1", "l_end": 8192, "name": "batch_uneven",
         "shapes": "512x65536,1003x131072,640x100000,2048x87381,777x262144,1500x70001,3000x65536,256x524288"},
        # the exhaustive search: the small workload of widths 1..256 ...
        search_case("exh_l256", "exh", 64, 65536, 256),
        # ... and long widths, as the reference of every loss figure
        search_case("exh_l8192", "exh", 128, 131072, 8192),
        # noise statistics of a whole beam before its search
        {"kind": "msd", "n_dm": 4096, "n": 262144, "levels": 14, "tau": 3.0, "name": "msd_beam"},
        # a training step of the tile proposal: labels from both searches, forward, backward, Adam
        {"kind": "train", "tiles": 256, "name": "train_step"},
        # the proposal-gated search of a block: features, network, flags, both searches, one candidate list
        {"kind": "gated", "n_dm": 512, "n": 65536, "l_end": 256, "share": 0.25, "name": "gated_block"},
    ]


def log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def block_shape(rng, most, lo_dm=4, lo_n=1024, hi_dm=4096, hi_n=1 << 19):
    """DM trials and samples over their whole ranges, at most `most` values in all; two lengths in three as they come."""
    while True:
        n_dm, n = log_int(rng, lo_dm, hi_dm), log_int(rng, lo_n, hi_n)
        if rng.random() < 1 / 3:
            n = (n + 255) // 256 * 256
        if n_dm * n <= most:
            return n_dm, n


def draw(rng):
    kind = rng.choice(["search", "search", "search", "candidates", "exh", "batch", "msd", "train", "gated"])
    if kind in ("search", "candidates"):
        n_dm, n = block_shape(rng, 1 << 29)
        l_end = log_int(rng, 64, min(16384, n // 2))
        method = rng.choice(["ig1", "ig1", "ig2", "ig3", "bd8", "bd16", "bd32"])
        return search_case(None, method, n_dm, n, l_end, planes=kind == "search", rho=rng.random() < 0.2,
                           lookahead=rng.random() < 0.3, runner=rng.random() < 0.7)
    if kind == "exh":
        while True:
            n_dm, n = block_shape(rng, 1 << 25)
            l_end = log_int(rng, 64, min(8192, n // 2))
            if n_dm * n * l_end <= 128 * 131072 * 8192:
                return search_case(None, "exh", n_dm, n, l_end, planes=rng.random() < 0.7)
    if kind == "batch":
        shapes, room = [], 1 << 28
        for _ in range(rng.randint(2, 12)):
            n_dm, n = block_shape(rng, 1 << 26, lo_dm=64, lo_n=16384)
            if n_dm * n <= room:
                shapes.append("%dx%d" % (n_dm, n))
                room -= n_dm * n
        return {"kind": "batch", "method": rng.choice(["ig1", "ig1", "bd16"]), "l_end": log_int(rng, 256, 8192),
                "shapes": ",".join(shapes)}
    if kind == "msd":
        n_dm, n = block_shape(rng, 1 << 30, lo_n=4096)
        return {"kind": "msd", "n_dm": n_dm, "n": n, "levels": rng.randint(1, min(14, int(math.log2(n)) - 1)),
                "tau": rng.choice([2.5, 3.0, 4.0])}
    if kind == "train":
        return {"kind": "train", "tiles": log_int(rng, 8, 256)}
    return {"kind": "gated", "n_dm": 64 * log_int(rng, 1, 16), "n": 4096 * log_int(rng, 1, 16),
            "l_end": log_int(rng, 64, 512), "share": round(rng.uniform(0.05, 0.6), 2)}


# ------------------------------------------------------------------------------------------------------------------
# Inputs
# ------------------------------------------------------------------------------------------------------------------
def generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def noise_block(n_dm, n, seed, widest, offset=0.0, scale=1.0, pulse_rows=8):
    """White noise with rectangular pulses of SNR 5 to 50, one in every `pulse_rows` rows."""
    x = torch.randn((n_dm, n), generator=generator(seed), device=DEV)
    r = np.random.default_rng(seed)
    for d in r.choice(n_dm, size=min(512, max(1, n_dm // pulse_rows)), replace=False):
        w = int(math.exp(r.uniform(0.0, math.log(max(2, widest)))))
        s = int(r.integers(0, max(1, n - w)))
        x[int(d), s:s + w] += float(r.uniform(5.0, 50.0)) / math.sqrt(w)
    if scale != 1.0 or offset != 0.0:
        x.mul_(scale).add_(offset)
    return x


def rho_table(n_dm, levels, seed):
    """Ratios of a red-noise sigma table: 1 at width 1, growing by up to 10% a level."""
    r = np.random.default_rng(seed + 1)
    t = np.cumprod(np.concatenate([np.ones((n_dm, 1)), 1.0 + 0.1 * r.random((n_dm, levels - 1))], axis=1), axis=1)
    return torch.from_numpy(t.astype(np.float32)).to(DEV)


def search_inputs(case, seed):
    x = noise_block(case["n_dm"], case["n"], seed, case["l_end"] // 2, offset=0.25, scale=1.5)
    mean = torch.full((case["n_dm"],), 0.25, device=DEV)
    sigma = torch.full((case["n_dm"],), 1.5, device=DEV)
    rho = rho_table(case["n_dm"], int(math.log2(case["l_end"])) + 1, seed) if case["rho"] else None
    n_out = max(1, case["n"] - case["l_end"] + 1) if case["lookahead"] else case["n"]
    return x, mean, sigma, rho, n_out


def batch_shapes(case):
    return [tuple(int(v) for v in s.split("x")) for s in case["shapes"].split(",")]


def weights(seed):
    """The proposal network's parameters, by name, as its training starts from them."""
    r = np.random.default_rng(seed)
    return {"W1": r.standard_normal((32, 5, 5)) * math.sqrt(2 / 25), "b1": 0.05 * r.standard_normal(32),
            "W2": r.standard_normal((32, 5, 32)) * math.sqrt(2 / 160), "b2": 0.05 * r.standard_normal(32),
            "W3": r.standard_normal((32, 5, 32)) * math.sqrt(2 / 160), "b3": 0.05 * r.standard_normal(32),
            "wh": r.standard_normal(32) * math.sqrt(1 / 32), "bh": 0.1}


def moments(seed):
    """Adam's moments in the middle of a training."""
    r = np.random.default_rng(seed + 2)
    m = (1e-3 * r.standard_normal(proposal.NPARAMS)).astype(np.float32)
    v = (1e-5 * (0.5 + r.random(proposal.NPARAMS))).astype(np.float32)
    return m, v


ADAM_STEP, LEARNING_RATE = 200, 2e-3
LABEL_L_END, LABEL_SNR, LABEL_MARGIN = 256, 6.0, 0.01


# ------------------------------------------------------------------------------------------------------------------
# prepare, run
# ------------------------------------------------------------------------------------------------------------------
def candidate_views(cand, count):
    """The candidate list as its whole-number columns and its SNRs (the entries after the last one stay zero)."""
    rec = cand.zero_().view(torch.int32).view(-1, 6)
    return {"cand": rec[:, :5], "cand_snr": rec[:, 5].view(torch.float32), "count": count}


def plane_views(res):
    lev = [res.level(i) for i in range(res.info.n_levels)]
    return {"Y": [y for y, _ in lev], "W": [w for _, w in lev]}


def prepare(case, seed):
    return {"search": prepare_search, "batch": prepare_batch, "msd": prepare_msd, "train": prepare_train,
            "gated": prepare_gated}[case["kind"]](case, seed)


def run(state):
    return state["run"](state)


def prepare_search(case, seed):
    x, mean, sigma, rho, n_out = search_inputs(case, seed)
    cfg = spd.Config(case["method"], case["l_end"], threshold=5.0, planes=case["planes"], rho=rho)
    r = spd.Runner(x, mean, sigma, cfg, n_out=n_out, cand_cap=CAND_CAP)
    outputs = candidate_views(r.result.cand, r.result.count)
    if case["planes"]:
        outputs.update(plane_views(r.result))
    return {"run": run_runner if case["runner"] else run_search, "runner": r, "cfg": cfg, "n_out": n_out,
            "outputs": outputs}


def run_runner(s):
    s["runner"].search()
    return s["outputs"]


def run_search(s):
    r = s["runner"]
    spd.search(r.x, r.mean, r.sigma, s["cfg"], n_out=s["n_out"], out=r.result, workspace=r.workspace)
    return s["outputs"]


def prepare_batch(case, seed):
    beams = []
    for i, (n_dm, n) in enumerate(batch_shapes(case)):
        x = noise_block(n_dm, n, 1000 * seed + i, case["l_end"] // 2)
        beams.append((x, torch.zeros(n_dm, device=DEV), torch.ones(n_dm, device=DEV)))
    b = spd.Batch(beams, spd.Config(case["method"], case["l_end"], threshold=5.0, planes=False), cand_cap=CAND_CAP)
    return {"run": run_batch, "batch": b, "outputs": [candidate_views(r.cand, r.count) for r in b.results]}


def run_batch(s):
    s["batch"].search()
    return s["outputs"]


def prepare_msd(case, seed):
    x = noise_block(case["n_dm"], case["n"], seed, 4096, offset=0.25, scale=1.5)
    b = ctypes.c_int64()
    spd._check(msd.lib().spd_msd_workspace(case["n_dm"], case["n"], case["levels"], ctypes.byref(b)), "spd_msd_workspace")
    return {"run": run_msd, "x": x, "levels": case["levels"], "tau": case["tau"],
            "workspace": torch.empty(int(b.value), dtype=torch.uint8, device=DEV)}


def run_msd(s):
    mean, sigma, rho, level_sd, passes = msd.msd(s["x"], s["levels"], tau=s["tau"], workspace=s["workspace"],
                                                 with_passes=True)
    return {"mean": mean, "sigma": sigma, "rho": rho, "level_sd": level_sd, "passes": passes}


def train_tiles(case, seed):
    return noise_block(case["tiles"] * proposal.TILE_ROWS, proposal.TILE_LEN, seed, 64, pulse_rows=64)


def prepare_train(case, seed):
    net = proposal.Network(proposal.pack(weights(seed)), max_tiles=case["tiles"])
    m, v = moments(seed)
    net.m.copy_(torch.from_numpy(m))
    net.v.copy_(torch.from_numpy(v))
    net.step = ADAM_STEP
    lab = proposal.Labeller(train_tiles(case, seed), l_end=LABEL_L_END, threshold=LABEL_SNR, margin=LABEL_MARGIN)
    return {"run": run_train, "net": net, "lab": lab, "logits": torch.empty(case["tiles"], device=DEV)}


def run_train(s):
    net, lab = s["net"], s["lab"]
    lab.run()
    net.backward(lab.feat, lab.labels, lab.n_tiles, s["logits"])
    net.adam(LEARNING_RATE)
    return {"lossy_max": lab.lossy_max, "exh_max": lab.exh_max, "labels": lab.labels, "logits": s["logits"],
            "loss": net.loss, "grads": net.grads, "params": net.params, "m": net.m, "v": net.v}


def gated_inputs(case, seed):
    return noise_block(case["n_dm"], case["n"], seed, 64, pulse_rows=4)


def prepare_gated(case, seed):
    x = gated_inputs(case, seed)
    mean, sigma = torch.zeros(case["n_dm"], device=DEV), torch.ones(case["n_dm"], device=DEV)
    tiles = (case["n_dm"] // proposal.TILE_ROWS) * (case["n"] // proposal.TILE_LEN)
    net = proposal.Network(proposal.pack(weights(seed)), max_tiles=tiles)
    g = proposal.GatedSearch(net, x, mean, sigma, l_end=case["l_end"], cand_cap=CAND_CAP)
    # the flag threshold that the program has chosen: so many of the tiles, half way between two logits
    g.propose()
    lg = np.sort(g.logits.cpu().numpy().astype(np.float64))[::-1]
    k = min(len(lg), max(1, round(case["share"] * len(lg))))
    g.logit_threshold = float(lg[k - 1] + lg[k]) / 2 if k < len(lg) else float(lg[-1]) - 1.0
    for t in (g.out.lossy.snr, g.out.exh.snr, g.out.lossy.width, g.out.exh.width):
        t.zero_()
    outputs = {"logits": g.logits, "flag": g.flag, "lossy": plane_views(g.out.lossy), "exh": plane_views(g.out.exh)}
    outputs.update(candidate_views(g.out.cand, g.out.count))
    return {"run": run_gated, "search": g, "outputs": outputs}


def run_gated(s):
    s["search"].run()
    return s["outputs"]


# ------------------------------------------------------------------------------------------------------------------
# The work that a pass cannot do without
# ------------------------------------------------------------------------------------------------------------------
def level_sets(method, l_end):
    """[(level k, [widths in samples])] of a search, from the paper's width equations."""
    if method == "exh":
        return [(0, list(range(1, l_end + 1)))]
    if method.startswith("bd"):
        out, off, k, L = [], 0, 0, int(method[2:])
        while off + (1 << k) <= l_end:
            out.append((k, [off + (m << k) for m in range(1, L + 1) if off + (m << k) <= l_end]))
            off += L << k
            k += 1
        return out
    d = int(method[2:])
    P = 2 << d
    w0 = sorted({W + q * max(1, W >> d) for W in (1 << j for j in range(d + 2)) for q in range(1 << d)
                 if W <= l_end and q * max(1, W >> d) < W and W + q * max(1, W >> d) <= l_end})
    out, k = [(0, w0)], 1
    while P << k <= l_end:
        out.append((k, [(P + q * (P >> d)) << k for q in range(1 << d) if (P + q * (P >> d)) << k <= l_end]))
        k += 1
    return out


def search_work(method, n_dm, n, n_out, l_end, planes):
    """Samples read once, planes (SNR and width) written once; an add, a multiply and a comparison per start and width."""
    levels = level_sets(method, l_end)
    slots = [n_dm * -(-n_out // (1 << k)) for k, _ in levels]
    return {"bytes": 4.0 * n_dm * n + (6.0 * sum(slots) if planes else 0.0),
            "flops": 3.0 * sum(s * len(w) for s, (_, w) in zip(slots, levels))}


def network_flops(tiles):
    return 2.0 * tiles * 64 * 256 * 32 * (5 * 5 + 5 * 32 + 5 * 32 + 1)


def work(case):
    kind = case["kind"]
    if kind == "search":
        n_out = max(1, case["n"] - case["l_end"] + 1) if case["lookahead"] else case["n"]
        return search_work(case["method"], case["n_dm"], case["n"], n_out, case["l_end"], case["planes"])
    if kind == "batch":
        parts = [search_work(case["method"], d, n, n, case["l_end"], False) for d, n in batch_shapes(case)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    if kind == "msd":
        # two estimates at least of every level's values (twice the samples in all), four operations a value
        return {"bytes": 4.0 * case["n_dm"] * case["n"], "flops": 16.0 * case["n_dm"] * case["n"]}
    if kind == "train":
        rows, n = case["tiles"] * 64, 4096
        f = sum(search_work(m, rows, n, n, LABEL_L_END, False)["flops"] for m in ("ig1", "exh"))
        return {"bytes": 4.0 * rows * n + 4.0 * 8 * proposal.NPARAMS, "flops": f + 3.0 * network_flops(case["tiles"])}
    tiles = case["n_dm"] * case["n"] // (64 * 4096)
    lossy = search_work("ig1", case["n_dm"], case["n"], case["n"], case["l_end"], True)
    exh = search_work("exh", case["n_dm"], case["n"], case["n"], case["l_end"], True)
    return {"bytes": lossy["bytes"] + case["share"] * 6.0 * case["n_dm"] * case["n"],
            "flops": lossy["flops"] + case["share"] * exh["flops"] + network_flops(tiles)}


# ------------------------------------------------------------------------------------------------------------------
# The outputs in 64 bits
# ------------------------------------------------------------------------------------------------------------------
NO_CAND = {"cand": None, "cand_snr": None, "count": None}


def sigma_factor(rho, L):
    """rho(L), linear in log2 L between the table's powers of two and held above them."""
    if rho is None:
        return 1.0
    a = math.log2(L)
    k = min(int(a + 1e-12), rho.shape[1] - 1)
    lo, hi = rho[:, k].double(), rho[:, min(k + 1, rho.shape[1] - 1)].double()
    return (lo + (a - k) * (hi - lo))[:, None]


def exact_planes(x, mean, sigma, levels, n_out, rho=None, rows=256):
    """[SNR plane] per level: the maximum over the level's widths of the normalised boxcar sums."""
    n_dm, n = x.shape
    out = [torch.empty((n_dm, -(-n_out // (1 << k))), dtype=torch.float64, device=x.device) for k, _ in levels]
    for d in range(0, n_dm, rows):
        z = (x[d:d + rows].double() - mean[d:d + rows, None].double()) / sigma[d:d + rows, None].double()
        P = torch.zeros((z.shape[0], n + 1), dtype=torch.float64, device=x.device)
        torch.cumsum(z, dim=1, out=P[:, 1:])
        r = None if rho is None else rho[d:d + rows]
        for (k, widths), Y in zip(levels, out):
            best = torch.full((z.shape[0], Y.shape[1]), -math.inf, dtype=torch.float64, device=x.device)
            for L in widths:
                if L > n:
                    continue
                m = min(Y.shape[1], ((n - L) >> k) + 1)
                s = P[:, L:L + ((m - 1) << k) + 1:1 << k] - P[:, :((m - 1) << k) + 1:1 << k]
                s /= math.sqrt(L) * sigma_factor(r, L)
                torch.maximum(best[:, :m], s, out=best[:, :m])
            Y[d:d + rows] = best
    return out


def exact_search(case, seed):
    if not case["planes"]:
        return None
    x, mean, sigma, rho, n_out = search_inputs(case, seed)
    Y = exact_planes(x, mean, sigma, level_sets(case["method"], case["l_end"]), n_out, rho)
    return dict(NO_CAND, Y=Y, W=[None] * len(Y))


def exact_msd(case, seed):
    x = noise_block(case["n_dm"], case["n"], seed, 4096, offset=0.25, scale=1.5)
    K, means, sds = case["levels"], [], []
    y = x
    for k in range(K):
        if k:
            y = y[:, :y.shape[1] // 2 * 2].double().reshape(y.shape[0], -1, 2).sum(dim=2)
        part = [rejected(y[d:d + 512].double(), case["tau"], 10) for d in range(0, y.shape[0], 512)]
        means.append(torch.cat([p[0] for p in part]))
        sds.append(torch.cat([p[1] for p in part]))
    sd = torch.stack(sds, dim=1)
    width = torch.tensor([math.sqrt(2.0 ** k) for k in range(K)], dtype=torch.float64, device=x.device)
    return {"mean": means[0], "sigma": sds[0], "rho": sd / (width * sd[:, :1]), "level_sd": sd, "passes": None}


def rejected(y, tau, max_iter):
    """Mean and standard deviation of each row after point-wise rejection until the kept count stays."""
    n = torch.full((y.shape[0],), float(y.shape[1]), dtype=torch.float64, device=y.device)
    m = y.mean(dim=1)
    sd = ((y - m[:, None]).square().sum(dim=1) / (n - 1)).sqrt()
    live = torch.ones_like(n, dtype=torch.bool)
    for _ in range(max_iter):
        d = y - m[:, None]
        d = torch.where(d.abs() <= (tau * sd)[:, None], d, torch.nan)
        cnt = (~d.isnan()).sum(dim=1).double()
        live &= (cnt != n) & (cnt >= 2)
        off = d.nansum(dim=1) / cnt
        var = (d - off[:, None]).square().nansum(dim=1) / (cnt - 1)
        m, sd, n = torch.where(live, m + off, m), torch.where(live, var.sqrt(), sd), torch.where(live, cnt, n)
        if not live.any():
            break
    return m, sd


def exact_logits(x, p):
    """Tile logits [tiles] of tiles x [tiles * 64][4096] under the network's parameters p."""
    f = []
    for k in range(4, 9):
        y = x.view(x.shape[0], -1, 1 << k).sum(dim=2) / 2.0 ** (k / 2)
        f.append(y.repeat_interleave(1 << (k - 4), dim=1))
    a = torch.stack(f, dim=1)
    for W, b in (("W1", "b1"), ("W2", "b2"), ("W3", "b3")):
        # one product over (tap, channel) per position
        pad = torch.nn.functional.pad(a, (2, 2))
        taps = torch.cat([pad[:, :, t:t + 256] for t in range(5)], dim=1)
        a = (p[W].reshape(32, -1) @ taps + p[b][:, None]).relu()
    s = (p["wh"] @ a + p["bh"]).view(-1, 64 * 256)
    return torch.logsumexp(s, dim=1) - math.log(64 * 256)


def exact_params(seed):
    return {k: torch.tensor(np.asarray(v, np.float32), dtype=torch.float64, device=DEV, requires_grad=True)
            for k, v in weights(seed).items()}


def packed(p):
    """The parameter vector's layout: W1's input channels padded to 8, three unused values at the end."""
    W1 = torch.zeros((32, 5, 8), dtype=torch.float64, device=DEV)
    W1[:, :, :5] = p["W1"]
    flat = [W1.reshape(-1)] + [p[k].reshape(-1) for k in ("b1", "W2", "b2", "W3", "b3", "wh", "bh")]
    return torch.cat(flat + [torch.zeros(3, dtype=torch.float64, device=DEV)])


def exact_train(case, seed):
    x = train_tiles(case, seed)
    rows, n = x.shape
    zero, one = torch.zeros(rows, device=DEV), torch.ones(rows, device=DEV)
    top = []
    for method in ("ig1", "exh"):
        Y = exact_planes(x, zero, one, level_sets(method, LABEL_L_END), n, rows=2048)
        top.append(torch.stack([y.reshape(case["tiles"], -1).amax(dim=1) for y in Y]).amax(dim=0))
    labels = ((top[1] > LABEL_SNR) & (top[1] > (1 + LABEL_MARGIN) * top[0])).double()
    p = exact_params(seed)
    logits, loss = [], 0.0
    for t in range(0, case["tiles"], 16):
        lg = exact_logits(x[64 * t:64 * (t + 16)].double(), p)
        part = torch.nn.functional.binary_cross_entropy_with_logits(lg, labels[t:t + 16], reduction="sum") / case["tiles"]
        part.backward()
        loss += float(part.detach())
        logits.append(lg.detach())
    g = packed({k: v.grad for k, v in p.items()})
    m, v = (torch.from_numpy(a).to(DEV).double() for a in moments(seed))
    m, v, t = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g, ADAM_STEP + 1
    w = packed({k: q.detach() for k, q in p.items()})
    w = w - LEARNING_RATE * (m / (1 - 0.9 ** t)) / ((v / (1 - 0.999 ** t)).sqrt() + 1e-8)
    return {"lossy_max": top[0], "exh_max": top[1], "labels": labels, "logits": torch.cat(logits),
            "loss": torch.tensor([loss], dtype=torch.float64), "grads": g, "params": w, "m": m, "v": v}


def exact_gated(case, seed):
    x = gated_inputs(case, seed)
    n_dm, n = x.shape
    zero, one = torch.zeros(n_dm, device=DEV), torch.ones(n_dm, device=DEV)
    Y = exact_planes(x, zero, one, level_sets("ig1", case["l_end"]), n)
    with torch.no_grad():
        p = exact_params(seed)
        logits = torch.cat([exact_logits(x[:, c:c + 4096].contiguous().double(), p) for c in range(0, n, 4096)])
    return dict(NO_CAND, logits=logits, flag=None, lossy={"Y": Y, "W": [None] * len(Y)},
                exh={"Y": [None], "W": [None]})


def exact(case, seed):
    f = {"search": exact_search, "msd": exact_msd, "train": exact_train, "gated": exact_gated}.get(case["kind"])
    return f(case, seed) if f else None
