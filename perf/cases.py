"""Performance cases: the work this library is used for, through its public entry points.

One pass is one call a program makes with its context, batch or server in
hand: a single argmax round, a whole greedy cover, a batch of covers, or a
burst of served requests.  Cohorts are random draws of the shapes and mutation
profiles of `paper_2603_16721_amd.synth` (heavy-tailed per-gene rates, normal
rates 0.3 x the tumour rates, a few planted combinations), made on the GPU
from the seed.

Every output is a whole number (gene ids, sorted indices, counts, integer
scores, mask words), so results are compared for equality and `exact` has no
64-bit value to give.  The per-depth counters are returned where they are
defined by the input alone (every prune mode but "bound", whose counters depend
on how fast the incumbent rises).
"""
import math
import time

import numpy as np
import torch

from paper_2603_16721_amd import pdfs, synth

ALPHA = (1, 10)


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # The smallest call: one h = 2 round of a small cohort (the h2_G500
        # workload's shape).  Launch and read-back latency is all it costs.
        dict(name="best_h2_g500", call="best", h=2, mode="bound", G=500, n_tumor=200,
             n_normal=100, profile="zipf1.2", density=0.01, planted=3),
        # A whole pair cover of a full-size cohort: the MFMA pair table decides.
        dict(name="wsc_h2_g5000", call="wsc", h=2, mode="bound", G=5000, n_tumor=1000,
             n_normal=400, profile="zipf1.1", density=0.005, planted=8),
        # The h3_G5000 workload (8 planted triples, stop at 95 % covered) in the
        # default prune mode ...
        dict(name="wsc_h3_bound_g5000", call="wsc", h=3, mode="bound", G=5000, n_tumor=1000,
             n_normal=400, profile="zipf1.1", density=0.005, planted=8, target=0.95),
        # ... and as the paper's empty-intersection walk with its counters.
        dict(name="wsc_h3_empty_g5000", call="wsc", h=3, mode="empty", G=5000, n_tumor=1000,
             n_normal=400, profile="zipf1.1", density=0.005, planted=8, target=0.95),
        # The h4_G20000 workload, the paper's scale (G about 20,000): the default
        # mode, and the empty-intersection walk that bench.py times (the largest).
        dict(name="wsc_h4_bound_g20000", call="wsc", h=4, mode="bound", G=20000, n_tumor=1000,
             n_normal=500, profile="lognormal", density=0.0033, planted=10),
        dict(name="wsc_h4_empty_g20000", call="wsc", h=4, mode="empty", G=20000, n_tumor=1000,
             n_normal=500, profile="lognormal", density=0.0033, planted=10),
        # One round for a caller that may not allocate, resuming from a
        # part-covered mask, odd sizes throughout.
        dict(name="noalloc_h4_g3067", call="noalloc", h=4, mode="bound", G=3067, n_tumor=351,
             n_normal=83, profile="zipf1.1", density=0.006, planted=4, uncovered=0.7),
        # More hits than four (the 2-9 hits of the method): one round of the
        # empty-intersection walk, and a whole cover in the default mode.
        dict(name="best_h5_empty_g5000", call="best", h=5, mode="empty", G=5000, n_tumor=1000,
             n_normal=400, profile="zipf1.1", density=0.005, planted=8),
        dict(name="wsc_h5_bound_g5000", call="wsc", h=5, mode="bound", G=5000, n_tumor=1000,
             n_normal=400, profile="zipf1.1", density=0.005, planted=8),
        # Many cohorts at once: mixed sizes and h in {3, 4} as in the batched
        # workload, in both modes.
        dict(name="batch8_bound", call="batch", h=0, mode="bound", G=20000, n_tumor=1200,
             n_normal=500, profile="zipf1.1", density=0.006, planted=4, n=8),
        dict(name="batch6_empty", call="batch", h=0, mode="empty", G=6000, n_tumor=800,
             n_normal=400, profile="zipf1.1", density=0.006, planted=4, n=6),
        # A burst of served requests (h in {2, 3, 4}) submitted from host memory,
        # ingest included, until the last answer is there.
        dict(name="serve12", call="serve", h=0, mode="bound", G=20000, n_tumor=1000,
             n_normal=500, profile="zipf1.1", density=0.005, planted=4, n=12),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["best", "wsc", "wsc", "wsc", "noalloc", "batch", "serve"])
    mode = rng.choice(["bound", "bound", "empty"])
    profile = rng.choice(["zipf1.1", "zipf1.1", "zipf1.2", "lognormal"])
    density = round(rng.uniform(0.003, 0.01), 5)
    n_tumor = _log(rng, 50, 1000 if mode == "empty" else 1200)
    n_normal = rng.choice([_log(rng, 50, 500), _log(rng, 50, 500), rng.randint(1, 64)])
    planted = rng.randint(2, 8)
    case = dict(call=call, mode=mode, n_tumor=n_tumor, n_normal=n_normal, profile=profile,
                planted=planted)
    if call in ("batch", "serve"):
        case["mode"] = mode if call == "batch" else "bound"
        case.update(h=0, n=rng.randint(2, 8), density=min(density, 0.006),
                    G=_log(rng, 1000, 6000 if case["mode"] == "empty" else 20000))
        return case
    h = rng.choice([2, 3, 3, 4, 4, 4] if call == "noalloc" else [1, 2, 3, 3, 4, 4, 4, 5, 6])
    if h >= 5:   # the deep walk's work grows with every depth
        G = _log(rng, 200, 5000)
        density = min(density, 0.005)
        case["mode"] = "bound" if call == "wsc" else mode
    elif mode == "empty" and h == 4:
        G = _log(rng, 200, 20000)
        density = round(min(density, 60.0 / G), 5)   # mutated genes per sample
    else:
        G = _log(rng, 200, 20000)
        density = round(min(density, 100.0 / G), 5)
    case.update(h=h, G=G, density=density)
    if call in ("best", "noalloc") and rng.random() < 0.5:
        case["uncovered"] = round(rng.uniform(0.1, 0.9), 3)
    if call == "wsc" and rng.random() < 0.3:
        case["target"] = round(rng.uniform(0.5, 0.95), 3)
    return case


# ------------------------------------------------------------------ the inputs
def _rates(profile, G, density, rng):
    """Per-gene mutation rates, highest first or in no order."""
    if profile == "lognormal":
        r = synth.lognormal_rates(G, rng)
        return np.minimum(r * (density / r.mean()), synth.LOGNORMAL_CAP)
    return synth.zipf_rates(G, float(profile[4:]), density)


def _pack(bits):
    """bool [G, n] on the GPU -> int64 [G, ceil(n/64)], sample s at bit s & 63 of word s >> 6."""
    G, n = bits.shape
    W = synth.words_for(n)
    by = torch.zeros((G, W * 64), dtype=torch.uint8, device=bits.device)
    by[:, :n] = bits
    weight = torch.tensor([1, 2, 4, 8, 16, 32, 64, 128], dtype=torch.uint8, device=bits.device)
    return (by.view(G, W * 8, 8) * weight).sum(2, dtype=torch.uint8).contiguous().view(torch.int64)


def _cohort(G, n_tumor, n_normal, h, profile, density, planted, seed):
    """Packed tumour and normal rows on the GPU."""
    rng = np.random.Generator(np.random.PCG64(seed))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    rates = _rates(profile, G, density, rng)[rng.permutation(G)]
    r = torch.from_numpy(rates.astype(np.float32)).cuda()[:, None]
    tumor = torch.rand((G, n_tumor), generator=gen, device="cuda") < r
    normal = torch.rand((G, n_normal), generator=gen, device="cuda") < \
        synth.NORMAL_RATE_FACTOR * r
    # planted combinations: rare genes, disjoint, each in samples of its own
    genes = rng.permutation(np.flatnonzero(rates <= np.median(rates)))
    samples = rng.permutation(n_tumor)
    for k in range(planted):
        m = min(int(rng.integers(10, 41)), n_tumor // (2 * planted))
        g, s = genes[k * h:(k + 1) * h], samples[:m]
        samples = samples[m:]
        if len(g) == h and m > 0:
            tumor[torch.from_numpy(g).cuda()[:, None], torch.from_numpy(s).cuda()[None, :]] = True
    return _pack(tumor), _pack(normal)


def _members(case, seed):
    """The cohorts of a batch or of a burst: (tumour, normal, n_tumor, n_normal, h) in host
    memory, the first at the case's full size."""
    out = []
    for i in range(case["n"]):
        # shares of the full size, spread over 0.1 .. 1
        f = 1.0 - 0.9 * (i * 0.618034 % 1.0)
        g = 1.0 - 0.9 * (i * 0.414214 % 1.0)
        G = max(200, int(case["G"] * f))
        nt, nn = max(50, int(case["n_tumor"] * g)), max(1, int(case["n_normal"] * g))
        h = 3 + i % 2 if case["call"] == "batch" else (3, 2, 4, 3)[i % 4]
        T, N = _cohort(G, nt, nn, h, case["profile"], case["density"], case["planted"],
                       seed * 1000 + i)
        out.append((T.cpu().numpy().view(np.uint64), N.cpu().numpy().view(np.uint64), nt, nn, h))
    return out


class _Handle:
    """A batch or server handle, given back with its owner."""

    def __init__(self, handle, destroy):
        self.handle, self._destroy = handle, destroy

    def __del__(self):
        self._destroy(self.handle)


def prepare(case, seed):
    call, mode = case["call"], case["mode"]
    if call in ("batch", "serve"):
        members = _members(case, seed)
        state = dict(case=case, members=members)
        if call == "batch":
            b = pdfs.pdfs_batch_create([m[:4] for m in members], mode)
            state["batch"] = _Handle(b, pdfs.pdfs_batch_destroy)
        else:
            s = pdfs.pdfs_server_create(mode, 0, 0, 8)
            state["server"] = _Handle(s, pdfs.pdfs_server_destroy)
        return state
    T, N = _cohort(case["G"], case["n_tumor"], case["n_normal"], case["h"], case["profile"],
                   case["density"], case["planted"], seed)
    state = dict(case=case, mask=None,
                 solver=pdfs.Solver(T, N, case["n_tumor"], case["n_normal"], mode))
    if "uncovered" in case:
        rng = np.random.Generator(np.random.PCG64([seed, 2]))
        bits = rng.random(case["n_tumor"]) < case["uncovered"]
        state["mask"] = synth.pack_rows(bits[None, :])[0]
    return state


# ------------------------------------------------------------------ one pass
FIELDS = ("tp", "fp", "tn", "score_num", "score_den", "uncovered_before", "newly_covered")


def _rows(rounds, h, most):
    """Chosen combinations, one row each: caller genes, sorted indices, counts and scores; rows
    of -1 up to the `most` rounds that the call can take."""
    out = np.full((most, 2 * h + len(FIELDS)), -1, dtype=np.int64)
    for i, r in enumerate(rounds):
        out[i] = r["genes"] + r["sorted_idx"] + [r[f] for f in FIELDS]
    return out


def _counters(stats, mode):
    if mode == "bound":
        return None
    keys = ("visited", "nonempty", "dfs_visits")
    one = ("rounds", "pair_macs", "dfs_leaves", "dfs_visit_words3", "dfs_visit_words4")
    return np.array([v for k in keys for v in stats[k]] + [stats[k] for k in one],
                    dtype=np.int64)


def run(state):
    case = state["case"]
    call, mode, h = case["call"], case["mode"], case["h"]
    p, q = ALPHA
    if call in ("best", "noalloc"):
        f = state["solver"].best if call == "best" else state["solver"].best_noalloc
        combo, stats = f(h, p, q, state["mask"])
        return {"combo": _rows([combo] if combo else [], h, 1), "counters": _counters(stats, mode)}
    if call == "wsc":
        target = int(math.ceil(case["target"] * case["n_tumor"])) if "target" in case else 0
        rounds, stats, left = state["solver"].wsc(h, p, q, target)
        return {"rounds": _rows(rounds, h, case["n_tumor"]), "uncovered": left.view(np.int64),
                "counters": _counters(stats, mode)}
    members = state["members"]
    if call == "batch":
        res, stats = pdfs.pdfs_batch_run(state["batch"].handle, [m[4] for m in members], p, q,
                                         n_tumors=[m[2] for m in members])
        return {"rounds": [_rows(r, m[4], m[2]) for r, m in zip(res, members)],
                "counters": _counters(stats, mode)}
    srv = state["server"].handle
    tickets = [pdfs.pdfs_server_submit(srv, T, N, nt, nn, hh, p, q) for T, N, nt, nn, hh in members]
    out = []
    for t, m in zip(tickets, members):
        while (answer := pdfs.pdfs_server_poll(srv, t, cap=m[2] + 1)) is None:
            time.sleep(2e-5)
        out.append(_rows(answer[0], m[4], m[2]))
    return {"rounds": out}


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    """Bytes: every cohort's rows read once and its answer (at most a combination per ten
    samples) written once.  Operations: one multiply-add per sample of every pair of genes that
    shares a sample (the co-occurrence counts that every h >= 2 search starts from)."""
    def one(G, nt, nn, h):
        rows = 8 * G * (synth.words_for(nt) + synth.words_for(nn))
        per_sample = case["density"] * G   # mutated genes of a sample, on average
        return (rows + (2 * h + len(FIELDS)) * 8 * max(1, nt // 10),
                2 * nt * per_sample * per_sample / 2 if h > 1 else nt * per_sample)

    if case["call"] in ("batch", "serve"):
        # members average a little over half of the full size in each direction
        b, f = one(case["G"], case["n_tumor"], case["n_normal"], 3)
        k = 1 + 0.3 * (case["n"] - 1)
        return {"bytes": int(b * k), "flops": int(f * k)}
    b, f = one(case["G"], case["n_tumor"], case["n_normal"], case["h"])
    return {"bytes": int(b), "flops": int(f)}


def exact(case, seed):
    """Outputs are whole numbers, compared for equality: no 64-bit value."""
    return None
