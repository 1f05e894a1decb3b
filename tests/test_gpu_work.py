"""The work counters of bound-pruned runs (pdfs_stats): exact where nothing can be
pruned (every normal carries every gene, so that no score bound reaches q * N_n),
and inside the empty-intersection walk's counts elsewhere; and the leaves whose
false positives are counted, which the empty-intersection mode reports too."""
import numpy as np
import pytest

from oracle import cpu
from paper_2603_16721_amd import synth
from tests.helpers import mask_of_bits
from tests.test_gpu_parity import pdfs  # noqa: F401

pytestmark = pytest.mark.gpu


def _formed(rows, perm, G, h):
    """Nodes formed and non-empty per depth of one round without pruning: every pair
    of active genes inside Alg. 2's bounds, then below a node the later ones of its
    parent's non-empty candidates."""
    act = [(i, rows[g]) for i, g in enumerate(perm) if rows[g]]
    vis, ne = [0] * (h + 1), [0] * (h + 1)

    def below(depth, inter, cand):   # cand: (samples) of the parent's later candidates
        vis[depth] += len(cand)
        kept = [x & inter for x in cand if x & inter]
        ne[depth] += len(kept)
        if depth < h:
            for i, x in enumerate(kept):
                below_entry(depth + 1, x, kept[i + 1:])

    def below_entry(depth, inter, cand):
        if cand:
            below(depth, inter, cand)

    for i, (sa, a) in enumerate(act):
        if sa > G - h:
            break
        for j in range(i + 1, len(act)):
            sb, b = act[j]
            if sb > G - h + 1:
                break
            if a & b:
                ne[2] += 1
                if h > 2:
                    below(3, a & b, [x for _, x in act[j + 1:]])
    vis[1] = G - h + 1
    ne[1] = sum(1 for s, _ in act if s <= G - h)
    vis[2] = sum(G - h + 1 - s for s, _ in act if s <= G - h)
    return vis, ne


EXACT = [
    # core genes, samples, density, one-sample genes, h
    (30, 40, 0.25, 20, 2),
    (60, 90, 0.12, 100, 3),      # leaves from the slices
    (24, 300, 0.3, 60, 3),       # and from the rows
    (34, 70, 0.25, 120, 4),      # lists one candidate a lane
    (90, 40, 0.15, 200, 4),      # lists in LDS
    (24, 200, 0.55, 60, 4),      # masks of several words
    (80, 130, 0.55, 200, 4),     # the general walk
    (26, 60, 0.3, 60, 5),
    (20, 60, 0.35, 60, 6),
    (16, 50, 0.4, 60, 8),
]


@pytest.mark.parametrize("case", EXACT, ids=[f"G{c[0]}_nt{c[1]}_h{c[4]}" for c in EXACT])
def test_unpruned_round_is_counted_exactly(pdfs, case):  # noqa: F811
    core, nt, d, tail, h = case
    G, nn = core + tail, 64
    tumor = np.zeros((G, nt), bool)
    tumor[:core] = synth.random_tiny(5, core, nt, 1, d, h).tumor
    tumor[core + np.arange(tail), (np.arange(tail) * 7) % nt] = True
    T, N = synth.pack_rows(tumor), synth.pack_rows(np.ones((G, nn), bool))
    rows = [sum(1 << int(s) for s in np.flatnonzero(tumor[g])) for g in range(G)]
    vis, ne = _formed(rows, list(cpu.order(T, N)), G, h)
    with pdfs.Solver(T, N, nt, nn, "bound") as s:
        calls = [lambda: s.wsc(h, 1, 1000, 0, 1)[1]]   # (single rounds of h = 2 are the table's)
        if h > 2:
            calls.append(lambda: s.best(h, 1, 1000)[1])
        if h in (3, 4):
            calls.append(lambda: s.best_noalloc(h, 1, 1000)[1])
        for call in calls:
            st = call()
            assert st["visited"][1:3] == vis[1:3]
            assert st["nonempty"][1:h + 1] == ne[1:]
            if h > 2:
                assert st["visited"][3:h + 1] == vis[3:]
                assert st["bound_pruned"] == [0] * 10
            if h in (3, 4):
                assert st["dfs_visits"][3:h + 1] == vis[3:]
                assert st["dfs_leaves"] == st["dfs_fp_leaves"] == ne[h]
                w = (nt + 63) // 64
                assert st["dfs_visit_words3"] == vis[3] * w
            act = sum(1 for r in rows if r)
            assert 0 < st["pair_macs"] <= act * (act - 1) // 2 * nt
        if h in (3, 4):
            s.set_prune_mode("empty")
            st = s.wsc(h, 1, 1000, 0, 5)[1]
            assert 0 < st["dfs_fp_leaves"] <= st["dfs_leaves"]


@pytest.mark.parametrize("G,nt,d,h", [(300, 200, 0.03, 2), (400, 300, 0.03, 3), (160, 200, 0.06, 4),
                                      (90, 150, 0.12, 5), (70, 100, 0.12, 6)])
def test_pruned_run_counts(pdfs, G, nt, d, h):  # noqa: F811
    I = synth.random_tiny(19, G, nt, 40, d, h)
    T, N = I.packed()
    mask = mask_of_bits(np.arange(nt) % 4 != 0)
    with pdfs.Solver(T, N, nt, 40, "bound") as s:
        for u in (None, mask):
            s.set_prune_mode("bound")
            _, b, _ = s.wsc(h, 1, 10, 0, 0, u)
            assert b["rounds"] > 2
            s.set_prune_mode("empty")
            _, e, _ = s.wsc(h, 1, 10, 0, 0, u)
            for l in range(1, h + 1):
                assert 0 < b["nonempty"][l] <= b["visited"][l]
                assert b["nonempty"][l] <= e["nonempty"][l]
                # (candidates past a depth's loop bound are formed with the others)
                assert b["visited"][l] <= e["visited"][l] + e["nonempty"][max(l - 1, 1)] * h
                assert b["bound_pruned"][l] <= b["nonempty"][l]
            assert b["bound_pruned"][h] == 0
            assert h == 2 or b["bound_pruned"][2] > 0
            assert 0 < b["pair_macs"] <= e["pair_macs"]
            if h in (3, 4):
                assert b["dfs_visits"][3:] == b["visited"][3:]
                assert b["dfs_leaves"] == b["nonempty"][h]
                # (none where no normal carries a leaf's first h - 1 genes)
                assert b["dfs_fp_leaves"] <= b["dfs_leaves"]
                assert e["dfs_fp_leaves"] <= e["dfs_leaves"]
                assert b["dfs_visits"][3] <= b["dfs_visit_words3"] <= b["dfs_visits"][3] * ((nt + 63) // 64)
