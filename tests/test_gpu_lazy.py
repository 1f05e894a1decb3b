"""Lazy rounds (k_lazy.hip) and the counters made after them (k_count.hip) at
the edges of their paths, against the oracle:
pairs with more samples than one mask word (the general walk), more candidates
than a level list holds, every list depth, candidate words past one wave, and
runs resumed from a mask on the same context.  Results are whole numbers, so
the comparison is equality."""
import time

import numpy as np
import pytest

from oracle import cpu
from paper_2603_16721_amd import synth
from tests.helpers import mask_of_bits
from tests.test_gpu_parity import _counters_equal, _same_rounds, pdfs  # noqa: F401

pytestmark = pytest.mark.gpu

EDGES = [
    # G, n_tumor, n_normal, density, h, alpha, max_rounds
    (50, 30, 10, 0.3, 2, (1, 10), 0),
    (300, 70, 33, 0.5, 3, (1, 10), 0),       # leaves straight from the slices
    (300, 1280, 20, 0.3, 3, (2, 3), 3),      # 11 bit slices
    (70, 200, 60, 0.5, 4, (1, 10), 0),       # more than 64 samples below a pair
    (330, 12, 40, 0.6, 4, (1, 10), 2),       # more than 256 candidates, few samples
    (64, 64, 5, 1.0, 4, (1, 10), 0),         # every row full: exactly 64 samples
    (65, 65, 5, 1.0, 5, (1, 10), 0),         # every row full: 65
    (130, 400, 20, 0.4, 5, (1, 10), 2),
    (40, 150, 64, 0.55, 6, (1, 10), 0),
    (34, 200, 40, 0.6, 9, (1, 10), 2),
    (9, 40, 512, 0.7, 9, (3, 1), 0),         # one combination
    (4200, 30, 40, 0.02, 4, (1, 10), 2),     # more than 64 candidate words
]


@pytest.mark.parametrize("case", EDGES, ids=[f"G{c[0]}_nt{c[1]}_h{c[4]}" for c in EDGES])
@pytest.mark.parametrize("mode", ["bound", "empty"])
def test_lazy_edges(pdfs, case, mode):  # noqa: F811
    G, nt, nn, d, h, (p, q), mr = case
    I = synth.random_tiny(31, G, nt, nn, d, h, alpha=(p, q))
    T, N = I.packed()
    mask = mask_of_bits(np.arange(nt) % 3 != 0)
    with pdfs.Solver(T, N, nt, nn, mode) as s:
        for u in (None, mask):
            exp = cpu.wsc(T, N, nt, nn, h, p, q, mode=mode, max_rounds=mr, U0=u)
            got, st, final = s.wsc(h, p, q, 0, mr, u)
            _same_rounds(got, exp.rounds)
            assert np.array_equal(final, exp.final_uncovered)
            if mode == "empty":
                _counters_equal(st, exp.counters, h)


# The allocation-free lazy round lays the transposed rows and the general walk's
# bitmaps over the unpacked rows: one to three row words, and wider.
@pytest.mark.parametrize("G,nt", [(70, 50), (600, 64), (4200, 100), (900, 130), (700, 700)])
@pytest.mark.parametrize("h", [3, 4])
def test_noalloc_lazy(pdfs, G, nt, h):  # noqa: F811
    I = synth.random_tiny(77, G, nt, 60, min(0.4, 12.0 / G + 0.02), h)
    T, N = I.packed()
    with pdfs.Solver(T, N, nt, 60, "bound") as s:
        for u in (None, mask_of_bits(np.arange(nt) % 4 != 1)):
            ref, _ = s.best(h, 1, 10, u)
            got, _ = s.best_noalloc(h, 1, 10, u)
            assert got == ref


# Pair lists made from the genes' samples: genes at the edges of the slice widths
# (3 | 4, 15 | 16, 127 | 128 samples), spans of 64 words with more pairs than a wave
# stages, more genes than the launch has waves, two genes, and lists regrown from 64.
@pytest.mark.parametrize("G,nt,per_gene,heavy", [
    (2, 64, 1, (64,)), (63, 64, 2, (3, 4)), (65, 65, 1, (65,)),
    (700, 300, 1, (3, 4, 15, 16, 127, 128, 300)),
    (4200, 600, 9, (600,)),
    (9000, 1280, 1, (1280, 127, 128)),
])
@pytest.mark.parametrize("mode", ["bound", "empty"])
def test_pair_lists_by_samples(pdfs, G, nt, per_gene, heavy, mode):  # noqa: F811
    rng = np.random.Generator(np.random.PCG64(91))
    rows = np.zeros((G, nt), bool)
    for g in range(G):
        k = heavy[g] if g < len(heavy) else per_gene
        rows[g, rng.choice(nt, k, replace=False)] = True
    T = synth.pack_rows(rows)
    N = synth.pack_rows(rng.random((G, 30)) < 0.05)
    # (the oracle's empty-mode walk of h = 3 takes minutes at the larger sizes)
    for h in range(2, min(G, 2 if mode == "empty" and G > 1000 else 3) + 1):
        exp = cpu.wsc(T, N, nt, 30, h, 1, 10, mode=mode, max_rounds=3)
        for cap in (0, 64):
            with pdfs.Solver(T, N, nt, 30, mode, pair_cap=cap) as s:
                got, st, final = s.wsc(h, 1, 10, 0, 3)
                _same_rounds(got, exp.rounds)
                assert np.array_equal(final, exp.final_uncovered)
                if mode == "empty":
                    _counters_equal(st, exp.counters, h)


# A server budget that holds a walked cover of h = 2 but not the lazy rounds' 19 MB
# of pairs: the request is accepted and solved.
@pytest.mark.parametrize("budget", [8 << 20, 1 << 30])
def test_served_h2_tight_budget(pdfs, budget):  # noqa: F811
    I = synth.random_tiny(45, 1500, 200, 40, 0.02, 2)
    T, N = I.packed()
    exp = cpu.wsc(T, N, 200, 40, 2, 1, 10, mode="bound")
    srv = pdfs.pdfs_server_create("bound", 0, budget, 2)
    try:
        t = pdfs.pdfs_server_submit(srv, T, N, 200, 40, 2, 1, 10)
        deadline = time.time() + 60
        r = None
        while r is None and time.time() < deadline:
            r = pdfs.pdfs_server_poll(srv, t, cap=201)
        _same_rounds(r[0], exp.rounds)
    finally:
        pdfs.pdfs_server_destroy(srv)
