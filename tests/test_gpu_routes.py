"""Lazy and walked rounds on both sides of the choice between them (lazy_pays),
against the oracle: dense and very small cohorts, whose rounds are walked, and
cohorts whose density sits in a few genes, whose lazy rounds reach the general
walk, the lists in LDS and every slice width.  Results are whole numbers, so the
comparison is equality.  A timed context tells the ways apart: the pair list is
made once per run of lazy rounds, once per walked round."""
import time

import numpy as np
import pytest

from oracle import cpu
from paper_2603_16721_amd import synth
from tests.helpers import mask_of_bits
from tests.test_gpu_parity import _counters_equal, _same_rounds, pdfs  # noqa: F401

pytestmark = pytest.mark.gpu


def _cohort(G, nt, nn, d, h, tail=0):
    """Even density d, then `tail` genes of one tumour sample each."""
    I = synth.random_tiny(57, G, nt, nn, d, h)
    tumor, normal = I.tumor, I.normal
    if tail:
        more = np.zeros((tail, nt), bool)
        more[np.arange(tail), (np.arange(tail) * 7) % nt] = True
        tumor = np.vstack([tumor, more])
        normal = np.vstack([normal, np.zeros((tail, nn), bool)])
    return synth.pack_rows(tumor), synth.pack_rows(normal)


def _check_wsc(s, T, N, nt, nn, h, mode, mr, u, per_round):
    exp = cpu.wsc(T, N, nt, nn, h, 1, 10, mode=mode, max_rounds=mr, U0=u)
    got, st, final = s.wsc(h, 1, 10, 0, mr, u)
    _same_rounds(got, exp.rounds)
    assert np.array_equal(final, exp.final_uncovered)
    if mode == "empty":
        _counters_equal(st, exp.counters, h)
    if per_round is not None:
        assert len(got) > 1
        assert st["kernel_launches"][0] == (len(got) if per_round else 1)


WALKED = [
    # G, n_tumor, n_normal, density, h, max_rounds, modes
    (4800, 70, 10, 0.16, 2, 5, ("bound", "empty")),
    (520, 600, 50, 0.5, 3, 5, ("bound", "empty")),
    (60, 300, 60, 0.5, 4, 8, ("bound", "empty")),
    (300, 520, 30, 0.4, 4, 5, ("bound",)),
    (100, 300, 40, 0.5, 5, 5, ("bound",)),
    (98, 270, 400, 0.5, 6, 5, ("bound",)),
]


@pytest.mark.parametrize("case", WALKED, ids=[f"G{c[0]}_nt{c[1]}_h{c[4]}" for c in WALKED])
def test_dense_covers_walk(pdfs, case):  # noqa: F811
    G, nt, nn, d, h, mr, modes = case
    T, N = _cohort(G, nt, nn, d, h)
    for mode in modes:
        for cap in (0, 64):
            with pdfs.Solver(T, N, nt, nn, mode, time_kernels=True, pair_cap=cap) as s:
                _check_wsc(s, T, N, nt, nn, h, mode, mr, None, per_round=True if cap == 0 else None)


@pytest.mark.parametrize("case", WALKED[1:4], ids=[f"G{c[0]}_nt{c[1]}_h{c[4]}" for c in WALKED[1:4]])
@pytest.mark.parametrize("cap", [0, 64])
def test_dense_covers_walk_captured(pdfs, case, cap):  # noqa: F811
    """Rounds replayed from captured graphs, runs in a row, from several masks."""
    import torch
    G, nt, nn, d, h, mr, modes = case
    T, N = _cohort(G, nt, nn, d, h)
    stream = torch.cuda.Stream()
    mask = mask_of_bits(np.arange(nt) % 8 != 0)
    for mode in modes:
        ctx = pdfs.pdfs_create(T, N, nt, nn, mode, 0, stream.cuda_stream, pdfs.PDFS_OPT_GRAPHS, cap)
        try:
            for u in (None, mask, None):
                exp = cpu.wsc(T, N, nt, nn, h, 1, 10, mode=mode, max_rounds=mr, U0=u)
                got, st, _ = pdfs.pdfs_wsc_run(ctx, h, 1, 10, 0, mr, u)
                _same_rounds(got, exp.rounds)
                if mode == "empty":
                    _counters_equal(st, exp.counters, h)
        finally:
            pdfs.pdfs_destroy(ctx)


# single rounds and covers of few genes or samples: walked and lazy in turn as the
# mask shrinks and the mode changes on one context
@pytest.mark.parametrize("G,nt,d,h", [(40, 100, 0.1, 5), (12, 30, 0.1, 3), (30, 60, 0.05, 6),
                                      (150, 500, 0.15, 4), (420, 300, 0.08, 3), (64, 90, 0.2, 5)])
def test_modes_and_masks_in_turn(pdfs, G, nt, d, h):  # noqa: F811
    nn = 40
    T, N = _cohort(G, nt, nn, d, h)
    few = mask_of_bits(np.arange(nt) % 5 == 0)
    with pdfs.Solver(T, N, nt, nn, "bound") as s:
        for mode in ("bound", "empty", "bound"):
            s.set_prune_mode(mode)
            for u in (None, few):
                for mr in (1, 3, 6):
                    _check_wsc(s, T, N, nt, nn, h, mode, mr, u, per_round=None)
                exp = cpu.best(T, N, nt, nn, h, 1, 10, U=u, mode=mode)
                got, _ = s.best(h, 1, 10, u)
                assert (got is not None) == exp.found
                if exp.found:
                    assert tuple(got["genes"]) == exp.genes and got["tp"] == exp.tp


LAZY = [
    # the dense core (G, n_tumor, n_normal, density), its one-sample tail, h, max_rounds
    (300, 1280, 20, 0.3, 1300, 3, 5),     # 11 bit slices
    (70, 200, 60, 0.5, 150, 4, 0),        # more than 64 samples below a pair
    (64, 64, 5, 1.0, 200, 4, 0),          # every row of the core full: exactly 64 samples
    (65, 65, 5, 1.0, 200, 5, 0),          # 65
    (80, 400, 20, 0.4, 260, 5, 5),        # the general walk with more than 64 candidates
    (28, 200, 40, 0.6, 110, 9, 5),
    (110, 300, 30, 0.5, 500, 4, 5),       # lists longer than a wave
]


@pytest.mark.parametrize("case", LAZY, ids=[f"G{c[0]}_nt{c[1]}_h{c[5]}" for c in LAZY])
@pytest.mark.parametrize("mode", ["bound", "empty"])
def test_heavy_core_stays_lazy(pdfs, case, mode):  # noqa: F811
    G, nt, nn, d, tail, h, mr = case
    T, N = _cohort(G, nt, nn, d, h, tail)
    mask = mask_of_bits(np.arange(nt) % 3 != 0)
    with pdfs.Solver(T, N, nt, nn, mode, time_kernels=True) as s:
        for u in (None, mask):
            one = d == 1.0   # the first round covers all of the core's samples
            _check_wsc(s, T, N, nt, nn, h, mode, mr, u, per_round=None if one else False)


def test_batch_of_dense_cohorts(pdfs):  # noqa: F811
    shapes = [(60, 300, 60, 0.5, 4), (80, 500, 20, 0.45, 4), (520, 600, 50, 0.5, 3)]
    data = [(*_cohort(*s), s[1], s[2], s[4]) for s in shapes]
    exp = [cpu.wsc(T, N, nt, nn, h, 1, 10, mode="bound").rounds for T, N, nt, nn, h in data]
    for mode in ("bound", "empty"):
        for path in ("auto", "streams", "one_launch"):
            b = pdfs.pdfs_batch_create([x[:4] for x in data], mode, path=path)
            try:
                for _ in range(2):
                    res, st = pdfs.pdfs_batch_run(b, [x[4] for x in data], 1, 10,
                                                  n_tumors=[x[2] for x in data])
                    for r, e in zip(res, exp):
                        _same_rounds(r, e)
                    assert st["rounds"] == sum(len(e) for e in exp)
            finally:
                pdfs.pdfs_batch_destroy(b)


# Served requests walk in captured rounds where the cohort is dense, and where the
# budget holds only the walked rounds' lists (empty-intersection mode: bound-pruned
# walks need more than the lazy rounds).
SERVED = [
    (60, 300, 60, 0.5, 4, 0, "bound"), (60, 300, 60, 0.5, 4, 0, "empty"),
    (520, 600, 50, 0.5, 3, 0, "bound"), (520, 600, 50, 0.5, 3, 0, "empty"),
    (100, 300, 40, 0.5, 5, 0, "bound"),
    (2500, 120, 40, 0.02, 3, 35 << 20, "empty"), (2500, 90, 40, 0.02, 4, 35 << 20, "empty"),
]


@pytest.mark.parametrize("case", SERVED, ids=[f"G{c[0]}_h{c[4]}_{c[6]}" for c in SERVED])
def test_served_walked(pdfs, case):  # noqa: F811
    G, nt, nn, d, h, budget, mode = case
    T, N = _cohort(G, nt, nn, d, h)
    exp = cpu.wsc(T, N, nt, nn, h, 1, 10, mode="bound")
    srv = pdfs.pdfs_server_create(mode, 0, budget, 2)
    try:
        t = [pdfs.pdfs_server_submit(srv, T, N, nt, nn, h, 1, 10) for _ in range(3)]
        deadline = time.time() + 60
        for k in t:
            r = None
            while r is None and time.time() < deadline:
                r = pdfs.pdfs_server_poll(srv, k, cap=nt + 1)
            _same_rounds(r[0], exp.rounds)
    finally:
        pdfs.pdfs_server_destroy(srv)


# The literal reading of T-: single rounds walked, covers and sparse rounds lazy.
@pytest.mark.parametrize("G,nt,d,h", [(200, 300, 0.06, 3), (120, 300, 0.06, 4), (60, 200, 0.1, 5),
                                      (300, 200, 0.01, 3)])
@pytest.mark.parametrize("mode", ["bound", "empty"])
def test_literal_rounds(pdfs, G, nt, d, h, mode):  # noqa: F811
    I = synth.random_tiny(23, G, nt, 50, d, h)
    T, N = I.packed()
    with pdfs.Solver(T, N, nt, 50, mode, tn_literal=True) as s:
        for u in (None, mask_of_bits(np.arange(nt) % 3 != 1)):
            for mr in (1, 8):
                exp = cpu.wsc(T, N, nt, 50, h, 1, 10, mode=mode, max_rounds=mr, U0=u, tn="literal")
                got, st, final = s.wsc(h, 1, 10, 0, mr, u)
                _same_rounds(got, exp.rounds)
                assert np.array_equal(final, exp.final_uncovered)
                if mode == "empty":
                    _counters_equal(st, exp.counters, h)
            if h < 5:
                exp = cpu.wsc(T, N, nt, 50, h, 1, 10, mode=mode, max_rounds=1, U0=u, tn="literal")
                got, _ = s.best_noalloc(h, 1, 10, u)
                _same_rounds([got], exp.rounds)


# The allocation-free round against the oracle: walked where the cohort is dense,
# lazy elsewhere, and lazy where the walk's lists would not hold every pair (2850
# genes, nearly all of whose 4.06 M pairs share a sample: a lazy round holds 4.12 M,
# a walked one 3.99 M).  Row widths of one to three words
# and wider place the lazy round's buffers differently.
@pytest.mark.parametrize("h", [3, 4])
@pytest.mark.parametrize("G,nt,d,tail", [(90, 400, 0.4, 0), (300, 700, 0.2, 0), (70, 50, 0.2, 0),
                                         (600, 64, 0.03, 0), (250, 100, 0.04, 2000),
                                         (900, 130, 0.03, 0), (60, 700, 0.5, 500)])
def test_noalloc_against_oracle(pdfs, G, nt, d, tail, h):  # noqa: F811
    T, N = _cohort(G, nt, 60, d, h, tail)
    with pdfs.Solver(T, N, nt, 60, "bound") as s:
        for u in (None, mask_of_bits(np.arange(nt) % 4 != 1)):
            exp = cpu.wsc(T, N, nt, 60, h, 1, 10, mode="bound", max_rounds=1, U0=u)
            got, _ = s.best_noalloc(h, 1, 10, u)
            _same_rounds([got], exp.rounds)


def test_noalloc_dense_and_large(pdfs):  # noqa: F811
    T, N = _cohort(2850, 100, 20, 0.42, 3)
    with pdfs.Solver(T, N, 100, 20, "bound") as s:
        exp = cpu.wsc(T, N, 100, 20, 3, 1, 10, mode="bound", max_rounds=1)
        got, _ = s.best_noalloc(3, 1, 10)
        _same_rounds([got], exp.rounds)
