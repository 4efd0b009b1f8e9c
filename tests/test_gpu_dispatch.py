"""What the library says about the kernels its searches run in."""
import sys

import numpy as np
import pytest

from paper_2307_11248_amd import qap
from paper_2307_11248_amd import workloads as W

pytestmark = pytest.mark.gpu


def note(msg):
    sys.__stderr__.write("[gpu-case] %s\n" % msg)
    sys.__stderr__.flush()


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    torch.cuda.init()
    yield


def instance(n, sym=False, span_f=99, span_d=255):
    rng = np.random.default_rng([n, sym])
    F, _ = W.random_instance(rng, n, 0, span_f, symmetric=sym, diag=True)
    D, _ = W.random_instance(rng, n, 0, span_d, symmetric=sym, diag=True)
    F[0, 0], F[1, 1], D[0, 0], D[1, 1] = 0, span_f, 0, span_d
    return F, D


def test_batch_groups_are_the_kernels_that_run():
    """One dispatch per block form (blocks of 32 a row, symmetric or not) and per tile-shape
    variant; the counts are those of the searches in tiles."""
    # (n, symmetric, span of F, forced tile rows, where it runs: a block form or a variant's slot)
    cases = [(20, False, 99, 0, "1g"), (32, False, 99, 0, "1g"), (30, True, 99, 0, "1s"), (64, False, 99, 0, "2g"),
             (256, False, 99, 0, "8g"), (256, True, 99, 0, "8s"), (50, False, 255, 2, 5), (40, False, 99, 2, 5),
             (100, False, 99, 8, 2), (200, False, 255, 0, 3), (300, False, 99, 0, 8)]
    note("batch groups of %d instances" % len(cases))
    hs = [qap.Handle(*instance(n, sym, sf)) for n, sym, sf, _, _ in cases]
    k = [1 + t % 3 for t in range(len(cases))]
    lohi = [W.paper_tenure_range(n) for n, *_ in cases]
    counts = np.zeros(9, dtype=int)
    for (n, _, _, _, where), kk in zip(cases, k):
        if not isinstance(where, str):
            counts[where] += kk
    with qap.Batch(hs, k, 10, [a for a, _ in lohi], [b for _, b in lohi], [1] * len(hs),
                   rows=[rows for _, _, _, rows, _ in cases]) as b:
        g, c = b.groups(counts=True)
        assert list(c) == list(counts), (list(c), list(counts))
        assert g == len({where for *_, where in cases})
        assert b.starts - c.sum() == sum(kk for kk, case in zip(k, cases) if isinstance(case[-1], str))
    for h in hs:
        h.close()


# the limits of the block form: spans, tenures, n, the shapes set on the handle
def test_block_form_says_which_searches_it_runs():
    note("block form query")
    for n, wide in ((60, 64), (256, 64), (257, 128), (512, 128)):
        with qap.Handle(*instance(n)) as h:
            assert h.block_form("tabu", 10, 20) and h.block_form("2opt")
            assert h.block_form("batch", 10, 20) == (n <= 256)
            assert h.block_form("tabu", 10, 10 + wide - 1) and not h.block_form("tabu", 10, 10 + wide)
            assert h.block_form("tabu", 1000, 1000) and not h.block_form("tabu", 1001, 1001)
            rows = h.tile_rows("tabu")[0]
            h.set_tile_rows("tabu", rows)
            assert not h.block_form("tabu", 10, 20) and h.block_form("2opt")
            h.prefer_tile_rows("tabu", rows)
            assert h.block_form("tabu", 10, 20)
            h.set_tile_rows("2opt", h.tile_rows("2opt")[0])
            assert not h.block_form("2opt")
            h.set_tile_rows("2opt", 0)
            assert h.block_form("2opt")
            for args in (("tabu", -1, 5), ("tabu", 6, 5), ("batch", 6, 5)):
                with pytest.raises(qap.QapError) as ei:
                    h.block_form(*args)
                assert ei.value.code == qap.QAP_E_INVALID
        for spans, block in (((127, 255), True), ((255, 127), True), ((128, 255), False), ((255, 255), False)):
            with qap.Handle(*instance(n, False, *spans)) as h:
                assert h.block_form("tabu", 10, 20) == block and h.block_form("2opt") == block, (n, spans)
