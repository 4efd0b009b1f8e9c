"""The tile kernels that serve what the block form does not, against the CPU oracle, bit for bit:
streamed tiles (also the wide form above n = 256) with the shape set, and by default dispatch for
instances whose entries span more than 127 in both matrices and for wider tenures -- alone, in
batches, served in chunks, and without allocation."""
import os
import sys
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import oracle
from paper_2307_11248_amd import qap
from paper_2307_11248_amd import workloads as W

pytestmark = pytest.mark.gpu

WORKERS = max(1, min(16, os.cpu_count() or 1))


def note(msg):
    sys.__stderr__.write("[gpu-case] %s\n" % msg)
    sys.__stderr__.flush()


def pmap(f, items):
    with ThreadPoolExecutor(WORKERS) as ex:
        return list(ex.map(f, items))


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    torch.cuda.init()
    yield


def instance(n, sym, top=255):
    """Entries from 0 to `top`, both ends in both matrices."""
    rng = np.random.default_rng([n, sym, top])
    F, D = W.random_instance(rng, n, 0, top, symmetric=sym, diag=True)
    for M in (F, D):
        M[0, 0], M[1, 1] = 0, top
    return F, D, rng


def check_tabu(F, D, perms, iters, lo, hi, seed, got):
    for j, r in enumerate(pmap(lambda j: oracle.tabu(F, D, perms[j], iters, lo, hi, seed, j), range(len(perms)))):
        assert (got[0][j] == r[0]).all() and got[1][j] == r[1] and got[2][j] == r[2], j


def check_two_opt(F, D, perms, cap, got):
    for j, r in enumerate(pmap(lambda p: oracle.two_opt(F, D, p, max_iters=cap), list(perms))):
        assert (got[0][j] == r[0]).all() and got[1][j] == r[1] and got[2][j] == r[2], j


# (the wide form keeps a compact tabu state while tenures fit its ring: short ones expire, 700
# iterations go round a ring of 512 moves)
@pytest.mark.parametrize("n,sym,lohi,iters", [
    (177, False, None, 400), (193, True, None, 300), (200, False, (20, 66), 400), (256, False, None, 300),
    (256, True, (0, 3), 300), (257, False, None, 200), (300, True, (1, 3), 400), (300, False, (5, 40), 400),
    (384, False, None, 200), (451, True, None, 200), (512, False, (51, 168), 700), (512, True, None, 200)])
def test_streamed_searches_with_the_shape_set(n, sym, lohi, iters):
    note("streamed, shape set n=%d sym=%d" % (n, sym))
    F, D, rng = instance(n, sym, 99)
    perms = W.starts(rng, n, 2)
    lo, hi = lohi or W.tabu_tenure_range(n)
    with qap.Handle(F, D) as h:
        h.set_tile_rows("tabu", -8)
        h.set_tile_rows("2opt", -8)
        t = h.tabu(perms, iters, lo, hi, 123)
        q = h.two_opt(perms, max_iters=60)
    check_tabu(F, D, perms, iters, lo, hi, 123, t)
    check_two_opt(F, D, perms, 60, q)


# every range of tile shapes that default dispatch picks from, then streamed, then wide
@pytest.mark.parametrize("n,sym", [(24, False), (70, False), (100, True), (128, True), (150, False), (176, True),
                                   (190, False), (230, True), (256, False), (300, False), (420, True), (512, False)])
def test_wide_entries_by_default_dispatch(n, sym):
    note("tiles by default n=%d sym=%d" % (n, sym))
    F, D, rng = instance(n, sym)
    perms = W.starts(rng, n, 2)
    lo, hi = W.tabu_tenure_range(n)
    iters = 250
    with qap.Handle(F, D) as h:
        t = h.tabu(perms, iters, lo, hi, 5)
        q = h.two_opt(perms, max_iters=80)
    check_tabu(F, D, perms, iters, lo, hi, 5, t)
    check_two_opt(F, D, perms, 80, q)


def test_wide_entries_in_a_batch():
    sizes, k, iters = [24, 50, 70, 100, 128, 150, 176, 190, 230, 256, 300], 2, 200
    note("tiles in a batch, sizes %s" % sizes)
    insts = [instance(n, t % 3 == 1) for t, n in enumerate(sizes)]
    starts = [W.starts(rng, n, k) for n, (_, _, rng) in zip(sizes, insts)]
    lohi = [W.tabu_tenure_range(n) for n in sizes]
    hs = [qap.Handle(F, D) for F, D, _ in insts]
    p, c, d = qap.tabu_batch(hs, np.concatenate([s.reshape(-1) for s in starts]), [k] * len(hs), iters,
                             [a for a, _ in lohi], [b for _, b in lohi], list(range(len(hs))))
    off = 0
    for t, (n, (F, D, _)) in enumerate(zip(sizes, insts)):
        got = (p[off:off + k * n].reshape(k, n), c[t * k:t * k + k], d[t * k:t * k + k])
        check_tabu(F, D, starts[t], iters, lohi[t][0], lohi[t][1], t, got)
        off += k * n
    for h in hs:
        h.close()


def test_wide_entries_and_tenures_served_in_chunks():
    """Requests of every tile shape of the chunked kernels and of their streamed form, by entries
    (both matrices span 255) and by tenures (64 values), beside some in block form."""
    note("tiles served in chunks")
    cases = [(24, 0, 255, None), (50, 1, 255, None), (70, 0, 255, None), (100, 1, 255, None), (128, 0, 255, None),
             (150, 1, 255, None), (165, 0, 255, None), (176, 1, 255, None), (190, 0, 255, None), (230, 1, 255, None),
             (256, 0, 255, None), (256, 1, 255, None), (300, 0, 255, None), (30, 0, 99, (10, 73)),
             (90, 1, 99, (80, 143)), (120, 0, 99, (3, 66)), (200, 0, 99, (100, 163)), (256, 1, 99, (25, 88)),
             (64, 0, 99, None), (210, 0, 99, None)]
    iters = 400
    want, tickets = [], []
    with qap.Server(1 << 30, 64, 0.1) as s:
        for t, (n, sym, top, ten) in enumerate(cases):
            F, D, rng = instance(n, sym, top)
            p = W.starts(rng, n, 1)[0]
            lo, hi = ten or W.tabu_tenure_range(n)
            want.append((F, D, p, lo, hi))
            tickets.append(s.submit(F, D, p, iters, lo, hi, 40 + t))
        for _ in range(100000):
            _, active, pending = s.step()
            if active == 0 and pending == 0:
                break
        assert s.stats()["chunks"] > 3 * len(cases)   # cut into chunks
        got = [s.result(t) for t in tickets]
    res = pmap(lambda a: oracle.tabu(a[1][0], a[1][1], a[1][2], iters, a[1][3], a[1][4], 40 + a[0], 0),
               list(enumerate(want)))
    for c, g, r in zip(cases, got, res):
        assert (g[0] == r[0]).all() and g[1] == r[1] and g[2] == r[2], c


# the tables and the tile state in the fixed scratch, a larger call and then a smaller one
@pytest.mark.parametrize("calls", [[(96, 64, False, 255), (40, 8, True, 255)], [(200, 6, False, 255), (180, 3, True, 255)],
                                   [(384, 4, False, 255), (300, 2, True, 255)]], ids=["tiles", "streamed", "wide"])
def test_noalloc_in_tiles(calls):
    import torch
    for i, (n, k, sym, top) in enumerate(calls):
        note("noalloc in tiles n=%d k=%d" % (n, k))
        F, D, rng = instance(n, sym, top)
        perms = W.starts(rng, n, k)
        lo, hi = W.tabu_tenure_range(n)
        p = torch.from_numpy(perms).cuda()
        c = torch.zeros(k, dtype=torch.int64, device="cuda")
        d = torch.zeros(k, dtype=torch.int32, device="cuda")
        with qap.Handle(F, D) as h:
            h.tabu_noalloc_async(p, 120, lo, hi, 77, c, d)
            torch.cuda.synchronize()
        got = [x.cpu().numpy()[:8] for x in (p, c, d)]
        check_tabu(F, D, perms[:8], 120, lo, hi, 77, got)
