"""Launches whose workgroups wait for lower tiles or chunks, where not every
workgroup is there when it is waited for (GPU).

The chip may be filled by other launches' waiting tiles while a launch's lower
tiles have not been dispatched, so a tile that is waited for and that nobody
has claimed is processed by the workgroup that waits.  The first test runs the
library built so that every wait gives up at once and two of three workgroups
leave without a look at their tile; the others run many such launches at once.
The oracle's bits each time.
"""
import os
import threading

import numpy as np
import pytest
import torch

import oracle
import paper_2310_00967_amd as micro
from paper_2310_00967_amd import _lib

from gpu_harness import first_mismatch, note

pytestmark = pytest.mark.gpu

DEV = "cuda"
TAKEOVER_LIB = os.path.join(os.path.dirname(os.path.abspath(__file__)), "libmicro_takeover.so")


@pytest.fixture
def takeover(monkeypatch):
    monkeypatch.setattr(_lib, "_lib", _lib.bind(TAKEOVER_LIB))


def vectors(N, seed):
    rng = np.random.default_rng(seed)
    g = rng.standard_normal(N).astype(np.float32)
    g[N // 3:N // 3 + 20_000] *= 30.0  # tiles with more pairs than they stage
    res = (rng.standard_normal(N) * 0.5).astype(np.float32)
    if N > 4:
        g[N // 2], g[0], g[N - 1] = np.nan, -np.inf, np.float32(2.5)
        res[N - 1] = 0.0
    return g, res


@pytest.mark.parametrize("length", [1, 1025, 3 * 1024, (1 << 19) - 1, (1 << 19) + 1, 512 * 4096, 512 * 4096 + 1,
                                    1 << 22])
@pytest.mark.parametrize("offset", [0, 3])
@pytest.mark.parametrize("entry", ["auto", "ticket", "noalloc", "topk", "ef"])
def test_tiles_of_absent_workgroups_are_taken_over(takeover, length, offset, entry):
    """One-row and four-row tiles, one look-back group and several, ragged ends
    and phases, with and without the second bound of a top-k hint and what a
    full pass accumulates beside the partition; two calls in a row, so the
    claims of one launch mean nothing to the next."""
    note(f"takeover length={length} offset={offset} entry={entry}")
    world, rank = (3, 1) if entry == "ef" else (1, 0)
    N = length * world
    g, res = vectors(N, length + offset)
    gbuf = torch.empty(N + 8, dtype=torch.float32, device=DEV)
    rbuf = torch.full((N + 8,), 7.0, dtype=torch.float32, device=DEV)
    g_dev, r_dev = gbuf[1:1 + N], rbuf[offset:offset + N]
    g_dev.copy_(torch.from_numpy(g))
    r_dev.copy_(torch.from_numpy(res))
    oi = torch.full((length + 4,), -9, dtype=torch.int32, device=DEV)
    ov = torch.full((length + 4,), -9.0, dtype=torch.float32, device=DEV)
    sp = None
    if entry != "noalloc":
        sp = micro.Sparsifier(N, device=DEV,
                              rule=micro.MICRO_RULE_TOPK if entry == "topk" else micro.MICRO_RULE_PROPORTIONAL,
                              variant=micro.MICRO_VARIANT_TICKET if entry == "ticket" else micro.MICRO_VARIANT_AUTO)
    theta = 2.5
    for call in range(2):
        if entry == "topk":
            theta = oracle.topk_step(g, res.copy(), rank, world, 0.01, 1.0)[3]  # an exact hint
            o_idx, o_val, k_or, th_or = oracle.topk_step(g, res, rank, world, 0.01, theta)
            k, th, _, _ = sp.step(g_dev, r_dev, rank, world, 0.01, theta, oi, ov)
        elif entry == "ef":
            o_idx, o_val, k_or, th_or = oracle.ef_step(g, res, 0, rank, world, 0.01, theta)[:4]
            k, th, _, _, _ = sp.ef_step(g_dev, r_dev, 0, rank, world, 0.01, theta, oi, ov)
        else:
            o_idx, o_val, k_or, th_or = oracle.step(g, res, rank, world, 0.01, theta)
            if entry == "noalloc":
                k, th = _lib.micro_sparsify_step_noalloc(g_dev.data_ptr(), r_dev.data_ptr(), N, rank, world, 0.01,
                                                         theta, oi.data_ptr(), ov.data_ptr())
            else:
                k, th, _, _ = sp.step(g_dev, r_dev, rank, world, 0.01, theta, oi, ov)
        torch.cuda.synchronize()
        where = (length, offset, entry, call)
        assert (k, th) == (k_or, th_or), where
        assert np.array_equal(oi[:k].cpu().numpy(), o_idx), where
        assert first_mismatch(ov[:k].cpu().numpy(), o_val) < 0, where
        assert entry == "topk" or bool((oi[k:] == -9).all()) and bool((ov[k:] == -9.0).all()), where
        assert first_mismatch(r_dev.cpu().numpy(), res) < 0, where
        assert bool((rbuf[:offset] == 7.0).all()) and bool((rbuf[offset + N:] == 7.0).all()), where
        if call == 0 and entry == "auto" and length == 1 << 22:
            # four-row tiles of 1024-value rows from the residual's 16-byte boundary
            starts = range(-offset, N, 1024)
            acc_rows = sum(int(np.sum((o_idx >= s) & (o_idx < s + 1024))) > 256 for s in starts)
            assert sp.last_stats()[1] == acc_rows, where
        theta = th_or
        oi.fill_(-9)
        ov.fill_(-9.0)
    if sp is not None:
        sp.close()


def on_streams(threads, work):
    """work(i) in a thread and on a stream of its own, for each i."""
    def run(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            work(i)

    torch.cuda.synchronize()
    pool = [threading.Thread(target=run, args=(i,)) for i in range(threads)]
    for t in pool:
        t.start()
    for t in pool:
        t.join()


@pytest.mark.parametrize("theta", [2.5, 0.7])  # 0.7: tiles with more pairs than they stage, five wavefronts each
def test_steps_on_many_streams_at_once(theta):
    """Eight contexts stepped by eight threads on streams of their own, each a
    launch of about a thousand tiles taken by workgroup index."""
    N, steps, threads = 4_000_003, 4, 8
    note(f"one-launch steps on many streams theta={theta}")
    rng = np.random.default_rng(3)
    g = rng.standard_normal(N, dtype=np.float32)
    res, want = np.zeros(N, np.float32), []
    for _ in range(steps):
        idx, val, k, _ = oracle.step(g, res, 0, 1, 0.01, theta)
        want.append((k, idx, val))
    g_dev = torch.from_numpy(g).to(DEV)
    out = [torch.zeros(N, dtype=torch.float32, device=DEV) for _ in range(threads)]
    got = [[] for _ in range(threads)]

    def work(i):
        sp = micro.Sparsifier(N, device=DEV)
        for _ in range(steps):
            k, _, idx, val = sp.step(g_dev, out[i], 0, 1, 0.01, theta)
            got[i].append((k, idx.cpu().numpy(), val.cpu().numpy()))
        sp.close()

    on_streams(threads, work)
    for i in range(threads):
        assert len(got[i]) == steps, i
        for (k, idx, val), (ko, io, vo) in zip(got[i], want):
            assert k == ko and np.array_equal(idx, io) and first_mismatch(val, vo) < 0, i
        assert first_mismatch(out[i].cpu().numpy(), res) < 0, i


def test_hinted_trims_on_many_streams_at_once():
    """Eight top-k contexts likewise, lists of about 150 of the trim's chunks."""
    N, steps, threads, density = 4_500_000, 4, 8, 0.12
    note("hinted trims on many streams")
    rng = np.random.default_rng(4)
    g = rng.standard_normal(N, dtype=np.float32)
    res, want, hint = np.zeros(N, np.float32), [], []
    for _ in range(steps):
        hint.append(oracle.topk_step(g, res.copy(), 0, 1, density, 1.0)[3])
        idx, val, k, th = oracle.topk_step(g, res, 0, 1, density, hint[-1])
        want.append((k, th, idx, val))
    g_dev = torch.from_numpy(g).to(DEV)
    out = [torch.zeros(N, dtype=torch.float32, device=DEV) for _ in range(threads)]
    got = [[] for _ in range(threads)]

    def work(i):
        sp = micro.Sparsifier(N, device=DEV, rule=micro.MICRO_RULE_TOPK)
        for t in range(steps):
            k, th, idx, val = sp.step(g_dev, out[i], 0, 1, density, hint[t])
            got[i].append((k, th, idx.cpu().numpy(), val.cpu().numpy()))
        sp.close()

    on_streams(threads, work)
    for i in range(threads):
        assert len(got[i]) == steps, i
        for (k, th, idx, val), (ko, to, io, vo) in zip(got[i], want):
            assert (k, th) == (ko, to) and np.array_equal(idx, io) and first_mismatch(val, vo) < 0, i
        assert first_mismatch(out[i].cpu().numpy(), res) < 0, i
