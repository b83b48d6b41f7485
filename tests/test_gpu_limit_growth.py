"""Workspace that only saves time gives way to what a call needs: under a byte
limit that holds a time series' lists, but not with that workspace beside them,
a later call whose lists are longer still succeeds, with the bits of a tree
without a limit.  The order of the reverse pass's pieces (leaf <- cell lists)
and the pieces of a mutual walk's near lists (also to its reverse pass)."""
import numpy as np
import pytest
import torch

from paper_2502_01496_amd import fmm as F
from paper_2502_01496_amd import workloads as W
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


def _forces(tree, X, Mt, h):
    A = torch.empty_like(X)
    F.fmm_moments(tree, X, Mt, h)
    F.fmm_forces(tree, A, F.FMM_REWALK)
    torch.cuda.synchronize()
    return A


def test_piece_order_gives_way():
    n = 24000
    x = np.random.default_rng(65).random((n, 3))
    X, Mt, H0, H1 = to_dev(x, np.full(n, 1.0 / n), np.full(n, 1e-4), np.full(n, 0.1))
    AB = torch.from_numpy(W.cotangent(n, 66)).cuda()

    def series(limit):
        t = F.fmm_build_tree(X, F.default_params(leaf_size=1, device_bytes_limit=limit))
        try:
            a0 = _forces(t, X, Mt, H0)
            XB, MB = torch.empty_like(X), torch.empty_like(Mt)
            F.fmm_forces_vjp(t, AB, XB, MB)
            held = F.fmm_tree_device_bytes(t)
            a1 = _forces(t, X, Mt, H1)  # longer near lists
            more = F.fmm_tree_device_bytes(t)
            a2 = _forces(t, X, Mt, H0)  # the first ones again: pieces without an order
            XB2, MB2 = torch.empty_like(X), torch.empty_like(Mt)
            F.fmm_forces_vjp(t, AB, XB2, MB2)
            return held, more, [a0, XB, MB, a1, a2, XB2, MB2]
        finally:
            F.fmm_tree_free(t)

    before, after, ref = series(0)
    say(f"[gpu limit] piece order: {before} B, {after} B with longer lists")
    assert after > before + 4096
    _, less, got = series(after - 4096)
    assert less < after - 4096
    assert torch.equal(ref[1], ref[5]) and torch.equal(ref[2], ref[6])
    assert all(torch.equal(a, b) for a, b in zip(got, ref))


def test_mutual_pieces_give_way(monkeypatch):
    n = 4096
    x, m, h = W.plummer(n, 67)
    X, Mt, H0, H1 = to_dev(x, m, h, np.full(n, 2.0 * np.abs(x).max()))

    def series(limit, piece=None):
        if piece:
            monkeypatch.setenv("FMM_MI355_PIECE", piece)
        t = F.fmm_build_tree(X, F.default_params(leaf_size=10, walk=F.FMM_WALK_MUTUAL,
                                                 device_bytes_limit=limit))
        monkeypatch.delenv("FMM_MI355_PIECE", raising=False)
        try:
            a0 = _forces(t, X, Mt, H0)
            held = F.fmm_tree_device_bytes(t)
            a1 = _forces(t, X, Mt, H1)
            more = F.fmm_tree_device_bytes(t)
            a2 = torch.empty_like(X)
            F.fmm_forces(t, a2)
            return held, more, [a0, a1, a2]
        finally:
            F.fmm_tree_free(t)

    whole0, whole1, _ = series(0, "1000000")  # no pieces
    split0, split1, ref = series(0)
    say(f"[gpu limit] mutual: {whole0} -> {whole1} B, with pieces {split0} -> {split1} B")
    assert whole1 + 1024 > split0 > whole0 + 1024  # the first call's pieces fit the limit
    _, less, got = series(whole1 + 1024)
    assert less <= whole1 + 1024
    assert all(torch.equal(a, b) for a, b in zip(got, ref))


def test_mutual_pieces_give_way_to_the_reverse_pass():
    n = 4096
    x, m, h = W.plummer(n, 67)
    X, Mt, H = to_dev(x, m, h)
    AB = torch.from_numpy(W.cotangent(n, 68)).cuda()

    def run(limit):
        t = F.fmm_build_tree(X, F.default_params(leaf_size=10, walk=F.FMM_WALK_MUTUAL,
                                                 device_bytes_limit=limit))
        try:
            a = _forces(t, X, Mt, H)
            XB, MB = torch.empty_like(X), torch.empty_like(Mt)
            F.fmm_forces_vjp(t, AB, XB, MB)
            return F.fmm_tree_device_bytes(t), [a, XB, MB]
        finally:
            F.fmm_tree_free(t)

    held, ref = run(0)
    less, got = run(held - 1)
    say(f"[gpu limit] mutual reverse pass: {held} B without a limit, {less} B under {held - 1} B")
    assert less < held
    assert all(torch.equal(a, b) for a, b in zip(got, ref))
