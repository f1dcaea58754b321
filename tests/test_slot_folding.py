"""Slot folding: slots s and S - s share a row of the slot matrices (A[S-s] = A[s], B[S-s] = -B[s]),
so the kernels with at least 64 padded slots keep the rows s <= S/2 and form both slots' scores
from the row's two half products.  The edges are slot counts at which rows lose their partner:
S odd, S even below the padded count (row S/2 is its own partner) and S equal to the padded
count (slot S/2 takes the unused entry of row 0).
"""
import numpy as np
import pytest
import torch

import oracle
from host_probe import run


def folded_slot(i, S, SP):
    """The slot of folded entry i (None: no slot), as csrc/bla_device.h defines it."""
    HP = SP // 2
    if i < HP:
        return i if 2 * i <= S and i < S else None
    s = i - HP
    if s == 0:
        return HP if S == SP else None
    return S - s if 2 * s < S else None


def test_the_library_orders_the_slots_so():
    lines = [list(map(int, line.split())) for line in run("slots")]
    assert len(lines) == 32 + 64 + 128
    for SP, S, *slots in lines:
        assert slots == [-1 if (x := folded_slot(i, S, SP)) is None else x for i in range(SP)], (SP, S)


@pytest.mark.parametrize("SP", [64, 128, 256])
def test_entries_cover_every_slot_once_and_rows_reproduce_the_matrices(SP):
    M = SP // 2
    for S in range(SP // 2 + 1, SP + 1):
        HP = SP // 2
        slots = [folded_slot(i, S, SP) for i in range(SP)]
        assert sorted(s for s in slots if s is not None) == list(range(S))
        A, B, _ = oracle.interp(M, S, 2.0 * M - 1.0)
        A = np.vstack([A, np.zeros((SP + 1 - S, M))])
        B = np.vstack([B, np.zeros((SP + 1 - S, M))])
        uc, us = np.random.default_rng(S).standard_normal((2, M))
        p, q = A[:HP] @ uc, B[:HP] @ us
        if S == SP:
            q[0] += A[HP] @ uc
        main, mirror = p + q, p - q
        main[0], mirror[0] = p[0], q[0]
        got = np.concatenate([main, mirror])
        z = A[:S] @ uc + B[:S] @ us
        for i, s in enumerate(slots):
            if s is not None:
                assert abs(got[i] - z[s]) < 1e-12
        # the readout weights from the slot weights
        e = np.random.default_rng(S + 1).random(S)
        x = np.array([0.0 if s is None else e[s] for s in slots])
        wp, wq = x[:HP] + x[HP:], x[:HP] - x[HP:]
        wp[0], wq[0] = x[0], x[HP]
        a, b = wp @ A[:HP], wq @ B[:HP]
        if S == SP:
            a = a + wq[0] * A[HP]
        assert np.allclose(a, e @ A[:S], atol=1e-12) and np.allclose(b, e @ B[:S], atol=1e-12)


CASES = [  # dtype, d, M, S, anchor
    (torch.bfloat16, 64, 32, 33, 0), (torch.bfloat16, 64, 32, 62, 1), (torch.bfloat16, 64, 20, 63, 0),
    (torch.bfloat16, 32, 64, 64, 1), (torch.bfloat16, 64, 64, 64, 0), (torch.bfloat16, 64, 64, 65, 1),
    (torch.bfloat16, 64, 64, 127, 0), (torch.bfloat16, 64, 64, 127, 1), (torch.bfloat16, 64, 64, 128, 0),
    (torch.bfloat16, 128, 64, 127, 0), (torch.bfloat16, 128, 64, 50, 1), (torch.bfloat16, 128, 64, 64, 0),
    (torch.bfloat16, 128, 32, 63, 1), (torch.bfloat16, 64, 100, 64, 0), (torch.bfloat16, 64, 100, 128, 1),
    (torch.bfloat16, 128, 128, 64, 0), (torch.bfloat16, 128, 128, 63, 1), (torch.bfloat16, 128, 128, 127, 0),
    (torch.bfloat16, 128, 128, 128, 1), (torch.bfloat16, 128, 128, 255, 0), (torch.bfloat16, 128, 128, 256, 0),
    (torch.float32, 64, 32, 63, 0), (torch.float32, 64, 32, 64, 1), (torch.float32, 32, 64, 127, 1),
    (torch.float32, 32, 64, 128, 0), (torch.float32, 64, 64, 66, 0),
]


def anchored_slots(state, T, M, S, pos):
    """Slot states [B,H,S,d] at position pos from mode states [B,H,2,M,d] (Sec. 3.3)."""
    m = np.arange(M)
    c = np.where(m == 0, 1.0, 2.0) / (2 * M - 1)
    out = []
    for h, Th in enumerate(T):
        ph = 2 * np.pi * m[None, :] / Th * (pos - np.arange(S)[:, None] * Th / S)  # [S, M]
        out.append((c * np.cos(ph)) @ state[:, h, 0] + (c * np.sin(ph)) @ state[:, h, 1])
    return np.stack(out, axis=1)


def two_parts(dtype, d, M, S, anchor, chunk=0):
    """A fresh sequence (the start mask hides slots of both sets) with a ragged last chunk, then its
    continuation past every threshold (the unmasked softmax)."""
    from test_gpu_parity import TOL, _bla, assert_close, gauss, to_dev
    bla = _bla()
    print(f"slot folding: {dtype} d={d} M={M} S={S} anchor={anchor} chunk={chunk}", flush=True)
    H, L = 2, 150
    T = [2.0 * M - 1.0, 2.3 * (2 * M - 1)]
    t0 = 0
    sk = sv = None
    for part in range(2):
        q, k, v = gauss(100 * part + S, 1, H, L, d, dtype)
        q = q * 4.0  # scores of order one, so that every slot's weight differs
        o, nk, nv = bla.forward(*(to_dev(x, dtype) for x in (q, k, v)), T, M, S, t0=t0, state_k=sk, state_v=sv,
                                phase_anchor=bool(anchor), chunk=chunk)
        torch.cuda.synchronize()
        sk64, sv64 = (None if x is None else x.double().cpu().numpy() for x in (sk, sv))
        if anchor:
            slots = [None if x is None else anchored_slots(x, T, M, S, t0 - 1) for x in (sk64, sv64)]
            ref = oracle.forward_anchored(q, k, v, T, M, S, t0=t0, slot_k=slots[0], slot_v=slots[1])[0]
        else:
            ref = oracle.forward(q, k, v, T, M, S, t0=t0, state_k=sk64, state_v=sv64)[0]
        assert_close(o.float().cpu().numpy(), ref, TOL[dtype], f"O part {part}")
        # far along the sequence: every threshold passed
        sk, sv, t0 = nk, nv, 4 * (2 * M - 1)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,d,M,S,anchor", CASES)
def test_forward(dtype, d, M, S, anchor):
    two_parts(dtype, d, M, S, anchor)


CHUNK_CASES = [  # dtype, chunk, d, M, S, anchor: odd S, S below the padded count and equal to it
    (torch.bfloat16, 16, 128, 64, 63, 1), (torch.bfloat16, 16, 64, 64, 127, 0), (torch.bfloat16, 16, 32, 64, 128, 1),
    (torch.bfloat16, 16, 64, 32, 50, 1), (torch.bfloat16, 32, 32, 64, 64, 1), (torch.bfloat16, 32, 64, 32, 63, 0),
    (torch.bfloat16, 32, 128, 64, 100, 1), (torch.bfloat16, 32, 128, 20, 33, 0), (torch.bfloat16, 32, 64, 64, 63, 1),
    (torch.bfloat16, 128, 64, 64, 64, 1), (torch.bfloat16, 128, 32, 64, 127, 1), (torch.bfloat16, 128, 128, 32, 63, 0),
    (torch.bfloat16, 128, 64, 32, 62, 1), (torch.float32, 16, 32, 64, 127, 0), (torch.float32, 16, 64, 64, 127, 1),
    (torch.float32, 16, 128, 32, 64, 1), (torch.float32, 32, 32, 32, 63, 0), (torch.float32, 32, 64, 64, 128, 1),
    (torch.float32, 128, 32, 20, 39, 1), (torch.float32, 128, 32, 32, 40, 0),
]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,chunk,d,M,S,anchor", CHUNK_CASES)
def test_forward_chunks(dtype, chunk, d, M, S, anchor):
    two_parts(dtype, d, M, S, anchor, chunk)


BWD_CASES = [  # d, M, S: the slot edges, and every way the waves of a side share mode and head-dim tiles
    (64, 64, 64), (64, 64, 63), (64, 64, 65), (64, 64, 127), (64, 64, 128), (64, 33, 34), (64, 32, 64), (64, 32, 63),
    (64, 32, 32), (64, 16, 31), (64, 5, 9), (32, 64, 128), (32, 64, 20), (32, 32, 64), (32, 17, 33), (32, 16, 16),
]


@pytest.mark.gpu
@pytest.mark.parametrize("d,M,S", BWD_CASES)
def test_backward(d, M, S):
    """A ragged last chunk, input states and gradients of the final states, from a masked start."""
    import bla_inputs as bi
    from test_gpu_backward import run_bwd, tensors
    (q, k, v, g), (sk, sv, gk, gv) = tensors(S + M, 2, 3, 64 * 5 - 17, d, M, torch.bfloat16, with_states=True)
    q = bi.round_bf16(q * 4.0)
    T = [2.0 * M - 1.0, 2.3 * (2 * M - 1), 4.0 * M]
    run_bwd(q, k, v, g, T, M, S, torch.bfloat16, t0=3, sk=sk, sv=sv, gk=gk, gv=gv, label=f"folding d={d} M={M} S={S}")
