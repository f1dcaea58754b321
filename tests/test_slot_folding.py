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


def folded_slot(i, S, SP):
    """The slot of folded entry i (None: no slot), as csrc/bla_device.h defines it."""
    HP = SP // 2
    if i < HP:
        return i if 2 * i <= S and i < S else None
    s = i - HP
    if s == 0:
        return HP if S == SP else None
    return S - s if 2 * s < S else None


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
    (torch.bfloat16, 128, 64, 127, 0), (torch.bfloat16, 64, 100, 64, 0), (torch.bfloat16, 64, 100, 128, 1),
    (torch.bfloat16, 128, 128, 64, 0), (torch.bfloat16, 128, 128, 63, 1), (torch.bfloat16, 128, 128, 127, 0),
    (torch.bfloat16, 128, 128, 128, 1), (torch.bfloat16, 128, 128, 255, 0), (torch.bfloat16, 128, 128, 256, 0),
    (torch.float32, 64, 32, 63, 0), (torch.float32, 64, 32, 64, 1), (torch.float32, 32, 64, 127, 1),
    (torch.float32, 32, 64, 128, 0), (torch.float32, 64, 64, 66, 0),
]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,d,M,S,anchor", CASES)
def test_forward(dtype, d, M, S, anchor):
    """A fresh sequence (the start mask hides slots of both sets) with a ragged last chunk, then its
    continuation past every threshold (the unmasked softmax)."""
    from test_gpu_parity import TOL, _bla, assert_close, gauss, to_dev
    bla = _bla()
    print(f"slot folding: {dtype} d={d} M={M} S={S} anchor={anchor}", flush=True)
    H, L = 2, 150
    T = [2.0 * M - 1.0, 2.3 * (2 * M - 1)]
    t0 = 0
    sk = sv = None
    for part in range(2):
        q, k, v = gauss(100 * part + S, 1, H, L, d, dtype)
        q = q * 4.0  # scores of order one, so that every slot's weight differs
        o, nk, nv = bla.forward(*(to_dev(x, dtype) for x in (q, k, v)), T, M, S, t0=t0, state_k=sk, state_v=sv,
                                phase_anchor=bool(anchor))
        torch.cuda.synchronize()
        sk64, sv64 = (None if x is None else x.double().cpu().numpy() for x in (sk, sv))
        if anchor and part == 0:
            ref = oracle.forward_anchored(q, k, v, T, M, S)[0]
        elif anchor:
            continue  # the anchored oracle keeps slot states, not mode states
        else:
            ref = oracle.forward(q, k, v, T, M, S, t0=t0, state_k=sk64, state_v=sv64)[0]
        assert_close(o.float().cpu().numpy(), ref, TOL[dtype], f"O part {part}")
        # far along the sequence: every threshold passed
        sk, sv, t0 = nk, nv, 4 * (2 * M - 1)


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
