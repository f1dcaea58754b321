"""The three ways the pair kernel's segments get their entering states: combined from the summaries
(few segments), left by the pass over a sequence's chunks (short sequences), left by the scan over
the summaries (long sequences).  Each continues from an input state and ends in a ragged chunk;
the bars are those of the forward's parity tests."""
import numpy as np
import pytest
import torch

from test_gpu_parity import gauss, run_case

pytestmark = pytest.mark.gpu

CASES = [  # B, H, chunks, d, M, S, T
    (1, 3, 4, 64, 64, 64, (127.0, 254.0, 130.5)),   # combined, four segments
    (1, 3, 5, 64, 64, 64, (127.0, 254.0, 130.5)),   # pass, five segments of a chunk
    (1, 3, 9, 64, 64, 64, (127.0, 254.0, 130.5)),   # pass, odd number of jobs and stages
    (1, 2, 80, 32, 16, 31, (31.0, 62.0)),           # pass, one wave per workgroup, its last length
    (1, 2, 81, 32, 16, 31, (31.0, 62.0)),           # scan
    (1, 1, 17, 64, 20, 39, (39.0,)),                # pass, padded modes
    (1, 2, 12, 64, 100, 30, (199.0, 250.0)),        # pass, 128 padded modes (four chunks per stage)
    (5, 5, 46, 32, 64, 127, (127.0, 254.0, 127.0, 254.0, 127.0)),  # pass, three chunks per segment
    (2, 16, 9, 128, 32, 63, tuple(63.0 * (1 + h % 2) for h in range(16))),  # pass, one unit per workgroup
    (5, 10, 90, 32, 16, 16, tuple(31.0 + h for h in range(10))),   # scan, several chunks per segment
]


@pytest.mark.parametrize("B,H,nch,d,M,S,T", CASES)
def test_entering_states(B, H, nch, d, M, S, T):
    L = 64 * nch - 23
    q, k, v = gauss(nch + M, B, H, L, d, torch.bfloat16)
    rng = np.random.default_rng(7)
    sk, sv = (rng.standard_normal((B, H, 2, M, d)).astype(np.float32) for _ in range(2))
    sk[:, :, 1, 0] = sv[:, :, 1, 0] = 0.0
    run_case(q, k, v, T, M, S, torch.bfloat16, t0=100, sk=sk, sv=sv, label=f"{B}x{H}x{L}x{d}")


BWD_CASES = [  # B, H, chunks, d, M, S, T: many summary blocks per sequence (scanned), and just too few
    (1, 2, 20, 64, 64, 64, (127.0, 254.0)),
    (1, 3, 8, 64, 20, 39, (39.0, 41.5, 78.0)),
    (1, 3, 7, 32, 16, 31, (31.0, 62.0, 31.0)),
    (2, 12, 40, 32, 32, 63, tuple(63.0 * (1 + h % 2) for h in range(12))),   # several blocks per segment
]


@pytest.mark.parametrize("B,H,nch,d,M,S,T", BWD_CASES)
def test_backward_blocks(B, H, nch, d, M, S, T):
    from test_gpu_backward import run_bwd, tensors
    (q, k, v, g), (sk, sv, gk, gv) = tensors(nch + M, B, H, 64 * nch - 23, d, M, torch.bfloat16, with_states=True)
    run_bwd(q, k, v, g, T, M, S, torch.bfloat16, t0=50, sk=sk, sv=sv, gk=gk, gv=gv, label=f"{B}x{H}x{nch} chunks",
            rows=[(0, 0), (B - 1, H - 1)])


def test_decay_call_between_table_reuses():
    """A decay forward builds no tables but writes its schedules into the workspace: a forward that
    asks for the tables an earlier one left there must build them again."""
    from test_gpu_parity import _bla, to_dev
    bla = _bla()
    B, H, L, d, M, S, T = 1, 4, 64 * 12, 64, 32, 32, (63.0, 126.0, 70.5, 90.0)
    q, k, v = (to_dev(x, torch.bfloat16) for x in gauss(5, B, H, L, d, torch.bfloat16))
    p = bla.make_params(B, H, L, d, M, S, torch.bfloat16)
    ws = torch.empty(max(bla.workspace_size(p), bla.decay_workspace_size(p)), dtype=torch.uint8, device="cuda")
    first = bla.forward(q, k, v, T, M, S, workspace=ws)
    bla.decay_forward(q, k, v, T, M, S, workspace=ws)
    again = bla.forward(q, k, v, T, M, S, workspace=ws, reuse_tables=True)
    torch.cuda.synchronize()
    for a, b in zip(first, again):
        assert torch.equal(a, b)
