"""reuse_tables: a call keeps the tables that an earlier call left in its workspace only while they
are still there and where it looks for them."""
import pytest
import torch

from test_gpu_parity import _bla, gauss, to_dev

pytestmark = pytest.mark.gpu


def test_fragment_tables_after_a_shorter_call():
    """d = M = S = 128 in bf16: calls of 960 and 1000 tokens have equal tables but unequal scratch."""
    bla = _bla()
    B, H, d, M, S = 1, 16, 128, 128, 128
    T = [(1.0 + h % 2) * (2 * M - 1) for h in range(H)]
    q, k, v = (to_dev(x, torch.bfloat16) for x in gauss(7, B, H, 1000, d, torch.bfloat16))
    short = tuple(x[:, :, :960].contiguous() for x in (q, k, v))
    size = bla.workspace_size(bla.make_params(B, H, 1000, d, M, S, torch.bfloat16))
    ws = torch.zeros(size, dtype=torch.uint8, device="cuda")
    bla.forward(*short, T, M, S, workspace=ws)
    got = bla.forward(q, k, v, T, M, S, workspace=ws, reuse_tables=True)
    fresh = bla.forward(q, k, v, T, M, S)
    torch.cuda.synchronize()
    for a, b in zip(got, fresh):
        assert torch.equal(a, b)
