"""reuse_tables: a call keeps the tables that an earlier call left in its workspace only while they
are still there and where it looks for them."""
import ctypes

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


def _layer_problem(bla):
    B, H, L, d, M, S = 1, 4, 64 * 12, 64, 32, 32
    T = (63.0, 126.0, 70.5, 90.0)
    D = H * d
    x = to_dev(gauss(6, 1, B, L, D, torch.bfloat16)[0][0], torch.bfloat16)
    w = [to_dev(gauss(8, 1, 1, D, n, torch.bfloat16)[0][0, 0], torch.bfloat16) / 16 for n in (3 * D, D)]
    p = bla.make_params(B, H, L, d, M, S, torch.bfloat16, reuse_tables=True)
    ws = torch.zeros(bla.layer_workspace_size(p), dtype=torch.uint8, device="cuda")

    def layer(workspace):
        y = torch.empty_like(x)
        st = bla.lib().bla_layer_forward(ctypes.byref(p), (ctypes.c_double * H)(*T), x.data_ptr(), w[0].data_ptr(),
                                         w[1].data_ptr(), None, None, y.data_ptr(), None, None, workspace.data_ptr(),
                                         workspace.numel(), torch.cuda.current_stream().cuda_stream)
        assert st == 0
        return y

    q, k, v = (to_dev(t, torch.bfloat16) for t in gauss(5, B, H, L, d, torch.bfloat16))
    return (q, k, v, T, M, S), layer, ws


def test_layer_between_calls_that_keep_tables():
    """The layer writes its projections where a forward's tables were."""
    bla = _bla()
    args, layer, ws = _layer_problem(bla)
    first = bla.forward(*args, workspace=ws)
    layer(ws)
    again = bla.forward(*args, workspace=ws, reuse_tables=True)
    torch.cuda.synchronize()
    for a, b in zip(first, again):
        assert torch.equal(a, b)


def test_forward_between_layers_that_keep_tables():
    """A layer keeps its operator's tables inside its workspace; a forward at the same address with
    scratch up to there writes over them."""
    bla = _bla()
    args, layer, ws = _layer_problem(bla)
    first = layer(ws)
    kept = layer(ws)
    q, k, v, T, M, S = args  # the forward below takes the whole workspace as its own
    big = bla.make_params(4, 4, 64 * 12, 64, M, S, torch.bfloat16)
    assert bla.workspace_size(big) <= ws.numel()
    four = [t.expand(4, -1, -1, -1).contiguous() for t in (q, k, v)]
    bla.forward(*four, T, M, S, workspace=ws)
    again = layer(ws)
    torch.cuda.synchronize()
    assert torch.equal(first, kept) and torch.equal(first, again)
