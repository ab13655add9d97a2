"""GPU parity of forward calls whose input dimension is no multiple of 128: the automatic path runs them on the matrix kernels
over rows of whole chunks, with anything behind a row's values.  Accumulators are exact, so Y without a bias is within three
roundings of fp32 of the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import sbn_synth
from gpu_util import DEV, assert_rel, hip_pack, oracle_pack, sbn

pytestmark = pytest.mark.gpu
Y_TOL = 4 * 2.0 ** -24


@pytest.mark.parametrize("N,M", [(2, 4), (6, 8), (4, 4), (1, 4), (2, 8)])
@pytest.mark.parametrize("tokens,d_out,d_in", [(1, 40, 8), (3, 130, 200), (16, 100, 1000), (17, 64, 136), (50, 1500, 1000), (64, 516, 192),
                                               (65, 512, 248), (600, 130, 648)])
@pytest.mark.parametrize("mode", ["plain", "kept", "given"])
def test_ragged_input_dimension(N, M, tokens, d_out, d_in, mode):
    s = sbn()
    W = sbn_synth.latent_weight(d_out, d_in, 4000 + d_out + d_in)
    X = sbn_synth.activations(tokens, d_in, 4001 + tokens)
    packed, gamma = hip_pack(W, N, M)
    _, g, Weff, _ = oracle_pack(W, N, M)
    y, _, r_xq, r_sx = oracle.sparse_ternary_linear(X.float().numpy(), Weff, g)
    Xd = X.to(DEV)
    Y = torch.full((tokens, d_out), float("nan"), dtype=torch.float32, device=DEV)
    ws = s.new_workspace(s.sbn_workspace_bytes(s.SBN_OP_LINEAR, tokens, d_out, d_in, N, M))
    ws.fill_(0x7f)                                   # whatever lies behind a row must not count
    if mode == "plain":
        s.sbn_sparse_ternary_linear(Xd, packed, gamma, Y, N, M, ws)
    else:
        # the caller's buffers hold exactly the rows: nothing in front of, between or behind them is the call's
        buf = torch.full((tokens * d_in + 512,), 99, dtype=torch.int8, device=DEV)
        xq = buf[256:256 + tokens * d_in].view(tokens, d_in)
        sx = torch.zeros(tokens, dtype=torch.float32, device=DEV)
        if mode == "kept":
            s.sbn_sparse_ternary_linear(Xd, packed, gamma, Y, N, M, ws, xq_out=xq, sx_out=sx)
        else:
            s.sbn_act_quant(Xd, xq, sx)
            s.sbn_sparse_ternary_linear(None, packed, gamma, Y, N, M, ws, xq_out=xq, sx_out=sx)
        torch.cuda.synchronize()
        assert np.array_equal(xq.cpu().numpy(), r_xq) and np.array_equal(sx.cpu().numpy(), r_sx)
        assert (buf[:256] == 99).all() and (buf[256 + tokens * d_in:] == 99).all()
    torch.cuda.synchronize()
    assert_rel(Y.cpu().numpy(), y, Y_TOL, f"{mode} {tokens} x {d_in} -> {d_out} at {N}:{M}")


@pytest.mark.parametrize("N,M", [(2, 4), (6, 8)])
@pytest.mark.parametrize("tokens", [5, 40])
def test_ragged_input_dimension_static_scratch(N, M, tokens):
    s = sbn()
    W = sbn_synth.latent_weight(72, 328, 4100)
    X = sbn_synth.activations(tokens, 328, 4101)
    packed, gamma = hip_pack(W, N, M)
    _, g, Weff, _ = oracle_pack(W, N, M)
    Y = torch.full((tokens, 72), float("nan"), dtype=torch.float32, device=DEV)
    s.sbn_sparse_ternary_linear_static(X.to(DEV), packed, gamma, Y, N, M)
    torch.cuda.synchronize()
    y, *_ = oracle.sparse_ternary_linear(X.float().numpy(), Weff, g)
    assert_rel(Y.cpu().numpy(), y, Y_TOL, "Y")


@pytest.mark.parametrize("N,M,tokens,d_out,d_in", [(2, 8, 4099, 2050, 64), (2, 8, 4080, 2050, 64),      # 8 Mi outputs: the dense path, and just below it
                                                   (6, 8, 8209, 8190, 192), (6, 8, 8190, 8190, 192),    # 64 Mi
                                                   (2, 4, 8209, 8190, 64), (2, 4, 14400, 8190, 320), (2, 4, 14300, 8190, 320)])   # 64 and 112 Mi
def test_half_chunks_with_many_outputs(N, M, tokens, d_out, d_in):
    s = sbn()
    W = sbn_synth.latent_weight(d_out, d_in, 4200 + d_in)
    X = sbn_synth.activations(tokens, d_in, 4201)
    packed, gamma = hip_pack(W, N, M)
    _, g, Weff, _ = oracle_pack(W, N, M)
    Y = torch.full((tokens, d_out), float("nan"), dtype=torch.float32, device=DEV)
    ws = s.new_workspace(s.sbn_workspace_bytes(s.SBN_OP_LINEAR, tokens, d_out, d_in, N, M))
    s.sbn_sparse_ternary_linear(X.to(DEV), packed, gamma, Y, N, M, ws)
    rows = np.unique(np.concatenate([np.arange(70), np.arange(tokens - 140, tokens), np.arange(0, tokens, 97)]))
    y, *_ = oracle.sparse_ternary_linear(X[torch.from_numpy(rows)].float().numpy(), Weff, g)
    assert torch.isfinite(Y).all()
    assert_rel(Y[torch.from_numpy(rows).to(DEV)].cpu().numpy(), y, Y_TOL, "Y")
