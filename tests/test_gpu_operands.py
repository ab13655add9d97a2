"""The operands of the backward products value by value: where one factor of a product selects single elements, a sum has one
term, the result is that operand itself (times gamma for dX) and has to be equal."""
import pytest
import torch

import sbn_synth
from gpu_util import DEV, hip_pack, oracle_pack, sbn

pytestmark = pytest.mark.gpu


def backward(dY, packed, gamma, xq, sx, N, M, dX=None, dW=None):
    s = sbn()
    tokens, d_out, d_in = dY.shape[0], dY.shape[1], xq.shape[1]
    ws = s.new_workspace(s.sbn_workspace_bytes(s.SBN_OP_BACKWARD, tokens, d_out, d_in, N, M))
    s.sbn_sparse_ternary_linear_backward(dY, packed, gamma, xq, sx, N, M, ws, d_in, dX=dX, dW=dW)
    torch.cuda.synchronize()


# d_out: one vector of eight, fewer than a block's 256 vectors, 256, 257 and two blocks less one; tokens off the row quads
@pytest.mark.parametrize("tokens,d_out", [(1, 8), (3, 8), (66, 8), (5, 24), (133, 264), (4, 2048), (67, 2048), (129, 2056), (6, 4088)])
def test_scaled_gradient(tokens, d_out):
    d_in = (tokens + 7) // 8 * 8
    g = torch.Generator().manual_seed(tokens + d_out)
    dY = (torch.randn(tokens, d_out, generator=g) * torch.exp2(torch.randint(-40, 40, (tokens, d_out), generator=g).float())).to(torch.bfloat16)
    dY[tokens - 1, d_out - 1] = 0
    sx = torch.rand(tokens, generator=g) * 100 + 1e-3
    xq = torch.zeros(tokens, d_in, dtype=torch.int8)
    xq[torch.arange(tokens), torch.arange(tokens)] = 1                  # dW[o, t] = dY[t, o] / s_x[t]
    dW = torch.full((d_out, d_in), float("nan"), dtype=torch.bfloat16, device=DEV)
    backward(dY.to(DEV), None, None, xq.to(DEV), sx.to(DEV), 2, 4, dW=dW)
    want = (dY.float() / sx[:, None]).to(torch.bfloat16)
    assert torch.equal(dW[:, :tokens].T.float().cpu(), want.float())


F32_TINY = 2.0 ** -126
# one scale per token: the ends of the range in which the quotient is not a division, around it, and the ends of the type
SCALES = [2.0 ** -20, 2.0 ** -20 * (1 - 2.0 ** -24), 2.0 ** 30 * (1 - 2.0 ** -24), 2.0 ** 30, 1.0, 127.0 / 3.3e38, 0.0, -0.0, -3.0, float("inf"), float("nan"),
          F32_TINY, F32_TINY / 8, 3e38, 2.0 ** 127, 127.0 / 4.5]
# gradients around the ends of that range and of the type
VALUES = [0.0, -0.0, 1.0, -1.0, 200.0, 3.3e38, -3.3e38, float("inf"), float("-inf"), float("nan"), 2.0 ** -90, 2.0 ** -90 * (1 - 2.0 ** -8), 2.0 ** 100,
          2.0 ** 100 * (1 - 2.0 ** -8), 2.0 ** -101, 2.0 ** -110, 2.0 ** -126, 2.0 ** -130, 2.0 ** -133, 1.5 * 2.0 ** -70, 3.0, 1e5, 1e-5, -2.0 ** -95]


@pytest.mark.parametrize("at", [0, 1, 6, 7])
@pytest.mark.parametrize("scale", SCALES)
def test_scaled_gradient_is_the_quotient_for_all_operands(scale, at):
    # the quotient itself, value by value: infinite where it overflows, NaN, zeros, subnormal.  A lane scales eight values of four rows
    # and chooses the form by all of them, so each value stands alone among seven ordinary ones.  One token: other rows'
    # infinities would meet the zeros of x~
    dY = torch.tensor([1.0, -0.75, 3.0, 0.0, 0.5, 1e-3, 7.0, -113.0]).repeat(len(VALUES), 1)
    dY[:, at] = torch.tensor(VALUES)
    dY = dY.reshape(1, -1).to(torch.bfloat16)
    sx = torch.tensor([scale], dtype=torch.float32)
    xq = torch.zeros(1, 8, dtype=torch.int8)
    xq[0, 0] = 1
    dW = torch.full((dY.shape[1], 8), 7.0, dtype=torch.bfloat16, device=DEV)
    backward(dY.to(DEV), None, None, xq.to(DEV), sx.to(DEV), 2, 4, dW=dW)
    want = (dY.float() / sx[:, None]).to(torch.bfloat16).float()[0]
    got = dW[:, 0].float().cpu()
    assert torch.equal(got.isnan(), want.isnan())
    assert torch.equal(got[~want.isnan()], want[~want.isnan()])         # (a sum that begins with +0 has no -0; == does not tell)


@pytest.mark.parametrize("tokens,d_in", [(1, 8), (63, 120), (64, 128), (65, 136), (130, 264), (200, 384)])
def test_transposed_rows(tokens, d_in):
    d_out = (tokens + 7) // 8 * 8
    xq = torch.randint(-128, 128, (tokens, d_in), dtype=torch.int8, generator=torch.Generator().manual_seed(d_in))
    sx = torch.full((tokens,), 2.0)
    dY = torch.zeros(tokens, d_out, dtype=torch.bfloat16)
    dY[torch.arange(tokens), torch.arange(tokens)] = 2                  # dW[t, k] = xq[t, k]
    dW = torch.full((d_out, d_in), float("nan"), dtype=torch.bfloat16, device=DEV)
    backward(dY.to(DEV), None, None, xq.to(DEV), sx.to(DEV), 2, 4, dW=dW)
    assert torch.equal(dW[:tokens].float().cpu(), xq.float())


@pytest.mark.parametrize("N,M", [(2, 4), (6, 8), (1, 4), (2, 8), (4, 4), (1, 2), (3, 4)])   # the last two through int8
@pytest.mark.parametrize("d_out,d_in", [(8, 8), (72, 136), (128, 256)])
def test_transposed_weights(N, M, d_out, d_in):
    W = sbn_synth.latent_weight(d_out, d_in, 1200 + d_in)
    packed, gamma = hip_pack(W, N, M)
    _, _, Weff, _ = oracle_pack(W, N, M)
    dY = torch.eye(d_out, dtype=torch.bfloat16, device=DEV)             # dX[o, k] = gamma W_eff[o, k]
    dX = torch.full((d_out, d_in), float("nan"), dtype=torch.bfloat16, device=DEV)
    backward(dY, packed, gamma, torch.zeros(d_out, d_in, dtype=torch.int8, device=DEV), torch.ones(d_out, device=DEV), N, M, dX=dX)
    assert torch.equal(dX.float().cpu(), (torch.from_numpy(Weff).float() * gamma.cpu()).to(torch.bfloat16).float())


@pytest.mark.parametrize("N,M", [(2, 4), (3, 4)])
@pytest.mark.parametrize("d_out", [56, 64, 120, 136, 192, 200, 256, 264, 320, 392, 520])
def test_weights_of_every_stage(N, M, d_out):
    # one to nine stages of 64: a slot of weights lasts for two of them, of gradients for one; the last is whole or ends within a vector
    d_in = 144
    W = sbn_synth.latent_weight(d_out, d_in, 1300 + d_out)
    packed, gamma = hip_pack(W, N, M)
    _, _, Weff, _ = oracle_pack(W, N, M)
    dY = torch.eye(d_out, dtype=torch.bfloat16, device=DEV)
    dX = torch.full((d_out, d_in), float("nan"), dtype=torch.bfloat16, device=DEV)
    backward(dY, packed, gamma, torch.zeros(d_out, d_in, dtype=torch.int8, device=DEV), torch.ones(d_out, device=DEV), N, M, dX=dX)
    assert torch.equal(dX.float().cpu(), (torch.from_numpy(Weff).float() * gamma.cpu()).to(torch.bfloat16).float())


@pytest.mark.parametrize("N,M", [(2, 4), (3, 4)])
@pytest.mark.parametrize("d_out", [56, 64, 120, 136, 192, 200, 256, 264, 320, 392, 520])
def test_weights_of_every_stage_in_large_tiles(N, M, d_out):
    # as above where the device takes tiles of 256 x 256 (one round of them; of 128 x 128 it would be two, 1.4 times as long)
    tokens = d_in = 4096
    packed, gamma = hip_pack(sbn_synth.latent_weight(d_out, d_in, 1400 + d_out), N, M)
    Weff = torch.empty(d_out, d_in, dtype=torch.int8, device=DEV)
    sbn().sbn_unpack(packed, d_out, d_in, N, M, W_eff=Weff)
    t = torch.arange(tokens, device=DEV)
    dY = torch.zeros(tokens, d_out, dtype=torch.bfloat16, device=DEV)
    dY[t, (t * 7) % d_out] = 1.0                                        # dX[t, k] = gamma W_eff[7 t mod d_out, k]
    dX = torch.full((tokens, d_in), float("nan"), dtype=torch.bfloat16, device=DEV)
    backward(dY, packed, gamma, torch.zeros(tokens, d_in, dtype=torch.int8, device=DEV), torch.ones(tokens, device=DEV), N, M, dX=dX)
    assert torch.equal(dX, (Weff.float() * gamma).to(torch.bfloat16)[(t * 7) % d_out])
