"""GPU parity of single decode calls whose blocks quantize the token rows themselves, at the edges of that kernel: wavefronts and
super-steps, the two token-slot forms, one and two row tiles per block, and just past each line to the separate quantizer.
The accumulators are exact, so Y is within three fp32 roundings of the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import sbn_synth
from gpu_util import DEV, assert_rel, hip_pack, oracle_pack, sbn

pytestmark = pytest.mark.gpu
Y_TOL = 4 * 2.0 ** -24


@pytest.mark.parametrize("N,M", [(2, 4), (8, 8), (1, 4)])
@pytest.mark.parametrize("tokens", [1, 2, 3, 15, 16])
@pytest.mark.parametrize("d_out,d_in", [(16, 128), (50, 520), (33, 2176), (6420, 640), (24, 8192), (24, 8320)])
def test_single_call_quantizes_its_rows(N, M, tokens, d_out, d_in):
    s = sbn()
    W = sbn_synth.latent_weight(d_out, d_in, 6000 + d_out + d_in)
    X = sbn_synth.adversarial_activations(tokens, d_in, 6001 + tokens)
    packed, gamma = hip_pack(W, N, M)
    _, g, Weff, _ = oracle_pack(W, N, M)
    y, *_ = oracle.sparse_ternary_linear(X.float().numpy(), Weff, g)
    Y = torch.full((tokens, d_out), float("nan"), dtype=torch.float32, device=DEV)
    ws = s.new_workspace(s.sbn_workspace_bytes(s.SBN_OP_LINEAR, tokens, d_out, d_in, N, M))
    s.sbn_sparse_ternary_linear(X.to(DEV), packed, gamma, Y, N, M, ws)
    torch.cuda.synchronize()
    assert_rel(Y.cpu().numpy(), y, Y_TOL, f"{tokens} x {d_in} -> {d_out} at {N}:{M}")


@pytest.mark.parametrize("N,M", [(2, 4), (1, 4)])
@pytest.mark.parametrize("tokens", [4, 5, 7, 8, 9, 11, 12, 13, 14])
@pytest.mark.parametrize("d_out,d_in", [(50, 520), (33, 2176), (40, 4096), (24, 6912)])
def test_single_call_token_slots(N, M, tokens, d_out, d_in):
    # two, four, eight, twelve and sixteen token slots, filled and not; wavefronts of one to four groups of four
    test_single_call_quantizes_its_rows(N, M, tokens, d_out, d_in)


@pytest.mark.parametrize("N,M", [(2, 4), (8, 8), (1, 4)])
@pytest.mark.parametrize("tokens", [1, 2, 4, 5])
@pytest.mark.parametrize("d_out,d_in", [(40, 8200), (6420, 8704), (18, 16384), (33, 16512), (24, 24704), (16, 32768), (24, 32776)])
def test_single_call_of_long_rows(N, M, tokens, d_out, d_in):
    # up to four tokens: two super-steps per wavefront up to 16384, four up to 32768, past that and from five tokens on the
    # separate quantizer; last super-steps of one chunk, of a whole round of wavefronts without any
    test_single_call_quantizes_its_rows(N, M, tokens, d_out, d_in)


def test_grouped_call_of_unequal_rounds():
    # one launch: rows of one super-step beside rows of 52, so wavefronts of the first have none in any round
    s = sbn()
    shapes = [(2, 40, 128), (1, 130, 26368), (2, 16, 8192)]
    Ws = [sbn_synth.latent_weight(o, k, 6200 + o) for _, o, k in shapes]
    Xs = [sbn_synth.adversarial_activations(t, k, 6201 + k) for t, _, k in shapes]
    packs = [hip_pack(W, 2, 4) for W in Ws]
    Ys = [torch.full((t, o), float("nan"), dtype=torch.float32, device=DEV) for t, o, _ in shapes]
    ws = s.new_workspace(sum(s.sbn_workspace_bytes(s.SBN_OP_LINEAR, t, o, k, 2, 4) for t, o, k in shapes))
    s.sbn_sparse_ternary_linear_grouped([X.to(DEV) for X in Xs], [p for p, _ in packs], [g for _, g in packs], Ys, 2, 4, ws)
    torch.cuda.synchronize()
    for W, X, Y in zip(Ws, Xs, Ys):
        _, g, Weff, _ = oracle_pack(W, 2, 4)
        y, *_ = oracle.sparse_ternary_linear(X.float().numpy(), Weff, g)
        assert_rel(Y.cpu().numpy(), y, Y_TOL, f"{tuple(Y.shape)}")


def test_grouped_call_of_unequal_problems():
    # one launch: input dimensions of one to seven super-steps and token counts of one to nine side by side
    s = sbn()
    shapes = [(3, 40, 128), (9, 130, 3584), (1, 16, 640)]
    Ws = [sbn_synth.latent_weight(o, k, 6100 + o) for _, o, k in shapes]
    Xs = [sbn_synth.activations(t, k, 6101 + k) for t, _, k in shapes]
    packs = [hip_pack(W, 2, 4) for W in Ws]
    Ys = [torch.full((t, o), float("nan"), dtype=torch.float32, device=DEV) for t, o, _ in shapes]
    ws = s.new_workspace(sum(s.sbn_workspace_bytes(s.SBN_OP_LINEAR, t, o, k, 2, 4) for t, o, k in shapes))
    s.sbn_sparse_ternary_linear_grouped([X.to(DEV) for X in Xs], [p for p, _ in packs], [g for _, g in packs], Ys, 2, 4, ws)
    torch.cuda.synchronize()
    for W, X, Y in zip(Ws, Xs, Ys):
        _, g, Weff, _ = oracle_pack(W, 2, 4)
        y, *_ = oracle.sparse_ternary_linear(X.float().numpy(), Weff, g)
        assert_rel(Y.cpu().numpy(), y, Y_TOL, f"{tuple(Y.shape)}")
