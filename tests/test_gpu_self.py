"""GPU parity of the kernel that quantizes the activations itself (calls of a few problems and tokens that want no quantized rows back)
against the oracle: every shape at its edges (rows and tokens past a block, output rows of no whole 16 bytes, input dimensions of
one chunk, of no whole super-step, of no whole chunk, of the longest row), both weight forms, bias, accumulators, several
problems in a call, and the public calls that take it."""
import functools

import numpy as np
import pytest
import torch

import oracle
import sbn_synth
from gpu_util import DEV, hip_pack, oracle_pack, sbn

pytestmark = pytest.mark.gpu
FORMS = range(8)


@functools.lru_cache(maxsize=None)
def _problem(tokens, d_out, d_in, N, M, adversarial=False):
    W = (sbn_synth.adversarial_weight if adversarial else sbn_synth.latent_weight)(d_out, d_in, 8200 + d_out + d_in)
    X = (sbn_synth.adversarial_activations if adversarial else sbn_synth.activations)(tokens, d_in, 8300 + tokens + d_in)
    _, gamma, Weff, _ = oracle_pack(W, N, M)
    y, acc, _, _ = oracle.sparse_ternary_linear(X.float().numpy(), Weff, gamma)
    return (X.to(DEV), *hip_pack(W, N, M), y, acc)


def _check(Y, y, bias, what):
    # the accumulator is exact: three roundings of the product (scale, accumulator to fp32, product), one of the sum with the bias
    b = 0.0 if bias is None else bias.cpu().numpy().astype(np.float64)[None, :]
    err = np.abs(Y.cpu().numpy().astype(np.float64) - (y + b))
    bound = 4 * 2.0 ** -24 * (np.abs(y) + np.abs(b))
    assert (err <= bound).all(), f"{what}: {(~(err <= bound)).sum()} values beyond the bound"


def _run(form, problems, N, M, bias=False, acc=False, adversarial=False):
    """problems: (tokens, d_out, d_in) of one call."""
    ps = [_problem(*p, N, M, adversarial) for p in problems]
    Ys = [torch.full((t, o), float("nan"), dtype=torch.float32, device=DEV) for t, o, _ in problems]
    accs = [torch.full((t, o), -7, dtype=torch.int32, device=DEV) for t, o, _ in problems] if acc else None
    biases = [torch.randn(o, generator=torch.Generator().manual_seed(o)).to(DEV) for _, o, _ in problems] if bias else None
    sbn().sbn_test_self_kernel(form, [p[0] for p in ps], [p[1] for p in ps], [p[2] for p in ps], Ys, N, M, biases, accs)
    torch.cuda.synchronize()
    for i, (p, ref) in enumerate(zip(problems, ps)):
        _check(Ys[i], ref[3], biases[i] if bias else None, f"problem {i} {p}")
        if acc:
            assert np.array_equal(accs[i].cpu().numpy(), ref[4]), f"accumulators of problem {i} {p}"


SHAPES = [(1, 16, 128), (4, 33, 256), (5, 130, 384), (8, 64, 512), (9, 257, 640), (16, 95, 1024), (17, 97, 2560), (31, 514, 1280), (64, 300, 2688),
          (33, 259, 4096), (12, 70, 5120), (50, 150, 1000), (20, 40, 72), (24, 64, 4104)]


@pytest.mark.parametrize("N,M", [(2, 4), (8, 8)])
@pytest.mark.parametrize("problem", SHAPES)
@pytest.mark.parametrize("bias,acc", [(False, False), (True, True)])
@pytest.mark.parametrize("form", FORMS)
def test_shape_edges(form, problem, N, M, bias, acc):
    _run(form, [problem], N, M, bias, acc)


@pytest.mark.parametrize("N,M", [(2, 4), (8, 8)])
@pytest.mark.parametrize("form", FORMS)
def test_longest_rows(form, N, M):
    if form >= 6:   # sixteen rows of 8192 values and the weights of sixteen wavefronts do not fit a multiprocessor
        with pytest.raises(sbn().SbnError):
            _run(form, [(20, 300, 8192)], N, M)
        return
    _run(form, [(20, 300, 8192)], N, M)
    _run(form, [(7, 70, 8184)], N, M)


@pytest.mark.parametrize("N,M", [(2, 4), (8, 8)])
@pytest.mark.parametrize("form", FORMS)
def test_adversarial_inputs_and_groups(form, N, M):
    _run(form, [(64, 256, 512)], N, M, adversarial=True)
    _run(form, [(17, 1100, 256), (40, 64, 384), (3, 518, 128), (64, 30, 2560), (1, 16, 256), (16, 200, 640), (9, 33, 128), (33, 95, 512)], N, M, bias=True, acc=True)
    # more blocks than multiprocessors: less of the weights in LDS at a time
    _run(form, [(72, 2100, 2560)], N, M)


@pytest.mark.parametrize("N,M", [(2, 4), (6, 8), (8, 8), (1, 4), (2, 8)])
@pytest.mark.parametrize("tokens,d_out,d_in", [(4, 16388, 512), (6, 300, 1024), (16, 130, 2560), (17, 130, 2560), (50, 1500, 1000), (64, 512, 8192),
                                               (128, 257, 768)])
def test_public_call_equals_its_two_steps(tokens, d_out, d_in, N, M):
    # quantized rows asked for: the quantizer's launch and the kernels on quantized rows; not asked for: one launch.  Bit for bit.
    s = sbn()
    X, packed, gamma, y, _ = _problem(tokens, d_out, d_in, N, M)
    ws = s.new_workspace(s.sbn_workspace_bytes(s.SBN_OP_LINEAR, tokens, d_out, d_in, N, M))
    Y = [torch.full((tokens, d_out), float("nan"), device=DEV) for _ in range(2)]
    s.sbn_sparse_ternary_linear(X, packed, gamma, Y[0], N, M, ws)
    xq, sx = torch.zeros(tokens, d_in, dtype=torch.int8, device=DEV), torch.zeros(tokens, device=DEV)
    s.sbn_sparse_ternary_linear(X, packed, gamma, Y[1], N, M, ws, xq_out=xq, sx_out=sx)
    torch.cuda.synchronize()
    assert torch.equal(Y[0], Y[1])
    _check(Y[0], y, None, "public call")


def test_grouped_call_and_its_replay():
    s = sbn()
    ps = [_problem(40, o, 2560, 2, 4) for o in (130, 514, 64)]
    X = ps[0][0]
    Ws = [(p[1], p[2]) for p in ps]
    Ys = [torch.full((40, o), float("nan"), device=DEV) for o in (130, 514, 64)]
    ws = s.new_workspace(sum(s.sbn_workspace_bytes(s.SBN_OP_LINEAR, 40, o, 2560, 2, 4) for o in (130, 514, 64)))
    group = s.LinearGroup([X] * 3, [w[0] for w in Ws], [w[1] for w in Ws], Ys, 2, 4, ws)
    group.run()
    torch.cuda.synchronize()
    for Y, p in zip(Ys, ps):
        _check(Y, p[3], None, "grouped call")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        group.run()
    for i in range(3):   # other activations at every replay
        X2 = sbn_synth.activations(40, 2560, 8400 + i).to(DEV)
        keep = X.clone()
        X.copy_(X2)
        for Y in Ys:
            Y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        got = [Y.clone() for Y in Ys]
        group.run()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, Ys)) and not any(torch.isnan(a).any() for a in got)
        X.copy_(keep)


@pytest.mark.parametrize("N,M", [(2, 4), (8, 8)])
@pytest.mark.parametrize("tokens,d_in", [(17, 2560), (64, 2560), (200, 512)])
def test_outputs_in_the_place_of_the_rows(tokens, d_in, N, M):
    # beyond 16 tokens Y may lie over X, whole or in part: the rows are quantized before anything is written
    s = sbn()
    d_out = d_in // 2
    X, packed, gamma, y, _ = _problem(tokens, d_out, d_in, N, M)
    ws = s.new_workspace(2 * s.sbn_workspace_bytes(s.SBN_OP_LINEAR, tokens, d_out, d_in, N, M))
    Y = X.clone().view(torch.float32)
    s.sbn_sparse_ternary_linear(Y.view(torch.bfloat16), packed, gamma, Y, N, M, ws)
    G = torch.cat([X, X]).view(torch.float32)
    Ys = [torch.full((tokens, d_out), float("nan"), device=DEV), G[tokens // 2 : tokens // 2 + tokens]]
    s.LinearGroup([G[:tokens].view(torch.bfloat16)] * 2, [packed] * 2, [gamma] * 2, Ys, N, M, ws).run()
    torch.cuda.synchronize()
    for got in (Y, *Ys):
        _check(got, y, None, "over the rows")


@pytest.mark.parametrize("N,M", [(2, 4), (8, 8)])
@pytest.mark.parametrize("form", FORMS)
def test_rows_that_are_not_finite_stay_alone(form, N, M):
    # what such a row gives is unspecified; here, as in the quantizer's own launch: an infinite or NaN scale's quotient, rows of zeros (the
    # low byte of a quiet NaN and of 0 + 1.5 * 2^23), so NaN outputs and accumulators of zero.  The other rows do not notice
    s = sbn()
    tokens, d_out, d_in = 21, 130, 1000
    X, packed, gamma, y, acc = _problem(tokens, d_out, d_in, N, M)
    X = X.clone()
    bad = {3: float("inf"), 7: float("-inf"), 8: float("nan"), 20: float("nan")}
    for row, v in bad.items():
        X[row, 17 * row] = v
    X[8, 5] = float("inf")
    Y = torch.full((tokens, d_out), 7.0, device=DEV)
    got = torch.full((tokens, d_out), -7, dtype=torch.int32, device=DEV)
    s.sbn_test_self_kernel(form, [X], [packed], [gamma], [Y], N, M, None, [got])
    xq, sx = torch.full((tokens, d_in), 5, dtype=torch.int8, device=DEV), torch.full((tokens,), 5.0, device=DEV)
    s.sbn_act_quant(X, xq, sx)
    torch.cuda.synchronize()
    rows, fine = list(bad), [t for t in range(tokens) if t not in bad]
    assert Y[rows].isnan().all() and (got[rows] == 0).all() and (xq[rows] == 0).all()
    assert (sx[[3, 7]] == 0).all() and sx[[8, 20]].isnan().all()
    _check(Y[fine], y[fine], None, "finite rows")
    assert np.array_equal(got[fine].cpu().numpy(), acc[fine])
