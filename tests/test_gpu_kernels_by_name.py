"""GPU parity of the three forward kernels between which SBN_PATH_SMFMAC chooses by the sizes of a call (small block tiles, the
streaming kernel for decode batches, the persistent kernel on pieces of 512 rows), each asked for by name, so that its edges
are covered whatever that choice is: rows and tokens past a tile, rows that are no multiple of four, one and an odd number
of chunks, both weight forms, bias, accumulator output, more problems than one launch holds."""
import functools

import numpy as np
import pytest
import torch

import oracle
import sbn_synth
from gpu_util import DEV, hip_pack, oracle_pack, sbn

pytestmark = pytest.mark.gpu


@functools.lru_cache(maxsize=None)
def _weights(d_out, d_in, N, M, adversarial=False):
    W = (sbn_synth.adversarial_weight if adversarial else sbn_synth.latent_weight)(d_out, d_in, 8000 + d_out + d_in)
    _, gamma, Weff, _ = oracle_pack(W, N, M)
    return (*hip_pack(W, N, M), gamma, Weff)


@functools.lru_cache(maxsize=None)
def _reference(tokens, d_out, d_in, N, M, adversarial=False):
    X = (sbn_synth.adversarial_activations if adversarial else sbn_synth.activations)(tokens, d_in, 8100 + tokens + d_in)
    _, _, gamma, Weff = _weights(d_out, d_in, N, M, adversarial)
    y, acc, xq, sx = oracle.sparse_ternary_linear(X.float().numpy(), Weff, gamma)
    return torch.from_numpy(xq).to(DEV), torch.from_numpy(sx).to(DEV), y, acc


def _check(Y, y, bias, what):
    # the accumulator is exact: three roundings of the product (scale, accumulator to fp32, product), one of the sum with the bias
    b = 0.0 if bias is None else bias.cpu().numpy().astype(np.float64)[None, :]
    err = np.abs(Y.cpu().numpy().astype(np.float64) - (y + b))
    bound = 4 * 2.0 ** -24 * (np.abs(y) + np.abs(b))
    assert (err <= bound).all(), f"{what}: {(~(err <= bound)).sum()} values beyond the bound"


def _run(kernel, problems, N, M, bias=False, acc=False, adversarial=False):
    """problems: (tokens, d_out, d_in) of one call."""
    s = sbn()
    refs = [_reference(*p, N, M, adversarial) for p in problems]
    packs = [_weights(o, k, N, M, adversarial) for _, o, k in problems]
    Ys = [torch.full((t, o), float("nan"), dtype=torch.float32, device=DEV) for t, o, _ in problems]
    accs = [torch.full((t, o), -7, dtype=torch.int32, device=DEV) for t, o, _ in problems] if acc else None
    biases = [torch.randn(o, generator=torch.Generator().manual_seed(o)).to(DEV) for _, o, _ in problems] if bias else None
    s.sbn_test_linear_kernel(kernel, [r[0] for r in refs], [r[1] for r in refs], [p[0] for p in packs], [p[1] for p in packs], Ys, N, M,
                             biases, accs)
    torch.cuda.synchronize()
    for i, (p, r) in enumerate(zip(problems, refs)):
        _check(Ys[i], r[2], biases[i] if bias else None, f"problem {i} {p}")
        if acc:
            assert np.array_equal(accs[i].cpu().numpy(), r[3]), f"accumulators of problem {i} {p}"


SHAPES = [(1, 16, 128), (16, 256, 256), (40, 130, 384), (97, 64, 2560), (129, 64, 128), (129, 1100, 128), (200, 300, 384), (200, 514, 640),
          (300, 520, 1280), (512, 1030, 128),
          # beyond 512 tokens the persistent kernel deals its pieces from a list
          (513, 520, 640), (600, 1030, 384), (1100, 515, 640), (2100, 70, 128)]


@pytest.mark.parametrize("N,M", [(2, 4), (8, 8)])
@pytest.mark.parametrize("problem", SHAPES)
@pytest.mark.parametrize("bias,acc", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("kernel", ["TILES", "PIECES"])
def test_kernel_edges(kernel, problem, N, M, bias, acc):
    _run(getattr(sbn(), "SBN_KERNEL_" + kernel), [problem], N, M, bias, acc)


@pytest.mark.parametrize("N,M", [(2, 4), (8, 8)])
@pytest.mark.parametrize("problem", [(1, 4, 128), (16, 256, 256), (17, 132, 384), (32, 1100, 640), (33, 520, 128), (64, 2052, 1280), (48, 64, 2560),
                                     (20, 65600, 128), (60, 65540, 256)])   # the last two: strips of 256 rows
def test_streaming_kernel_edges(problem, N, M):
    _run(sbn().SBN_KERNEL_STREAM, [problem], N, M)


@pytest.mark.parametrize("N,M", [(2, 4), (8, 8)])
@pytest.mark.parametrize("kernel", ["TILES", "STREAM", "PIECES"])
def test_kernel_adversarial_inputs(kernel, N, M):
    _run(getattr(sbn(), "SBN_KERNEL_" + kernel), [(64, 256, 512)], N, M, adversarial=True)


@pytest.mark.parametrize("N,M", [(2, 4), (8, 8)])
@pytest.mark.parametrize("kernel,count", [("TILES", 3), ("TILES", 91), ("PIECES", 3), ("PIECES", 71), ("STREAM", 10), ("STREAM", 131)])
def test_kernel_groups(kernel, count, N, M):
    # unequal problems in one call: token counts that are no multiple of a unit, ragged last rows, and, in the long calls, more
    # problems than a launch holds (40 tiles, 32 or 8 of the pieces, 56 of the stream); the pieces: both ways of dealing in turn
    base = [(1100, 256), (520, 384), (64, 128), (2052, 128)] if kernel == "STREAM" else [(1100, 256), (518, 384), (64, 128)]
    toks = {"TILES": [17, 64, 100, 128, 200, 257, 600, 33], "PIECES": [17, 64, 100, 128, 200, 257, 512, 33] + [600] * 11 + [40],
            "STREAM": [17, 64, 33, 20, 48, 32, 1, 16, 64, 64]}[kernel]
    problems = [(toks[i % len(toks)], *base[i % len(base)]) for i in range(count)]
    _run(getattr(sbn(), "SBN_KERNEL_" + kernel), problems, N, M, bias=kernel != "STREAM" and count == 3)


@pytest.mark.parametrize("N,M", [(2, 4), (8, 8)])
@pytest.mark.parametrize("tokens", [33, 600])
@pytest.mark.parametrize("d_in", [1 << 17, (1 << 17) + 128])
def test_pieces_longest_sums(N, M, tokens, d_in):
    # the pieces multiply by 64 times the codes up to rows of 2^17 values, beyond by the codes: the largest sums there are, on either side
    s, d_out = sbn(), 70
    W = torch.full((d_out, d_in), 0.02, dtype=torch.bfloat16)
    W[1] = -W[1]
    W[2, ::3] = 0.0
    packed, gamma = hip_pack(W, N, M)
    _, g, Weff, _ = oracle_pack(W, N, M)
    xq = torch.from_numpy(np.random.default_rng(d_in).integers(-128, 128, (tokens, d_in), dtype=np.int8))
    xq[0], xq[1], xq[2] = -128, 127, 0
    sx = torch.full((tokens,), 30.0)
    Y, acc = torch.full((tokens, d_out), float("nan"), device=DEV), torch.full((tokens, d_out), -7, dtype=torch.int32, device=DEV)
    s.sbn_test_linear_kernel(s.SBN_KERNEL_PIECES, [xq.to(DEV)], [sx.to(DEV)], [packed], [gamma], [Y], N, M, None, [acc])
    Y2 = torch.full_like(Y, float("nan"))   # whole rows leave on another path where no accumulators are wanted
    s.sbn_test_linear_kernel(s.SBN_KERNEL_PIECES, [xq.to(DEV)], [sx.to(DEV)], [packed], [gamma], [Y2], N, M)
    kept, which = np.unique(Weff, axis=0, return_inverse=True)   # few different rows
    want = (xq.double() @ torch.from_numpy(kept).double().T).numpy().astype(np.int64)[:, which.reshape(-1)]   # exact: below 2^53
    assert np.abs(want).max() == 128 * d_in * N // M
    assert np.array_equal(acc.cpu().numpy(), want)
    _check(Y, want * float(g) / 30.0, None, "Y")
    assert torch.equal(Y, Y2)


@pytest.mark.parametrize("N,M", [(2, 4), (8, 8)])
def test_pieces_scales_below_the_normal_range(N, M):
    # gamma / s_x near and below the smallest normal number: the same two roundings as in the plain formula
    s, (tokens, d_out, d_in) = sbn(), (96, 128, 256)
    packed, gamma, _, Weff = _weights(d_out, d_in, N, M)
    xq, _, _, acc = _reference(tokens, d_out, d_in, N, M)
    sx = torch.full((tokens,), 30.0)
    sx[5:40] = torch.logspace(27, 38.4, 35)
    Y = torch.full((tokens, d_out), float("nan"), device=DEV)
    s.sbn_test_linear_kernel(s.SBN_KERNEL_PIECES, [xq], [sx.to(DEV)], [packed], [gamma], [Y], N, M)
    scale = (gamma.cpu().numpy() / sx.numpy()).astype(np.float32)
    assert (scale < 2.0 ** -126).any()
    assert np.array_equal(Y.cpu().numpy(), acc.astype(np.float32) * scale[:, None])


@pytest.mark.parametrize("N,M", [(2, 4), (8, 8)])
@pytest.mark.parametrize("problems", [
    [(9000, 6000, 128)], [(9100, 5000, 256)], [(9000, 6000, 384)], [(8200, 6500, 640)],     # 1, 2, 3, 5 chunks: fewer than the ring, odd counts
    [(4000, 3000, 640), (4000, 2600, 640), (5000, 3001, 640)],                              # rows of one length, others' outputs
    [(3000, 4000, 384), (4100, 3000, 512), (2000, 2100, 128), (3333, 4444, 512)],           # the stream of requests is started anew in between
    [(700, 1100, 384), (650, 900, 384), (97 * 8, 600, 896)],                                # from a list: pieces of all widths behind each other
    [(8200, 6148, 128)], [(4100, 2564, 256), (700, 1496, 128)],                              # rows of outputs of no whole 64 bytes, in the caches
    [(512, 13000, 128), (65, 17, 256)], [(300, 4700, 384), (512, 6001, 128), (100, 9000, 256)], [(33, 2000, 128)],   # decode batches: runs of uneven length, few blocks
])
def test_pieces_one_behind_the_other(N, M, problems):
    s = sbn()
    xqs, sxs, packs, Ys, refs = [], [], [], [], []
    for i, (t, o, k) in enumerate(problems):
        gen = torch.Generator(device=DEV).manual_seed(17 * i + t)
        packed, gamma = hip_pack(sbn_synth.latent_weight(o, k, 8200 + i), N, M)
        Weff = torch.zeros((o, k), dtype=torch.int8, device=DEV)
        s.sbn_unpack(packed, o, k, N, M, Weff)
        xq = torch.randint(-128, 128, (t, k), generator=gen, device=DEV, dtype=torch.int8)
        sx = torch.rand(t, generator=gen, device=DEV) * 50 + 10
        xqs.append(xq); sxs.append(sx); packs.append((packed, gamma))
        Ys.append(torch.full((t, o), float("nan"), device=DEV))
        # sums below 2^24 are exact in fp32 whatever their order; then the formula's two roundings
        acc = xq.float() @ Weff.float().T
        assert k * 128 < 1 << 24
        refs.append(acc * (gamma / sx)[:, None])
    s.sbn_test_linear_kernel(s.SBN_KERNEL_PIECES, xqs, sxs, [p[0] for p in packs], [p[1] for p in packs], Ys, N, M)
    for Y, ref in zip(Ys, refs):
        assert torch.equal(Y, ref)


@pytest.mark.parametrize("N,M", [(2, 4), (8, 8)])
@pytest.mark.parametrize("offset", [0, 16, 32, 48, 64])
@pytest.mark.parametrize("tokens,d_out,bias", [(600, 1024, False), (1100, 528, True), (97, 80, True)])
def test_pieces_outputs_that_begin_anywhere(N, M, offset, tokens, d_out, bias):
    # whole sectors of 64 bytes leave on one path, runs that share theirs on another: the same values, and nothing beside the outputs
    s, d_in = sbn(), 384
    packed, gamma, _, _ = _weights(d_out, d_in, N, M)
    xq, sx, _, acc = _reference(tokens, d_out, d_in, N, M)
    b = torch.randn(d_out, generator=torch.Generator().manual_seed(d_out)).to(DEV) if bias else None
    buf = torch.full((32 + tokens * d_out + 32,), float("nan"), device=DEV)
    assert buf.data_ptr() % 64 == 0
    Y = buf[offset // 4:offset // 4 + tokens * d_out].view(tokens, d_out)
    s.sbn_test_linear_kernel(s.SBN_KERNEL_PIECES, [xq], [sx], [packed], [gamma], [Y], N, M, [b] if bias else None)
    want = acc.astype(np.float32) * (gamma.cpu().numpy() / sx.cpu().numpy())[:, None]
    assert np.array_equal(Y.cpu().numpy(), want if b is None else want + b.cpu().numpy())
    assert buf.isnan().sum() == 64


@pytest.mark.parametrize("tokens,d_out,d_in", [(33000, 4100, 2048), (33000, 4100, 256), (33000, 4096, 256), (8200, 2064, 256)])
def test_pieces_many_outputs_with_a_bias(tokens, d_out, d_in):
    # more than 512 MB: past the caches in runs (long rows of no whole sectors), through them, past them in tiles; 68 MB of whole sectors
    # and short rows of inputs: through them in runs
    s = sbn()
    packed, gamma = hip_pack(sbn_synth.latent_weight(d_out, d_in, 8300), 2, 4)
    Weff = torch.zeros((d_out, d_in), dtype=torch.int8, device=DEV)
    s.sbn_unpack(packed, d_out, d_in, 2, 4, Weff)
    gen = torch.Generator(device=DEV).manual_seed(d_in)
    xq = torch.randint(-128, 128, (tokens, d_in), generator=gen, device=DEV, dtype=torch.int8)
    sx, bias = torch.rand(tokens, generator=gen, device=DEV) * 50 + 10, torch.randn(d_out, generator=gen, device=DEV)
    Y = torch.full((tokens, d_out), float("nan"), device=DEV)
    s.sbn_test_linear_kernel(s.SBN_KERNEL_PIECES, [xq], [sx], [packed], [gamma], [Y], 2, 4, [bias])
    want = (xq.float() @ Weff.float().T) * (gamma / sx)[:, None]   # sums below 2^24, exact in fp32
    assert torch.equal(Y, want + bias)


@pytest.mark.parametrize("N,M", [(2, 4), (8, 8)])
@pytest.mark.parametrize("tokens", [1, 2, 31, 66, 545])
@pytest.mark.parametrize("d_out", [1, 31, 33, 63, 65, 127, 515, 68, 124, 572])
def test_pieces_widths_past_whole_tiles(N, M, tokens, d_out):
    # odd widths and accumulators leave a word at a time, a ragged last wavefront of whole vectors with the others; nothing beside them
    s, d_in = sbn(), 256
    packed, gamma, _, _ = _weights(d_out, d_in, N, M)
    xq, sx, _, acc = _reference(tokens, d_out, d_in, N, M)
    b = torch.randn(d_out, generator=torch.Generator().manual_seed(d_out)).to(DEV)
    want = acc.astype(np.float32) * (gamma.cpu().numpy() / sx.cpu().numpy())[:, None]
    for bias in (None, b):
        for with_acc in (False, True):
            buf = torch.full((tokens * d_out + 256,), float("nan"), device=DEV)
            sums = torch.full((tokens * d_out + 256,), -7, dtype=torch.int32, device=DEV)
            s.sbn_test_linear_kernel(s.SBN_KERNEL_PIECES, [xq], [sx], [packed], [gamma], [buf[:tokens * d_out].view(tokens, d_out)], N, M,
                                     None if bias is None else [bias], [sums[:tokens * d_out].view(tokens, d_out)] if with_acc else None)
            got = buf.cpu().numpy()
            assert np.array_equal(got[:-256].reshape(tokens, d_out), want if bias is None else want + b.cpu().numpy()) and np.isnan(got[-256:]).all()
            if with_acc:
                assert np.array_equal(sums[:-256].view(tokens, d_out).cpu().numpy(), acc) and (sums[-256:] == -7).all()
