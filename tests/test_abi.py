"""Host-side checks of the C ABI that need no GPU: the library loads, exports every symbol the
header declares, answers the size queries, and rejects bad arguments before launching anything."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "sbn.h")
PROBE_HEADER = os.path.join(ROOT, "include", "sbn_probe.h")


@pytest.fixture(scope="module")
def sbn():
    import paper_2603_05168_amd as m
    return m


def declared_functions(header=HEADER):
    text = open(header).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(sbn_[a-z0-9_]+)\s*\(", text)))


def test_header_declares_the_boundary():
    names = declared_functions()
    for must in ("sbn_quantize_mask_pack", "sbn_sparse_ternary_linear", "sbn_sparse_ternary_linear_backward",
                 "sbn_sparse_ternary_linear_backward_grouped",
                 "sbn_packed_bytes", "sbn_workspace_bytes", "sbn_unpack", "sbn_last_error"):
        assert must in names


def test_library_exports_every_declared_symbol(sbn):
    lib = ctypes.CDLL(sbn.lib_path())
    for name in declared_functions():
        assert hasattr(lib, name), f"{name} is declared in include/sbn.h but not exported"
    for name in declared_functions():
        assert hasattr(sbn, name), f"{name} has no Python binding of the same name"


def test_every_header_is_covered_and_the_probe_library_exports_its_symbol():
    # include/ holds exactly the layer's header and the benchmark probes' header, each with a library of its own
    assert sorted(os.listdir(os.path.join(ROOT, "include"))) == ["sbn.h", "sbn_probe.h"]
    from paper_2603_05168_amd import probe
    lib = ctypes.CDLL(probe.lib_path())
    names = declared_functions(PROBE_HEADER)
    assert names == ["sbn_ceiling_probe"]
    for name in names:
        assert hasattr(lib, name) and hasattr(probe, name)
    assert "sbn_ceiling_probe" not in declared_functions()       # measurement support stays out of the layer's boundary


def test_spin_limit_hook_is_callable_without_a_gpu(sbn):
    sbn.sbn_test_set_spin_limits(0, -1)
    sbn.sbn_test_set_spin_limits()


@pytest.mark.parametrize("N,M", [(2, 4), (8, 8)])
def test_choice_between_the_forward_kernels(sbn, N, M):
    # sizes at which the kernels measure far apart (on 256 multiprocessors, which the library assumes without a GPU)
    tiles, stream, pieces = sbn.SBN_KERNEL_TILES, sbn.SBN_KERNEL_STREAM, sbn.SBN_KERNEL_PIECES
    for problem in ((17, 2560, 2560), (64, 6912, 2560), (256, 2560, 6912), (384, 1024, 4096), (512, 2560, 2560), (1024, 6912, 2560)):
        assert sbn.sbn_test_chosen_kernels([problem], N, M) == [tiles], problem
    for problem in ((3000, 2560, 2560), (777, 2560, 6912), (2048, 1024, 4096), (1500, 768, 3072), (16384, 768, 6912)):
        assert sbn.sbn_test_chosen_kernels([problem], N, M) == [pieces], problem
    assert sbn.sbn_test_chosen_kernels([(32, 2560, 6912)] * 64, N, M) == [stream] * 64
    # output rows of no whole 16 bytes are stored in words, which costs the pieces more (2181 tokens, 512 -> 475: 11.4 us against
    # 7.6; 512 -> 6911 at 8000: 179 against 111); few rows of outputs on many long rows of tokens cost the tiles more (8000
    # tokens, 6912 -> 512: 64 us against 33)
    for problem in ((2181, 512, 475), (4000, 512, 2559), (8000, 512, 6911), (1000, 2560, 2559), (500, 2560, 6911)):
        assert sbn.sbn_test_chosen_kernels([problem], N, M) == [tiles], problem
    for problem in ((8000, 6912, 512), (8000, 6912, 476), (8000, 2560, 512)):
        assert sbn.sbn_test_chosen_kernels([problem], N, M) == [pieces], problem
    # a long shallow layer beside a deep one of a few tokens: every problem counts with its own input dimension (278 us in tiles,
    # 158 this way)
    assert sbn.sbn_test_chosen_kernels([(16384, 768, 6912), (17, 8192, 768)], N, M) == [pieces, stream]
    assert sbn.sbn_test_chosen_kernels([(200, 2560, 2560)] * 3, N, M) == [tiles] * 3
    # 128 tokens of 2^25 values are more bytes than the pieces can address; a call's problems are of one kernel
    for tokens in (97, 600, 4096):
        for d_out in (8, 1000, 8000):
            assert sbn.sbn_test_chosen_kernels([(tokens, 1 << 25, d_out)], N, M) == [tiles] and not sbn.sbn_test_takes_blocks([(tokens, 1 << 25, d_out)], N, M)
    assert sbn.sbn_test_chosen_kernels([(3000, 2560, 2560), (128, 1 << 25, 8)], N, M) == [tiles] * 2


def test_packed_bytes(sbn):
    assert sbn.sbn_packed_bytes(6912, 2560, 2, 4) == 6912 * 2560 // 4
    assert sbn.sbn_packed_bytes(6912, 2560, 1, 4) == 6912 * 2560 // 8
    assert sbn.sbn_packed_bytes(2560, 6912, 2, 8) == 2560 * 6912 * 5 // 32
    assert sbn.sbn_packed_bytes(3, 8, 2, 4) == 3 * 32            # one zero-padded chunk per row
    assert sbn.sbn_packed_bytes(16, 256, 8, 8) == 16 * 256 // 4  # dense ternary: 2 bits per weight, no indices


def test_packed_bytes_matches_oracle_layout(sbn):
    import oracle
    for N, M in ((2, 4), (1, 4), (2, 8), (6, 8), (4, 4), (1, 2), (7, 8)):
        for d_in in (8, 128, 136, 2560):
            assert sbn.sbn_packed_bytes(24, d_in, N, M) == oracle.packed_bytes(24, d_in, N, M)


@pytest.mark.parametrize("args", [(0, 256, 2, 4), (16, 0, 2, 4), (16, 130, 2, 4), (16, 256, 0, 4), (16, 256, 5, 4),
                                  (16, 256, 2, 3), (16, 256, 2, 16)])
def test_bad_shapes_are_einval(sbn, args):
    with pytest.raises(sbn.SbnError) as e:
        sbn.sbn_packed_bytes(*args)
    assert e.value.status == sbn.SBN_EINVAL


def test_workspace_queries(sbn):
    for op in (sbn.SBN_OP_QUANTIZE_MASK_PACK, sbn.SBN_OP_LINEAR, sbn.SBN_OP_BACKWARD, sbn.SBN_OP_MASK_FLIPS):
        assert sbn.sbn_workspace_bytes(op, 16, 256, 256, 2, 4) > 0
    with pytest.raises(sbn.SbnError):
        sbn.sbn_workspace_bytes(7, 16, 256, 256, 2, 4)
    with pytest.raises(sbn.SbnError):
        sbn.sbn_workspace_bytes(sbn.SBN_OP_LINEAR, 0, 256, 256, 2, 4)


def test_argument_errors_come_before_any_launch(sbn):
    """Null and misaligned pointers, short workspaces and unsupported requests return their status
    on the host; no GPU is present here, so reaching a launch would fail differently."""
    lib = ctypes.CDLL(sbn.lib_path())
    lib.sbn_quantize_mask_pack.restype = ctypes.c_int
    lib.sbn_sparse_ternary_linear.restype = ctypes.c_int
    lib.sbn_sparse_ternary_linear_backward.restype = ctypes.c_int
    vp, i64, ci, sz = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int, ctypes.c_size_t
    A = 0x10000  # fake, aligned, never dereferenced on the host
    # null packed
    assert lib.sbn_quantize_mask_pack(vp(A), ci(1), i64(16), i64(256), i64(256), ci(2), ci(4), vp(0), vp(A), vp(A),
                                      sz(1 << 20), vp(0)) == sbn.SBN_EINVAL
    # ld_w < d_in
    assert lib.sbn_quantize_mask_pack(vp(A), ci(1), i64(16), i64(256), i64(128), ci(2), ci(4), vp(A), vp(A), vp(A),
                                      sz(1 << 20), vp(0)) == sbn.SBN_EINVAL
    # misaligned packed
    assert lib.sbn_quantize_mask_pack(vp(A), ci(1), i64(16), i64(256), i64(256), ci(2), ci(4), vp(A + 4), vp(A), vp(A),
                                      sz(1 << 20), vp(0)) == sbn.SBN_EALIGN
    # workspace too small
    assert lib.sbn_quantize_mask_pack(vp(A), ci(1), i64(16), i64(256), i64(256), ci(2), ci(4), vp(A), vp(A), vp(A),
                                      sz(8), vp(0)) == sbn.SBN_ESIZE
    lin = lambda **kw: lib.sbn_sparse_ternary_linear(  # noqa: E731
        vp(kw.get("X", A)), i64(kw.get("tokens", 8)), i64(kw.get("d_in", 256)), i64(256), ci(kw.get("N", 2)),
        ci(kw.get("M", 4)), vp(A), vp(A), vp(0), vp(kw.get("Y", A)), vp(0), vp(0), vp(0), ci(kw.get("path", 0)), vp(A),
        sz(kw.get("ws", 1 << 24)), vp(0))
    assert lin(Y=0) == sbn.SBN_EINVAL
    assert lin(X=0) == sbn.SBN_EINVAL                       # no X and no pre-quantized inputs
    assert lin(X=A + 2) == sbn.SBN_EALIGN
    assert lin(path=9) == sbn.SBN_EINVAL
    assert lin(ws=16) == sbn.SBN_ESIZE
    assert lin(tokens=64, path=sbn.SBN_PATH_GEMV) == sbn.SBN_EUNSUPPORTED  # decode kernel takes <= 16 tokens
    assert lin(d_in=200, path=sbn.SBN_PATH_SMFMAC) == sbn.SBN_EUNSUPPORTED
    # backward: nothing requested
    assert lib.sbn_sparse_ternary_linear_backward(vp(A), i64(8), i64(256), i64(256), ci(2), ci(4), vp(A), vp(A), vp(A),
                                                  vp(A), vp(0), vp(0), ci(0), vp(A), sz(1 << 24), vp(0)) == sbn.SBN_EINVAL
    # backward: unknown flag bit
    assert lib.sbn_sparse_ternary_linear_backward(vp(A), i64(8), i64(256), i64(256), ci(2), ci(4), vp(A), vp(A), vp(A),
                                                  vp(A), vp(A), vp(A), ci(4), vp(A), sz(1 << 24), vp(0)) == sbn.SBN_EINVAL
    assert lin(d_in=200, path=sbn.SBN_PATH_DENSE_MFMA) == sbn.SBN_EUNSUPPORTED   # dense MFMA rows are multiples of 64
    # grouped backward: count out of range, null array, a layer that asks for nothing, short workspace, misaligned dY
    lib.sbn_sparse_ternary_linear_backward_grouped.restype = ctypes.c_int
    def bwd_grouped(count=2, dy=(A, A), dx=(A, A), dw=(A, A), ws=1 << 26, arrays_ok=True, flags=0):
        P = lambda vals: (vp * 2)(*[vp(v) if v else None for v in vals])   # noqa: E731
        I = lambda v: (i64 * 2)(v, v)                                       # noqa: E731
        return lib.sbn_sparse_ternary_linear_backward_grouped(
            ci(count), P(dy), I(8), I(256), I(256), ci(2), ci(4), P((A, A)), P((A, A)), P((A, A)), P((A, A)),
            P(dx) if arrays_ok else None, P(dw), ci(flags), vp(A), sz(ws), vp(0))
    assert bwd_grouped(count=0) == sbn.SBN_EINVAL
    assert bwd_grouped(count=9) == sbn.SBN_EINVAL
    assert bwd_grouped(arrays_ok=False) == sbn.SBN_EINVAL
    assert bwd_grouped(dx=(A, 0), dw=(A, 0)) == sbn.SBN_EINVAL
    assert bwd_grouped(flags=8) == sbn.SBN_EINVAL
    assert bwd_grouped(dy=(A, A + 2)) == sbn.SBN_EALIGN
    assert bwd_grouped(ws=1 << 12) == sbn.SBN_ESIZE
    # in-place pack with flip counts: null counters, misaligned counters, fp32 weights, a pattern and a row length
    # outside what the flip-counting kernels cover
    lib.sbn_quantize_mask_pack_flips_batched.restype = ctypes.c_int
    one_p, one_i = (vp * 1), (i64 * 1)

    def pflips(wdt=1, d_out=16, d_in=256, N=2, M=4, fl=A):
        return lib.sbn_quantize_mask_pack_flips_batched(ci(1), one_p(A), ci(wdt), one_i(d_out), one_i(d_in), ci(N), ci(M), one_p(A),
                                                        one_p(A), vp(fl), vp(A), sz(1 << 20), vp(0))
    assert pflips(fl=0) == sbn.SBN_EINVAL
    assert pflips(fl=A + 4) == sbn.SBN_EALIGN
    assert pflips(wdt=0) == sbn.SBN_EUNSUPPORTED
    assert pflips(N=6, M=8) == sbn.SBN_EUNSUPPORTED
    assert pflips(d_in=200) == sbn.SBN_EUNSUPPORTED
    # mask flips: null input, misaligned count, short workspace
    lib.sbn_mask_flips.restype = ctypes.c_int
    flips = lambda **kw: lib.sbn_mask_flips(  # noqa: E731
        vp(kw.get("a", A)), vp(A), i64(64), i64(256), ci(2), ci(4), vp(kw.get("out", A)), vp(A), sz(kw.get("ws", 1 << 16)), vp(0))
    assert flips(a=0) == sbn.SBN_EINVAL
    assert flips(out=A + 4) == sbn.SBN_EALIGN
    assert flips(ws=8) == sbn.SBN_ESIZE
    # conversion of packed forms: null, target that cannot hold the pattern, same form, ragged rows
    lib.sbn_convert_packed.restype = ctypes.c_int
    conv = lambda **kw: lib.sbn_convert_packed(  # noqa: E731
        vp(kw.get("src", A)), i64(64), i64(kw.get("d_in", 256)), ci(kw.get("N", 6)), ci(kw.get("M", 8)),
        ci(kw.get("to_N", 8)), ci(kw.get("to_M", 8)), vp(kw.get("out", A)), vp(0))
    assert conv(src=0) == sbn.SBN_EINVAL
    assert conv(out=A + 4) == sbn.SBN_EALIGN
    assert conv(to_N=2, to_M=4) == sbn.SBN_EUNSUPPORTED          # 6:8 keeps more than two of an aligned four
    assert conv(N=2, M=4, to_N=2, to_M=4) == sbn.SBN_EUNSUPPORTED  # already in that form
    assert conv(to_N=1, to_M=4) == sbn.SBN_EUNSUPPORTED          # only 2:4 and N = M are decode forms
    assert conv(d_in=200) == sbn.SBN_EUNSUPPORTED                # whole 128-weight chunks only
    assert conv(to_N=9, to_M=8) == sbn.SBN_EINVAL
    # kernels by name: no such kernel, null rows, misaligned outputs, and what a kernel does not take
    lib.sbn_test_linear_kernel.restype = ctypes.c_int

    def kernel(which=0, xq=A, Y=A, tokens=8, d_in=256, d_out=64, N=2, M=4, bias=0):
        return lib.sbn_test_linear_kernel(ci(which), ci(1), one_p(xq), one_p(A), one_i(tokens), one_i(d_in), one_i(d_out), ci(N), ci(M),
                                          one_p(A), one_p(A), one_p(bias), one_p(Y), None, vp(0))
    assert kernel(which=3) == sbn.SBN_EINVAL
    assert kernel(xq=0) == sbn.SBN_EINVAL
    assert kernel(Y=A + 4) == sbn.SBN_EALIGN
    assert kernel(d_in=200) == sbn.SBN_EUNSUPPORTED
    assert kernel(N=6, M=8) == sbn.SBN_EUNSUPPORTED
    assert kernel(which=2, d_in=1 << 25) == sbn.SBN_EUNSUPPORTED
    for refused in ({"tokens": 65}, {"d_out": 66}, {"bias": A}):
        assert kernel(which=1, **refused) == sbn.SBN_EUNSUPPORTED
    # ceiling probes (their own library): unknown kind, missing host output, buffer too small to stream
    from paper_2603_05168_amd import probe
    plib = ctypes.CDLL(probe.lib_path())
    plib.sbn_ceiling_probe.restype = ctypes.c_int
    work = ctypes.c_double(0.0)
    assert plib.sbn_ceiling_probe(ci(7), vp(A), sz(1 << 22), ci(1), ctypes.byref(work), vp(0)) == -1
    assert plib.sbn_ceiling_probe(ci(0), vp(A), sz(1 << 22), ci(1), vp(0), vp(0)) == -1
    assert plib.sbn_ceiling_probe(ci(0), vp(A), sz(1 << 22), ci(0), ctypes.byref(work), vp(0)) == -1
    assert plib.sbn_ceiling_probe(ci(3), vp(A), sz(4096), ci(1), ctypes.byref(work), vp(0)) == -1
    assert plib.sbn_ceiling_probe(ci(3), vp(A + 16), sz(1 << 22), ci(1), ctypes.byref(work), vp(0)) == -4
    assert sbn.sbn_last_error() == ""


def test_backward_refuses_rows_it_cannot_address(sbn):
    """On either side of each limit; a workspace of no bytes tells what was taken from what was refused before any launch."""
    lib = ctypes.CDLL(sbn.lib_path())
    lib.sbn_sparse_ternary_linear_backward.restype = lib.sbn_sparse_ternary_linear_backward_grouped.restype = ctypes.c_int
    vp, i64, ci, sz = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int, ctypes.c_size_t
    A = 0x10000

    def both(tokens, d_in, d_out, dX, dW):
        one = lib.sbn_sparse_ternary_linear_backward(vp(A), i64(tokens), i64(d_in), i64(d_out), ci(2), ci(4), vp(A), vp(A), vp(A), vp(A),
                                                     vp(dX), vp(dW), ci(0), vp(A), sz(0), vp(0))
        P, I = (lambda v: (vp * 1)(v or None)), (lambda v: (i64 * 1)(v))   # noqa: E731
        many = lib.sbn_sparse_ternary_linear_backward_grouped(ci(1), P(A), I(tokens), I(d_in), I(d_out), ci(2), ci(4), P(A), P(A), P(A), P(A),
                                                              P(dX), P(dW), ci(0), vp(A), sz(0), vp(0))
        assert one == many
        return one

    end = 1 << 32
    # dW: seven rows of transposed activations, 2 bytes per token padded to 64, and a stage; 63 rows of gradients and a tile's columns
    most = (end - 129) // 7 // 128 * 64
    for d_in in (8, 2560):
        assert both(most, d_in, 8, 0, A) == sbn.SBN_ESIZE and both(most + 1, d_in, 8, 0, A) == sbn.SBN_EUNSUPPORTED
        assert both(most + 1, d_in, 8, A, 0) == sbn.SBN_ESIZE
    most = (end - 513) // 63 // 2 // 8 * 8
    assert both(64, 8, most, 0, A) == sbn.SBN_ESIZE and both(64, 8, most + 8, 0, A) == sbn.SBN_EUNSUPPORTED
    # dX: eight rows of transposed weights, a byte per output padded to 128
    most = (end - 1) // 8 // 128 * 128
    for tokens in (1, 4096):
        assert both(tokens, 8, most, A, 0) == sbn.SBN_ESIZE and both(tokens, 8, most + 8, A, 0) == sbn.SBN_EUNSUPPORTED
    # what 256 rows, or as many as there are, behind one offset of 32 bits could be computed with
    for tokens, d_in, d_out, dX, dW in ((1 << 23, 2560, 3840, A, A), (8421000, 2560, 8, A, A), (256, 8, 8421000, A, A), (64, 8, 34087000, 0, A),
                                        (306783000, 8, 8, 0, A), (8, 8, 306783000, A, 0)):
        assert both(tokens, d_in, d_out, dX, dW) == sbn.SBN_ESIZE


def test_self_kernel_hook_refuses_on_the_host(sbn):
    lib = ctypes.CDLL(sbn.lib_path())
    lib.sbn_test_self_kernel.restype = ctypes.c_int
    ci, A = ctypes.c_int, 0x10000

    def one(v, t=ctypes.c_void_p):
        return (t * 9)(*[v] * 9)

    def call(form=0, count=1, X=A, Y=A, tokens=8, d_in=256, d_out=64, N=2, M=4):
        return lib.sbn_test_self_kernel(ci(form), ci(count), one(X), one(tokens, ctypes.c_int64), one(d_in, ctypes.c_int64), one(d_out, ctypes.c_int64),
                                        ci(N), ci(M), one(A), one(A), None, one(Y), None, ctypes.c_void_p(0))
    assert call(form=8) == sbn.SBN_EINVAL and call(form=-1) == sbn.SBN_EINVAL
    assert call(X=0) == sbn.SBN_EINVAL
    assert call(X=A + 8) == sbn.SBN_EALIGN and call(Y=A + 4) == sbn.SBN_EALIGN
    for refused in ({"count": 9}, {"d_in": 8200}, {"d_in": 12}, {"tokens": 4097}, {"N": 6, "M": 8}):
        assert call(**refused) == sbn.SBN_EUNSUPPORTED, refused


@pytest.mark.parametrize("N,M", [(2, 4), (8, 8)])
def test_choice_of_block_tiles(sbn, N, M):
    # sizes at which the kernels measure far apart (on 256 multiprocessors, which the library assumes without a GPU)
    for problem in ((640, 2560, 2560), (256, 2560, 6912), (512, 4096, 4096)):
        assert sbn.sbn_test_takes_blocks([problem], N, M), problem
    # more than two rounds of the device, or few tokens through a long layer
    for problem in ((2048, 2560, 6912), (777, 2560, 6912), (1400, 4096, 4096), (96, 8192, 2560), (16384, 768, 6912)):
        assert not sbn.sbn_test_takes_blocks([problem], N, M), problem
    assert not sbn.sbn_test_takes_blocks([(64, 2560, 256)] * 9, N, M)      # more problems than a launch holds


def test_kernels_of_forward_calls(sbn):
    # what a call launches, quantizer included; sizes at which the kernels measure apart.  The first rows are those of
    # test_public_call_equals_its_two_steps (1000 values run as 1024), whose two calls have to take two routes
    self_, decode, blocks, tiles, pieces = sbn.SBN_KERNEL_SELF, sbn.SBN_KERNEL_DECODE, sbn.SBN_KERNEL_BLOCKS, sbn.SBN_KERNEL_TILES, sbn.SBN_KERNEL_PIECES

    def kind(problems, N, M, **how):
        kernels = set(sbn.sbn_test_forward_kernels(problems, N, M, **how))
        assert len(kernels) == 1
        k = kernels.pop()
        return self_ if k >= self_ else blocks if k >= blocks else k

    for N, M in ((2, 4), (8, 8)):
        for problem in ((4, 512, 16388), (6, 1024, 300), (16, 2560, 130), (17, 2560, 130), (50, 1024, 1500), (128, 768, 257)):
            assert kind([problem], N, M) == self_, problem
            assert kind([problem], N, M, rows=False) != self_, problem
        assert kind([(40, 2560, o) for o in (130, 514, 64)], N, M) == self_
        assert kind([(64, 2560, 2560)] * 3, N, M) == self_ and kind([(64, 2560, 6912)] * 2, N, M) == self_
        assert kind([(1, 2560, 2560)], N, M) == decode and kind([(4, 2560, 2560)] * 3, N, M) == decode and kind([(4, 6912, 2560)], N, M) == decode
        assert kind([(8, 2560, 2560)] * 9, N, M) == decode            # more problems than a launch of the self kernel holds
        for problem in ((640, 2560, 2560), (256, 2560, 6912), (512, 4096, 4096)):
            assert kind([problem], N, M) == kind([problem], N, M, rows=False) == blocks, problem
        assert kind([(777, 2560, 6912)], N, M) == kind([(3000, 2560, 2560)], N, M) == pieces
        assert kind([(2181, 512, 475)], N, M) == kind([(4000, 512, 2559)], N, M) == tiles
    assert kind([(64, 8192, 512)], 2, 4) == self_ and kind([(64, 8192, 512)], 8, 8) == tiles
    # single-launch calls are refused where the rows are too long or too many
    assert kind([(64, 8320, 512)], 2, 4) != self_ and kind([(513, 512, 512)], 2, 4) != self_
    for refused in ([(4, 256, 64), (40, 256, 64)], [(4, 200, 64)]):
        with pytest.raises(sbn.SbnError):
            sbn.sbn_test_forward_kernels(refused, 2, 4)


@pytest.mark.parametrize("N,M", [(2, 4), (8, 8)])
@pytest.mark.parametrize("tokens,d_in,d_out", [(17, 2560, 1280), (64, 2560, 1280), (128, 512, 256), (8, 2560, 1280)])
def test_outputs_over_the_rows_are_no_single_launch(sbn, tokens, d_in, d_out, N, M):
    # its blocks write outputs while others still read the rows
    X, rows, out = 1 << 44, 2 * tokens * d_in, 4 * tokens * d_out

    def takes_self(problems, X, Y):
        return sbn.sbn_test_forward_kernels(problems, N, M, X=X, Y=Y)[0] >= sbn.SBN_KERNEL_SELF

    one = [(tokens, d_in, d_out)]
    for Y in (X, X + 16, X + rows - 16, X - out + 16):
        assert not takes_self(one, [X], [Y])
    for Y in (X + rows, X - out):
        assert takes_self(one, [X], [Y])
    far = 1 << 45
    assert takes_self(one * 2, [X, X], [far, far + out])
    assert not takes_self(one * 2, [X, X], [far, X]) and not takes_self(one * 2, [X, X + rows], [X + rows, far])


@pytest.mark.parametrize("N,M", [(2, 4), (8, 8)])
def test_kernels_of_decode_calls(sbn, N, M):
    # tokens, d_in, d_out, problems, whether one launch with the quantizer inside was the faster one where both were measured
    calls = [(3, 2560, 9000, 1, True), (4, 2560, 6912, 2, True), (4, 512, 8192, 1, True), (3, 1536, 9883, 1, True), (5, 2048, 5504, 2, True),
             (3, 1024, 8192, 1, False), (4, 1024, 8192, 1, False), (4, 1024, 4096, 2, False), (3, 1280, 5840, 2, False), (3, 384, 15808, 4, False),
             (5, 1024, 4096, 2, False), (3, 1152, 18754, 2, False), (2, 2560, 9000, 1, False), (4, 2560, 2560, 3, False), (3, 4096, 12208, 1, False),
             (6, 4096, 4096, 1, False), (6, 2560, 2560, 1, True), (6, 512, 492, 2, False), (7, 512, 900, 4, False), (7, 512, 2360, 4, True),
             (6, 1024, 1024, 1, True), (8, 768, 4376, 3, True), (8, 4096, 1000, 2, True), (8, 512, 300, 2, False), (9, 512, 300, 2, True), (16, 8192, 300, 1, True),
             # strips of 128 rows that leave no shape with four rounds at most
             (16, 8192, 8193, 7, True), (16, 8192, 8192, 8, False), (16, 8192, 8065, 8, True)]
    for tokens, d_in, d_out, count, one in calls:
        kernel = sbn.sbn_test_forward_kernels([(tokens, d_in, d_out)] * count, N, M, X=[1 << 44] * count)[0]
        assert (kernel >= sbn.SBN_KERNEL_SELF) == one, (tokens, d_in, d_out, count)
    many = [(16, 8192, 8193)] * 7 + [(16, 8192, 8184)]
    assert set(sbn.sbn_test_forward_kernels(many, N, M)) == {sbn.SBN_KERNEL_DECODE}
