"""GPU parity: libqift's HIP path against the CPU oracle, through the C ABI.

Bit-exact: packed words, act_q, act_sum, act_scale, int32 accumulators and
the fp16 output against the oracle's fp32 epilogue expression; within the
max-abs-rel 1e-3 criterion against the oracle's fp64 epilogue.  Inputs come
from the seeded generators; expected values only from ``oracle``.  The
linears run with the per-token code sums computed in the kernels (the
boundary's call takes none) unless a test passes the quantizer's sums.
"""
import numpy as np
import pytest
import torch

from oracle import hadamard, levels, linear as olin, pack as opack, quant
from paper_2606_02823_amd import synth

from route_probe import ask

pytestmark = pytest.mark.gpu

FMTS = [levels.FMT_W2_MNZ, levels.FMT_W2_POT, levels.FMT_W4_SYM]


@pytest.fixture(scope="module")
def Q():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_02823_amd import qift
    qift.lib()
    return qift


def dev(a):
    a = np.ascontiguousarray(a)
    if a.dtype == np.uint32:
        a = a.view(np.int32)
    return torch.from_numpy(a).cuda()


def host(t):
    return t.cpu().numpy()


def bits16(a):
    return np.ascontiguousarray(a).view(np.uint16)


def pack_dev(Q, L, s_w, fmt):
    if fmt == levels.FMT_W4_SYM:
        return Q.pack_w4(dev(L), dev(s_w))
    return Q.pack_w2(dev(L), dev(s_w), fmt)


def check_act(act, x, b, clip=(1, 1), tokens=None):
    q_ref, sx_ref, sum_ref, _ = quant.act_quant(x if tokens is None else x[tokens], b, clip)
    q, sx, sm = host(act.q), host(act.scale), host(act.sum)
    if tokens is not None:
        q, sx, sm = q[tokens], sx[tokens], sm[tokens]
    assert np.array_equal(q, q_ref)
    assert np.array_equal(sx.view(np.uint32), sx_ref.view(np.uint32))
    assert np.array_equal(sm, sum_ref)
    return q_ref, sx_ref


def check_linear(y, acc, L, q_ref, sx_ref, s_w, rows=None, tokens=None):
    y, acc = host(y), host(acc)
    if rows is not None:
        y, acc, L, s_w = y[:, rows], acc[:, rows], L[rows], s_w[rows]
    if tokens is not None:
        y, acc = y[tokens], acc[tokens]
    acc_ref = olin.int_dot(L, q_ref)
    assert np.array_equal(acc, acc_ref)
    assert np.array_equal(bits16(y), bits16(olin.epilogue_fp32(acc_ref, sx_ref, s_w)))
    assert olin.max_abs_rel(y, olin.epilogue_ref(acc_ref, sx_ref, s_w)) <= olin.TOL_REL


def run_linear(Q, pk, act, M, N, use_sum=False, workspace=None):
    acc = torch.empty((M, N), dtype=torch.int32, device="cuda")
    y = Q.linear(pk, act, acc_out=acc, use_sum=use_sum, workspace=workspace)
    torch.cuda.synchronize()
    return y, acc


# ----------------------------------------------------------------------------- config 0


@pytest.mark.parametrize("fmt", FMTS)
def test_cfg0_pipeline(Q, fmt):
    c = synth.CONFIGS[0]
    shp = c.linears[0]
    N, K, b, M = shp.N, shp.K, shp.block, c.Ms[0]
    W = synth.weights_fp32(0, 0, "lin", N, K)
    L, s_w = quant.quantize_weights(hadamard.rotate_weights(W, b), fmt)
    pk = pack_dev(Q, L, s_w, fmt)
    assert np.array_equal(host(pk.words).view(np.uint32), opack.pack(L, fmt))
    x = synth.config_activations(c, 0, 0, M, K)
    act = Q.rotate_quant_act(dev(x), b)
    q_ref, sx_ref = check_act(act, x, b)
    y, acc = run_linear(Q, pk, act, M, N)
    check_linear(y, acc, L, q_ref, sx_ref, s_w)
    # the plain entry (no accumulator output) gives the same y
    y2 = Q.linear(pk, act)
    torch.cuda.synchronize()
    assert torch.equal(y2, y)


# ----------------------------------------------------------------------------- ragged tiles


@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("M", [1, 5, 16, 17, 32, 47, 64, 65, 130])
def test_linear_ragged(Q, fmt, M):
    # N not a multiple of 16, K spanning a partial 1024-chunk, every token-tile count
    N, K, b = 1000, 1088, 64
    L = synth.draw_levels(fmt, N, K, cfg=90, layer=M)
    s_w = synth.draw_scales(fmt, N, cfg=90, layer=M)
    x = synth.activations_fp16(90, M, 0, M, K, 11, 30.0)
    pk = pack_dev(Q, L, s_w, fmt)
    assert np.array_equal(host(pk.words).view(np.uint32), opack.pack(L, fmt))
    act = Q.rotate_quant_act(dev(x), b)
    q_ref, sx_ref = check_act(act, x, b)
    y, acc = run_linear(Q, pk, act, M, N)
    check_linear(y, acc, L, q_ref, sx_ref, s_w)
    # the quantizer's sums passed in (qift_*_linear_ex) give the same results
    y2, acc2 = run_linear(Q, pk, act, M, N, use_sum=True)
    assert torch.equal(acc2, acc) and torch.equal(y2.view(torch.int16), y.view(torch.int16))
    # and so does the boundary's call without accumulators or sums
    y3 = Q.linear(pk, act)
    torch.cuda.synchronize()
    assert torch.equal(y3.view(torch.int16), y.view(torch.int16))


def check_route(kernel, fmt, M, N, K):
    """The linear without a workspace runs the kernel that a test is about (up to 16 tokens: codes of 16 more bytes a
    token within about 130 KB are in the decode kernel's LDS)."""
    assert ask([(fmt == levels.FMT_W4_SYM, N, K, M, K <= 16384 and M * (K + 16) <= 130 * 1024, 0)])[0][0] == kernel


def split_bytes(S, M, N):
    return -(-(S * M * (-(-N // 4) * 4) * 4) // 256) * 256 + S * M * 4


def gemm_ranges(M, N, K, fmt):
    """K-ranges of the split GEMM: 256-k steps, at least 4 a range (W4 128 and 8), about 512 workgroups."""
    bk, s0 = (128, 8) if fmt == levels.FMT_W4_SYM else (256, 4)
    KT, tiles = -(-K // bk), -(-N // 256) * -(-M // 64)
    S = min(-(-512 // tiles), 512 // tiles, KT // s0)
    return -(-KT // -(-KT // S))


def skinny_ranges(N, K):
    """K-ranges of the skinny split: 4 16-row tiles a workgroup, about 256 workgroups, at most 16 units a range."""
    gx, ut = -(-(-(-N // 16)) // 4), -(-K // 256)
    S = min(max((256 + gx // 2) // gx, -(-ut // 16)), ut)
    return -(-ut // -(-ut // S))


def check_split(Q, M, N, K, b, fmt, cfg, form):
    """The linear with the workspace it asks for and without one: bit-identical to the oracle, with and without the
    quantizer's code sums.  form: the split that the workspace's size shows (None: the size is 0)."""
    L = synth.draw_levels(fmt, N, K, cfg=cfg, layer=M + fmt)
    s_w = synth.draw_scales(fmt, N, cfg=cfg, layer=M + fmt)
    x = synth.activations_fp16(cfg, M, 0, M, K, max(1, K // 100), 30.0)
    pk = pack_dev(Q, L, s_w, fmt)
    act = Q.rotate_quant_act(dev(x), b)
    q_ref, sx_ref = check_act(act, x, b)
    need = Q.workspace_bytes(pk, M)
    S = {None: 0, "gemm": gemm_ranges(M, N, K, fmt), "skinny": skinny_ranges(N, K)}[form]
    assert need == (split_bytes(S, M, N) if form else 0)
    # every row up to 4096, beyond them the first and last and 300 between
    rows = None if N <= 4096 else np.unique(np.concatenate([np.arange(8), np.random.default_rng(N).choice(N, 300),
                                                            np.arange(N - 8, N)]))
    y0, acc0 = run_linear(Q, pk, act, M, N)
    check_linear(y0, acc0, L, q_ref, sx_ref, s_w, rows=rows)
    # a workspace that is not needed is accepted and left alone
    ws = torch.full((need if need else 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    for use_sum in (False, True):
        y, acc = run_linear(Q, pk, act, M, N, use_sum=use_sum, workspace=ws)
        assert torch.equal(acc, acc0) and torch.equal(y.view(torch.int16), y0.view(torch.int16))
    if not need:
        assert bool((ws == 0x5A).all())


@pytest.mark.parametrize("fmt", [levels.FMT_W2_MNZ, levels.FMT_W2_POT])
@pytest.mark.parametrize("M,N,K,form", [(65, 1000, 1088, None), (130, 1000, 1088, None), (300, 1000, 4096, "gemm"),
                                        (200, 1000, 14336, "gemm"), (96, 1000, 4160, "gemm"), (320, 16400, 2048, None)])
def test_w2_prefill_with_and_without_split(Q, fmt, M, N, K, form):
    # W2 (MNZ, PoT) at M > 64, ragged rows and tokens, K with a partial last step; the split GEMM where the 256 x 64
    # tiles are few for the length of K (K = 4160 has 17 steps: ranges of 5, 5, 5 and 2, the last one ending in a
    # partial step), else the unsplit one
    check_split(Q, M, N, K, 64, fmt, 97, form)


@pytest.mark.parametrize("M,N,K,form", [(65, 300, 4160, "gemm"), (200, 300, 4160, "gemm"), (128, 1000, 14336, "gemm"),
                                        (96, 4096, 1088, None), (130, 2064, 8192, "gemm"), (40, 16400, 4160, None),
                                        (64, 16384, 2048, None), (48, 4096, 14336, None), (24, 4096, 14336, "gemm"),
                                        (30, 28672, 4096, None), (33, 4096, 16384, "gemm")])
def test_w4_prefill_split_over_k(Q, M, N, K, form):
    # W4 with a workspace: the GEMM split over K (S >= 3 ranges of at least 8 steps of 128 k; K = 4160 has 33 steps:
    # ranges of 9, 9, 9 and 6, the last step partial; K = 1088 has 9, too few), from 24 tokens on for long linears
    # that the batch kernel leaves
    check_split(Q, M, N, K, 64, levels.FMT_W4_SYM, 95, form)


SKINNY_SHAPES = [(f, *shape) for fmts, shapes in (
    (FMTS, [(17, 300, 1088), (23, 999, 4736), (32, 5000, 2112), (32, 12300, 1088), (31, 12300, 2112), (47, 300, 2112),
            (64, 300, 1088), (40, 5000, 2112), (64, 12300, 1088), (40, 12300, 2112)]),
    ([levels.FMT_W2_MNZ, levels.FMT_W2_POT], [(20, 40968, 4160)]),
    ([levels.FMT_W4_SYM], [(20, 3000, 11008), (27, 2600, 16384)])) for f in fmts for shape in shapes]


@pytest.mark.parametrize("fmt,M,N,K", SKINNY_SHAPES)
def test_skinny_linear(Q, fmt, M, N, K):
    # the skinny kernel unsplit: two and four token tiles, one to four row tiles a workgroup, one to eight 256-k units
    # a slice, rows, tokens and k that end inside a tile
    check_route("skinny", fmt, M, N, K)
    check_split(Q, M, N, K, 64, fmt, 88, None)


@pytest.mark.parametrize("fmt", [levels.FMT_W2_MNZ, levels.FMT_W2_POT])
@pytest.mark.parametrize("M,N,K,form", [(17, 1000, 1088, None), (32, 1000, 14336, "skinny"), (33, 4096, 4096, None),
                                        (64, 1000, 14336, None), (64, 4096, 14336, None), (20, 2064, 8192, None),
                                        (40, 300, 16384, "skinny"), (64, 6144, 4096, None), (47, 28672, 4096, None),
                                        (16, 1000, 14336, "skinny"), (13, 4096, 14336, "skinny"), (16, 1000, 4096, None),
                                        (32, 28672, 4096, None), (40, 16400, 4160, None),
                                        # one, two and four token tiles; ranges that end inside the last unit
                                        (10, 1000, 16384, "skinny"), (11, 999, 16320, "skinny"), (17, 2048, 11008, "skinny"),
                                        (33, 1001, 14400, "skinny"), (47, 1000, 14336, "skinny"),
                                        (40, 24832, 8192, "gemm"), (33, 22016, 11008, "gemm")])
def test_skinny_split_over_k(Q, fmt, M, N, K, form):
    # up to 64 tokens with a workspace: the skinny split for the longest K with few 16-row tiles (up to 16 tokens
    # where the decode kernel's LDS does not hold the codes), the split GEMM for wide and long linears
    b = 4096 if K % 4096 == 0 else (2048 if K % 2048 == 0 else 64)
    check_split(Q, M, N, K, b, fmt, 98, form)


@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("K", [384, 4096, 6144, 14336])
@pytest.mark.parametrize("N", [1, 3, 273, 277, 279, 4097])
def test_odd_row_counts(Q, fmt, K, N):
    # the last channel of an odd N shares its dword with the end of the scales' array: every kernel's token range,
    # the fused entry (1-4 tokens) and the linear on codes
    b = 128 if K == 384 else 2048
    L = synth.draw_levels(fmt, N, K, cfg=89, layer=N)
    s_w = synth.draw_scales(fmt, N, cfg=89, layer=N)
    pk = pack_dev(Q, L, s_w, fmt)
    rows = None if N < 4096 else np.unique(np.concatenate([np.arange(64), np.arange(N - 64, N)]))
    for M in (1, 4, 16, 20, 48, 70):
        x = synth.activations_fp16(89, M, 0, M, K, 5, 30.0)
        act = Q.rotate_quant_act(dev(x), b)
        q_ref, sx_ref = check_act(act, x, b)
        for use_sum in (False, True):
            y, acc = run_linear(Q, pk, act, M, N, use_sum=use_sum)
            check_linear(y, acc, L, q_ref, sx_ref, s_w, rows=rows)
        if M <= 4:
            acc = torch.empty((M, N), dtype=torch.int32, device="cuda")
            y = Q.rotate_quant_linear(pk, dev(x), b, acc_out=acc)
            torch.cuda.synchronize()
            check_linear(y, acc, L, q_ref, sx_ref, s_w, rows=rows)


@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("M,K", [(1, 20480), (7, 20480), (9, 20480), (11, 20480), (16, 32768)])
def test_linear_long_k(Q, fmt, M, K):
    # K beyond the decode-on-codes kernel's limit: the decode kernels with codes staged in LDS (M = 1) or read from
    # memory (7 tokens, W4 to 11), then the batch kernel
    N, b = 300, 4096
    check_route("batch" if M >= (12 if fmt == levels.FMT_W4_SYM else 9) else "decode", fmt, M, N, K)
    L = synth.draw_levels(fmt, N, K, cfg=91, layer=M)
    s_w = synth.draw_scales(fmt, N, cfg=91, layer=M)
    x = synth.activations_fp16(91, M, 0, M, K, K // 100, 30.0)
    pk = pack_dev(Q, L, s_w, fmt)
    act = Q.rotate_quant_act(dev(x), b)
    q_ref, sx_ref = check_act(act, x, b)
    y, acc = run_linear(Q, pk, act, M, N)
    check_linear(y, acc, L, q_ref, sx_ref, s_w)


@pytest.mark.parametrize("fmt", FMTS)
def test_linear_extremes(Q, fmt):
    # all-outer levels against all +-7 activations: the largest |acc| of each format
    N, K, b, M = 48, 14336, 2048, 3
    vals = {levels.FMT_W2_MNZ: (3, -3), levels.FMT_W2_POT: (4, -4), levels.FMT_W4_SYM: (7, -7)}[fmt]
    L = np.empty((N, K), dtype=np.int8)
    L[: N // 2] = vals[0]
    L[N // 2:] = vals[1]
    s_w = np.full(N, 0.5, dtype=np.float16)
    s_w[0] = np.float16(65504.0)          # overflow of the product goes to inf
    s_w[1] = 0                            # a zero scale
    x = np.zeros((M, K), dtype=np.float16)
    x[0, ::b] = 60000.0                   # one spike per block -> every q = +7, y overflows to inf
    x[1] = np.float16(2.0 ** -24)         # smallest subnormals
    x[2] = synth.activations_fp16(94, 0, 0, 1, K, 143, 30.0)[0]
    pk = pack_dev(Q, L, s_w, fmt)
    act = Q.rotate_quant_act(dev(x), b)
    q_ref, sx_ref = check_act(act, x, b)
    y, acc = run_linear(Q, pk, act, M, N)
    check_linear(y, acc, L, q_ref, sx_ref, s_w)


def test_pack_rejects_levels_outside_the_set(Q):
    # the pack calls validate every level and return QIFT_ERR_CODE (status -5)
    L = np.full((16, 64), 1, dtype=np.int8)
    L[3, 7] = 0
    s = np.ones(16, dtype=np.float16)
    for fmt, bad in ((Q.W2_MNZ, 0), (Q.W2_MNZ, 2), (Q.W2_POT, 3), (Q.W2_LUT, 4), (Q.W4_SYM, -8), (Q.W4_SYM, 8)):
        L[3, 7] = bad
        with pytest.raises(Q.QiftError, match="QIFT_ERR_CODE") as e:
            if fmt == Q.W4_SYM:
                Q.pack_w4(dev(L), dev(s))
            else:
                Q.pack_w2(dev(L), dev(s), fmt)
        assert e.value.status == -5
    # a clean call afterwards starts from a zero count
    L[3, 7] = 1
    Q.pack_w2(dev(L), dev(s), Q.W2_MNZ)
    Q.pack_w4(dev(L), dev(s))


# ----------------------------------------------------------------------------- activation quantizer


ACT_CASES = [(64, 2), (128, 4), (256, 8), (512, 16), (256, 32), (1024, 64), (11008, 64), (1024, 128),
             (768, 256), (4096, 512), (2048, 1024), (14336, 2048), (4096, 4096), (12288, 4096),
             (16384, 4096), (20480, 4096), (8192, 8192), (32768, 8192), (24576, 2048)]


@pytest.mark.parametrize("K,b", ACT_CASES)
def test_rotate_quant_act_blocks(Q, K, b):
    M = 4
    x = synth.activations_fp16(91, K // 64, b, M, K, max(1, K // 100), 30.0)
    x[1] = 0                                                # all-zero token
    rng = np.random.default_rng(K + b)
    mags = 10.0 ** rng.uniform(-7.5, 4.8, size=K)           # subnormals .. near fp16 max
    x[2] = (mags * rng.choice([-1, 1], size=K)).astype(np.float16)
    x[2, :2] = [65504.0, -65504.0]
    act = Q.rotate_quant_act(dev(x), b)
    check_act(act, x, b)


@pytest.mark.parametrize("M,K,b", [(1, 14336, 2048), (16, 11008, 64), (256, 14336, 2048), (257, 14336, 2048),
                                   (3, 12288, 4096), (64, 8192, 256)])
def test_rotate_quant_act_tile_parallel(Q, M, K, b):
    # up to 256 tokens of several 4096-tiles the tiles are rotated at once by groups of four waves,
    # one token per workgroup; from 257 tokens on four tiles by two groups, fewer by the persistent kernel: the
    # same codes either way
    x = synth.activations_fp16(93, M, b, M, K, max(1, K // 100), 30.0)
    if M > 2:
        x[1] = 0                                            # all-zero token
    act = Q.rotate_quant_act(dev(x), b)
    check_act(act, x, b)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("M,K,b", [(257, 12352, 64), (257, 16384, 4096), (300, 14336, 256), (259, 12352, 2),
                                   (261, 13312, 1024), (2049, 14336, 2048)])
def test_rotate_quant_act_two_groups(Q, M, K, b, bf16):
    # past 256 tokens a token of four 4096-tiles is rotated by two groups of waves, two tiles each: every
    # compiled block exponent (and others), a last tile of a few elements, full tiles; exact as elsewhere
    x = synth.activations_fp16(95, M, b, M, K, max(1, K // 100), 30.0)
    x[1] = 0                                                # all-zero token
    x[2] = 0
    x[2, K - 1] = 3.0                                       # only the last tile holds anything
    tokens = np.array([0, 1, 2, 3, 255, 256, M - 2, M - 1])
    if bf16:
        x = torch.from_numpy(x).to(torch.bfloat16)
        x[3, K - 64:] *= 2.0 ** 90                          # beyond fp16's range
        act = Q.rotate_quant_act(x.cuda(), b)
        q_ref, sx_ref, sum_ref, _ = quant.act_quant_staged(x[tokens].float().numpy(), b, (1, 1))
    else:
        act = Q.rotate_quant_act(dev(x), b)
        q_ref, sx_ref, sum_ref, _ = quant.act_quant(x[tokens], b, (1, 1))
    assert np.array_equal(host(act.q)[tokens], q_ref)
    assert np.array_equal(host(act.scale)[tokens].view(np.uint32), sx_ref.view(np.uint32))
    assert np.array_equal(host(act.sum)[tokens], sum_ref)


def test_rotate_quant_act_exact_ties(Q):
    u = 2.0 ** -10
    pairs = [(9.5, 4.5), (10.5, 3.5), (7.5, 6.5), (8.5, 5.5), (4.5, 9.5)]
    x = np.zeros((2, 64), dtype=np.float16)
    for i in range(32):
        a, bb = pairs[i % len(pairs)]
        x[0, 2 * i], x[0, 2 * i + 1] = a * u, bb * u
        x[1, 2 * i], x[1, 2 * i + 1] = -bb * u, -a * u
    act = Q.rotate_quant_act(dev(x), 2)
    q_ref, _ = check_act(act, x, 2)
    assert set(np.abs(q_ref[0, 1::2]).tolist()) == {0, 2, 4}


@pytest.mark.parametrize("clip", [(9, 10), (1, 2), (15, 16)])
def test_rotate_quant_act_clip_ratio(Q, clip):
    K, b = 4096, 4096
    x = synth.activations_fp16(92, 0, 0, 8, K, 41, 30.0)
    act = Q.rotate_quant_act(dev(x), b, clip=clip)
    check_act(act, x, b, clip)


def _bf16_any(rng, M, K, b):
    """bf16 activations across the finite bf16 range (no narrowing): rows of N(0, 1) at scales from
    2^-30 to 2^30 (values below 2^-17 and from 2^16 in magnitude among them), extreme values
    (subnormals, the largest finite magnitude), a row far below 2^-24, a row mixing 2^-120 and 2^100,
    and a block holding only two values, whose transform alternates 7 2^-100 and 2.5 2^-100 (a
    rounding tie off the fp16 grid)."""
    x = rng.normal(0, 1, (M, K)) * 2.0 ** rng.uniform(-30, 30, (M, 1))
    x[0] *= 2.0 ** -60
    if M > 1:
        x[1] = rng.normal(0, 1, K)
        x[1, ::2] *= 2.0 ** -120
        x[1, 1::2] *= 2.0 ** 100
    if M > 2:
        x[2] = 0
        x[2, 0], x[2, 1] = 4.75 * 2.0 ** -100, 2.25 * 2.0 ** -100   # block 0: [7, 2.5, 7, 2.5, ...] 2^-100
    ext = [2.0 ** -133, -(2.0 ** -126), 3.3e38, -(2.0 ** 100), 2.0 ** -17, 65280.0, 65536.0, 1e-30]
    for m in range(3, M):
        x[m, rng.choice(K, size=len(ext), replace=False)] = ext
    xb = torch.from_numpy(x).to(torch.bfloat16)
    assert torch.isfinite(xb.float()).all()
    return xb


def check_act_bf16(act, x, b, clip=(1, 1)):
    q_ref, sx_ref, sum_ref, _ = quant.act_quant_staged(x, b, clip)
    assert np.array_equal(host(act.q), q_ref)
    assert np.array_equal(host(act.scale).view(np.uint32), sx_ref.view(np.uint32))
    assert np.array_equal(host(act.sum), sum_ref)
    return q_ref, sx_ref


@pytest.mark.parametrize("M,K,b", [(5, 4096, 4096), (4, 11008, 64), (4, 8192, 128), (4, 32768, 4096),
                                   (4, 14336, 2048), (4, 256, 2)])
def test_rotate_quant_act_bf16(Q, M, K, b):
    """bf16 input (qift_rotate_quant_act_bf16) over the whole finite bf16 range: bit-exact against the
    oracle's staged fp64 reading (exact on the fp16 grid)."""
    rng = np.random.default_rng(M * 7919 + K)
    x = _bf16_any(rng, M, K, b)
    for clip in ((1, 1), (9, 10)):
        act = Q.rotate_quant_act(x.cuda(), b, clip=clip)
        check_act_bf16(act, x.float().numpy(), b, clip)


@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("M,N,K,b", [(1, 4096, 4096, 4096), (3, 1040, 4096, 4096), (4, 528, 14336, 2048),
                                     (2, 640, 11008, 64)])
def test_fused_rotate_quant_linear_bf16(Q, fmt, M, N, K, b):
    """bf16 tokens into the fused entry (QIFT_SPEC_BF16): codes, accumulators and y bit-exact."""
    rng = np.random.default_rng(N + K + fmt)
    x = _bf16_any(rng, M, K, b)
    L = synth.draw_levels(fmt, N, K, cfg=90, layer=fmt, slot=M)
    s_w = synth.draw_scales(fmt, N, cfg=90, layer=fmt, slot=M)
    pk = pack_dev(Q, L, s_w, fmt)
    aq = Q.alloc_act(M, K, torch.device("cuda"))
    acc = torch.empty((M, N), dtype=torch.int32, device="cuda")
    y = Q.rotate_quant_linear(pk, x.cuda(), b, acc_out=acc, act_out=aq)
    torch.cuda.synchronize()
    q_ref, sx_ref = check_act_bf16(aq, x.float().numpy(), b)
    acc_ref = olin.int_dot(L, q_ref)
    assert np.array_equal(host(acc), acc_ref)
    assert np.array_equal(bits16(host(y)), bits16(olin.epilogue_fp32(acc_ref, sx_ref, s_w)))


# ----------------------------------------------------------------------------- full-size configs


def _config_linear(Q, cfg, layer, shp, fmt, M, rows=None, tokens=None):
    L = synth.draw_levels(fmt, shp.N, shp.K, cfg=cfg, layer=layer, slot=synth.LINEAR_ID[shp.name])
    s_w = synth.draw_scales(fmt, shp.N, cfg=cfg, layer=layer, slot=synth.LINEAR_ID[shp.name])
    c = synth.CONFIGS[cfg]
    x = synth.config_activations(c, layer, synth.SITE_OF[shp.name], M, shp.K)
    pk = pack_dev(Q, L, s_w, fmt)
    words = host(pk.words).view(np.uint32)
    if rows is None:
        assert np.array_equal(words, opack.pack(L, fmt))
    else:
        assert np.array_equal(words[rows], opack.pack(L[rows], fmt))
    act = Q.rotate_quant_act(dev(x), shp.block)
    q_ref, sx_ref = check_act(act, x, shp.block, tokens=tokens)
    y, acc = run_linear(Q, pk, act, M, shp.N)
    check_linear(y, acc, L, q_ref, sx_ref, s_w, rows=rows, tokens=tokens)


@pytest.mark.parametrize("name", ["q", "k", "v", "o", "gate", "up", "down"])
def test_cfg1_llama2_layer(Q, name):
    shp = next(s for s in synth.CONFIGS[1].linears if s.name == name)
    _config_linear(Q, 1, 0, shp, levels.FMT_W2_MNZ, 1)


@pytest.mark.parametrize("N", [12288, 22016])
def test_cfg1_row_concatenated(Q, N):
    # q|k|v and gate|up stacked along N, as the decode benchmark launches them
    shp = synth.LinearShape("q" if N == 12288 else "gate", N, 4096, 4096)
    _config_linear(Q, 1, 1, shp, levels.FMT_W2_MNZ, 1)


@pytest.mark.parametrize("M", [1, 4, 16])
@pytest.mark.parametrize("name", ["q", "k", "o", "gate", "down"])
def test_cfg2_llama31_decode(Q, M, name):
    shp = next(s for s in synth.CONFIGS[2].linears if s.name == name)
    _config_linear(Q, 2, 31 if name == "k" else 0, shp, levels.FMT_W2_MNZ, M)


@pytest.mark.parametrize("M", [1, 8, 64])
@pytest.mark.parametrize("name", ["gate", "up", "down"])
def test_cfg3_pot_mlp(Q, M, name):
    shp = next(s for s in synth.CONFIGS[3].linears if s.name == name)
    _config_linear(Q, 3, 0, shp, levels.FMT_W2_POT, M)


@pytest.mark.parametrize("fmt", [levels.FMT_W4_SYM, levels.FMT_W2_MNZ])
@pytest.mark.parametrize("name", ["q", "k", "gate", "down"])
def test_cfg4_prefill_sampled(Q, fmt, name):
    shp = next(s for s in synth.CONFIGS[4].linears if s.name == name)
    layer = 0 if fmt == levels.FMT_W4_SYM else 16
    rng = np.random.default_rng(hash((fmt, name)) & 0xFFFF)
    rows = np.sort(rng.choice(shp.N, size=96, replace=False))
    rows[-1] = shp.N - 1
    tokens = np.sort(rng.choice(2048, size=48, replace=False))
    tokens[-1] = 2047
    _config_linear(Q, 4, layer, shp, fmt, 2048, rows=rows, tokens=tokens)


@pytest.mark.parametrize("fmt", [levels.FMT_W4_SYM, levels.FMT_W2_MNZ])
def test_cfg4_row_concatenated(Q, fmt):
    # gate|up stacked along N (28672 rows), as the prefill benchmark launches it: the widest GEMM grid
    shp = synth.LinearShape("gate", 28672, 4096, 4096)
    layer = 1 if fmt == levels.FMT_W4_SYM else 17
    rng = np.random.default_rng(7 + fmt)
    rows = np.sort(rng.choice(shp.N, size=96, replace=False))
    rows[0], rows[-1] = 0, shp.N - 1
    tokens = np.sort(rng.choice(2048, size=48, replace=False))
    tokens[0], tokens[-1] = 0, 2047
    _config_linear(Q, 4, layer, shp, fmt, 2048, rows=rows, tokens=tokens)


@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("K", [64, 128, 320, 512, 576, 896])
def test_gemm_pipeline_tails(Q, fmt, K):
    # the prefill GEMM (M > 64, no workspace) over every count of k-steps that ends its pipeline
    # differently: W4 steps over 128 k with three stages (1, 1, 3, 4, 5, 7 steps: the unrolled loop
    # body, then one or two more, the last step partial at K = 64, 320, 576), W2 over 256 k with two
    # (1, 1, 2, 2, 3, 4 steps); 300 rows and 200 tokens leave partial tiles both ways
    N, M = 300, 200
    L = synth.draw_levels(fmt, N, K, cfg=96, layer=K)
    s_w = synth.draw_scales(fmt, N, cfg=96, layer=K)
    x = synth.activations_fp16(96, K, 0, M, K, 7, 30.0)
    pk = pack_dev(Q, L, s_w, fmt)
    act = Q.rotate_quant_act(dev(x), 64)
    q_ref, sx_ref = check_act(act, x, 64)
    for use_sum in (False, True):
        y, acc = run_linear(Q, pk, act, M, N, use_sum=use_sum)
        check_linear(y, acc, L, q_ref, sx_ref, s_w)


@pytest.mark.parametrize("fmt", FMTS)
def test_linear_wide_grid_ragged(Q, fmt):
    # a grid wide enough for the 128-token W4 tiles, with ragged rows, tokens and a half k-step
    N, K, b, M = 16400, 1088, 64, 2000
    L = synth.draw_levels(fmt, N, K, cfg=94)
    s_w = synth.draw_scales(fmt, N, cfg=94)
    x = synth.activations_fp16(94, 0, 0, M, K, 11, 30.0)
    pk = pack_dev(Q, L, s_w, fmt)
    act = Q.rotate_quant_act(dev(x), b)
    q_ref, sx_ref = check_act(act, x, b)
    y, acc = run_linear(Q, pk, act, M, N)
    check_linear(y, acc, L, q_ref, sx_ref, s_w)


def test_linear_deterministic(Q):
    N, K, M = 4096, 14336, 16
    L = synth.draw_levels(levels.FMT_W2_MNZ, N, K, cfg=93)
    s_w = synth.draw_scales(levels.FMT_W2_MNZ, N, cfg=93)
    x = synth.activations_fp16(93, 0, 0, M, K, 143, 30.0)
    pk = pack_dev(Q, L, s_w, levels.FMT_W2_MNZ)
    act = Q.rotate_quant_act(dev(x), 2048)
    y1, a1 = run_linear(Q, pk, act, M, N)
    y2, a2 = run_linear(Q, pk, act, M, N)
    assert torch.equal(a1, a2) and torch.equal(y1.view(torch.int16), y2.view(torch.int16))


# ----------------------------------------------------------------------------- decode paths


@pytest.mark.parametrize("M,K,b", [(8, 14336, 2048), (16, 14336, 2048), (16, 4096, 4096), (12, 11008, 64)])
def test_decode_activation_paths(Q, M, K, b):
    # activations staged in LDS (M*K small), above 64 KiB of LDS, or read from global (M*K large)
    N = 784
    fmt = levels.FMT_W2_MNZ
    L = synth.draw_levels(fmt, N, K, cfg=95, layer=M)
    s_w = synth.draw_scales(fmt, N, cfg=95, layer=M)
    x = synth.activations_fp16(95, M, 1, M, K, K // 100, 30.0)
    pk = pack_dev(Q, L, s_w, fmt)
    act = Q.rotate_quant_act(dev(x), b)
    q_ref, sx_ref = check_act(act, x, b)
    y, acc = run_linear(Q, pk, act, M, N)
    check_linear(y, acc, L, q_ref, sx_ref, s_w)


# N covers every tiles-per-workgroup count of the decode kernel (ceil(N/16/256) = 1..6)
FUSED_SHAPES = [(512, 256, 256), (1000, 1088, 64), (4096, 4096, 4096), (2064, 11008, 64),
                (4096, 14336, 2048), (1040, 16384, 4096), (784, 8192, 8), (8208, 4096, 4096),
                (12288, 4096, 4096), (16400, 2048, 2048), (22016, 4096, 4096), (24592, 1024, 1024),
                (1040, 2048, 32), (6144, 4096, 4096), (28672, 4096, 4096)]


@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("N,K,b", FUSED_SHAPES)
@pytest.mark.parametrize("M", [1, 4])
def test_fused_rotate_quant_linear(Q, fmt, N, K, b, M):
    L = synth.draw_levels(fmt, N, K, cfg=96, layer=K + M)
    s_w = synth.draw_scales(fmt, N, cfg=96, layer=K + M)
    x = synth.activations_fp16(96, K + M, 2, M, K, max(1, K // 100), 30.0)
    pk = pack_dev(Q, L, s_w, fmt)
    xd = dev(x)
    act = Q.alloc_act(M, K)
    acc = torch.empty((M, N), dtype=torch.int32, device="cuda")
    y = Q.rotate_quant_linear(pk, xd, b, acc_out=acc, act_out=act)
    torch.cuda.synchronize()
    q_ref, sx_ref = check_act(act, x, b)
    check_linear(y, acc, L, q_ref, sx_ref, s_w)
    # bit-identical to the two-call form
    act2 = Q.rotate_quant_act(xd, b)
    y2, acc2 = run_linear(Q, pk, act2, M, N)
    assert torch.equal(acc, acc2) and torch.equal(y.view(torch.int16), y2.view(torch.int16))


@pytest.mark.parametrize("M", [2, 3])
def test_fused_clip_and_no_act_output(Q, M):
    N, K, b = 1024, 4096, 4096
    fmt = levels.FMT_W2_POT
    L = synth.draw_levels(fmt, N, K, cfg=97, layer=M)
    s_w = synth.draw_scales(fmt, N, cfg=97, layer=M)
    x = synth.activations_fp16(97, M, 0, M, K, 41, 30.0)
    x[M - 1] = 0                                    # a zero token inside the batch
    pk = pack_dev(Q, L, s_w, fmt)
    y = Q.rotate_quant_linear(pk, dev(x), b, clip=(9, 10))
    torch.cuda.synchronize()
    q_ref, sx_ref, _, _ = quant.act_quant(x, b, (9, 10))
    acc_ref = olin.int_dot(L, q_ref)
    assert np.array_equal(bits16(host(y)), bits16(olin.epilogue_fp32(acc_ref, sx_ref, s_w)))


# ----------------------------------------------------------------------------- graph replay


def test_graph_replay_matches_eager(Q):
    # one decode layer slice captured as a hipGraph, replayed several times with eager work
    # and synchronizations in between; every replay must equal the eager result
    K, b = 4096, 4096
    shapes = [(3 * 1024, levels.FMT_W2_MNZ), (2048, levels.FMT_W2_POT), (1024, levels.FMT_W4_SYM)]
    pks = []
    for i, (N, fmt) in enumerate(shapes):
        L = synth.draw_levels(fmt, N, K, cfg=98, layer=i)
        pks.append(pack_dev(Q, L, synth.draw_scales(fmt, N, cfg=98, layer=i), fmt))
    x = dev(synth.activations_fp16(98, 0, 0, 1, K, 41, 30.0))
    xs = dev(synth.activations_fp16(98, 1, 0, 16, K, 41, 30.0))
    acts = Q.alloc_act(16, K)
    outs = [torch.empty((1, N), dtype=torch.float16, device="cuda") for N, _ in shapes]
    outs16 = [torch.empty((16, N), dtype=torch.float16, device="cuda") for N, _ in shapes]

    def step():
        for pk, o in zip(pks, outs):
            Q.rotate_quant_linear(pk, x, b, out=o)
        Q.rotate_quant_act(xs, b, out=acts)
        for pk, o in zip(pks, outs16):
            Q.linear(pk, acts, out=o)

    step()
    torch.cuda.synchronize()
    eager = [o.clone() for o in outs + outs16]
    g = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        step()
    torch.cuda.current_stream().wait_stream(s)
    with torch.cuda.graph(g):
        step()
    for _ in range(4):
        for o in outs + outs16:
            o.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for o, e in zip(outs + outs16, eager):
            assert torch.equal(o.view(torch.int16), e.view(torch.int16))


@pytest.mark.parametrize("nwords", [4, 16_388, 262_156, 10_485_764])
def test_hbm_read_probe_reads_every_word(Q, nwords):
    # the bandwidth probe must touch every 32-bit word once: its per-segment XORs are the host's
    words = np.random.default_rng(nwords).integers(0, 2**32, size=nwords, dtype=np.uint64).astype(np.uint32)
    buf = dev(words)
    parts = torch.full((Q.read_probe_slots(4 * nwords),), -1, dtype=torch.int32, device="cuda")
    Q.hbm_read_probe(buf, parts)
    torch.cuda.synchronize()
    seg = Q.READ_PROBE_SEGMENT // 4
    expect = [np.bitwise_xor.reduce(words[i:i + seg]) for i in range(0, nwords, seg)]
    assert np.array_equal(host(parts).view(np.uint32), np.array(expect, dtype=np.uint32))


@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("M,N,K,tokens", [(65, 264, 64, 64), (128, 256, 128, 64), (97, 520, 576, 64), (129, 1000, 1536, 64),
                                          (200, 999, 1664, 64), (64, 16400, 704, 64), (33, 16385, 1088, 64),
                                          (130, 28672, 640, 96), (192, 28672, 1088, 96), (140, 22016, 704, 96),
                                          (190, 23000, 64, 96), (151, 22001, 320, 96), (161, 28600, 1536, 96),
                                          (200, 22016, 1536, 128), (250, 28672, 640, 128), (380, 16390, 320, 128)])
def test_tiled_gemm(Q, fmt, M, N, K, tokens):
    # The tiled GEMM's edges: K from half a step (128 k) over partial and odd line groups (512 k of W2,
    # 256 k of W4: K = 1536 is three of W2's, K = 320 one and a quarter of W4's); tokens that end inside a
    # 32-token tile; rows that end inside a 256-row tile; outputs at 16-byte, 4-byte and odd offsets (N
    # mod 8); tiles of 64, 96 and 128 tokens.  Run once on warm
    # and once on cold caches, where the loads arrive late.  Bit-identical to the oracle (all rows of the
    # small shapes, 200 of the wide ones) with and without accumulators and code sums.
    check_route("gemm", fmt, M, N, K)
    assert ask([(fmt == levels.FMT_W4_SYM, N, K, M, 0, 0)])[0][3] == tokens
    b = 64
    L = synth.draw_levels(fmt, N, K, cfg=94, layer=M + fmt)
    s_w = synth.draw_scales(fmt, N, cfg=94, layer=M + fmt)
    x = synth.activations_fp16(94, M, 0, M, K, 5, 30.0)
    pk = pack_dev(Q, L, s_w, fmt)
    act = Q.rotate_quant_act(dev(x), b)
    q_ref, sx_ref = check_act(act, x, b)
    rows = None if N <= 1000 else np.unique(np.concatenate([np.arange(8), np.random.default_rng(M).choice(N, 200),
                                                            np.arange(N - 8, N)]))
    cold = torch.empty(512 << 20, dtype=torch.uint8, device="cuda")
    first = None
    for use_sum in (False, True):
        y, acc = run_linear(Q, pk, act, M, N, use_sum=use_sum)
        if first is None:
            first = y
            check_linear(y, acc, L, q_ref, sx_ref, s_w, rows=rows)
        for _ in range(2):
            cold.fill_(1)
            y2 = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
            Q.linear(pk, act, out=y2, use_sum=use_sum)
            torch.cuda.synchronize()
            assert torch.equal(y2.view(torch.int16), first.view(torch.int16))
        assert torch.equal(y.view(torch.int16), first.view(torch.int16))


@pytest.mark.parametrize("K", [1 << 21, (1 << 21) + 64, 3 << 20])
def test_tiled_gemm_w4_without_sums_very_long_k(Q, K):
    # without code sums W4's operands are 16 times the levels up to K = 2^21 and the levels beyond, where 16 times
    # the accumulator of extreme rows would leave int32 (49 x 3 x 2^20 x 16 > 2^31)
    M, N = 65, 20
    rng = np.random.default_rng(K)
    L = rng.integers(-7, 8, (N, K), dtype=np.int8)
    q = rng.integers(-7, 8, (M, K), dtype=np.int8)
    L[0], L[1], q[0], q[64] = 7, -7, 7, -7
    s_w = np.full(N, 2.0 ** -10, dtype=np.float16)
    sx = np.full(M, 2.0 ** -10, dtype=np.float32)
    pk = Q.pack_w4(dev(L), dev(s_w))
    y, acc = run_linear(Q, pk, Q.QAct(dev(q), dev(sx)), M, N)
    ref = np.zeros((M, N), dtype=np.int64)
    for k in range(0, K, 1 << 18):   # 49 x 2^18 < 2^24: exact in fp32
        ref += (q[:, k:k + (1 << 18)].astype(np.float32) @ L[:, k:k + (1 << 18)].T.astype(np.float32)).astype(np.int64)
    assert np.array_equal(host(acc), ref)
    assert np.array_equal(bits16(host(y)), bits16(olin.epilogue_fp32(ref.astype(np.int32), sx, s_w)))


@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("K,b", [(64, 2), (64, 64), (128, 8), (192, 64), (256, 256), (384, 128), (640, 128), (768, 256),
                                 (1024, 32), (1024, 512), (1024, 1024), (1088, 64)])
def test_fused_one_wave_per_token(Q, fmt, K, b):
    # tokens of up to 1024 elements are rotated by one wave each: every block exponent up to 10, K that
    # ends inside a wave's window (and 1088, one past the limit), 1 to 4 tokens, a zero token, fp16 and
    # bf16, the paper's clip ratio; codes, scales, sums, accumulators and y bit-exact
    N = 72
    L = synth.draw_levels(fmt, N, K, cfg=93, layer=K + b)
    s_w = synth.draw_scales(fmt, N, cfg=93, layer=K + b)
    pk = pack_dev(Q, L, s_w, fmt)
    for M in (1, 2, 3, 4):
        x = synth.activations_fp16(93, K + M, 0, M, K, 3, 30.0)
        if M == 3:
            x[1] = 0
        act = Q.alloc_act(M, K)
        acc = torch.empty((M, N), dtype=torch.int32, device="cuda")
        y = Q.rotate_quant_linear(pk, dev(x), b, acc_out=acc, act_out=act)
        torch.cuda.synchronize()
        q_ref, sx_ref = check_act(act, x, b)
        check_linear(y, acc, L, q_ref, sx_ref, s_w)
        y = Q.rotate_quant_linear(pk, dev(x), b, clip=(9, 10), acc_out=acc)
        torch.cuda.synchronize()
        q_ref, sx_ref, _, _ = quant.act_quant(x, b, (9, 10))
        check_linear(y, acc, L, q_ref, sx_ref, s_w)
    xb = _bf16_any(np.random.default_rng(K + b), 4, K, b)
    aq = Q.alloc_act(4, K)
    acc = torch.empty((4, N), dtype=torch.int32, device="cuda")
    Q.rotate_quant_linear(pk, xb.cuda(), b, acc_out=acc, act_out=aq)
    torch.cuda.synchronize()
    q_ref, _ = check_act_bf16(aq, xb.float().numpy(), b)
    assert np.array_equal(host(acc), olin.int_dot(L, q_ref))


W2_FMTS, W4_ONLY = [levels.FMT_W2_MNZ, levels.FMT_W2_POT], [levels.FMT_W4_SYM]
BATCH_SHAPES = [(f, *shape) for fmts, shapes in (
    (FMTS, [(17, 4100, 4096), (16, 4096, 4096), (15, 300, 8256), (33, 520, 4160), (32, 8200, 4096), (33, 999, 4736),
            (64, 4096, 2048), (48, 40, 2112), (64, 12288, 4096), (9, 16400, 4672), (16, 70, 16448), (40, 33, 20480),
            (24, 16385, 2048), (24, 25000, 3136), (64, 24576, 2048), (16, 25000, 4160), (40, 6000, 4096), (47, 9000, 4160),
            (33, 20000, 2112), (50, 5000, 2048)]),
    (W2_FMTS, [(15, 300, 4736), (28, 520, 4160), (9, 6200, 4096), (12, 4160, 4096), (5, 16384, 4160), (20, 16385, 2048), (16, 12300, 4160),
               (40, 25000, 16448)]),
    (W4_ONLY, [(36, 25000, 2112), (64, 25000, 2112), (16, 8200, 14336)])) for f in fmts for shape in shapes]


@pytest.mark.parametrize("fmt,M,N,K", BATCH_SHAPES)
def test_batch_linear(Q, fmt, M, N, K):
    # The batch kernel's edges: one to four 32-row tiles a workgroup (N up to and past 8192, 16384, 24576), loads of
    # 16, 32, 48 and 64 tokens, one and two token tiles (and two workgroups of one where N <= 4096), slices of K that end inside a step
    # or a line group, slices past K (K = 2048 and 2112 over 4 and 8 waves), odd counts of line groups; rows
    # and tokens that end inside a tile.  Warm and cold caches (late loads).  Bit-identical to the oracle,
    # with and without accumulators, code sums and a workspace.
    check_route("batch", fmt, M, N, K)
    b = 64
    L = synth.draw_levels(fmt, N, K, cfg=92, layer=M + fmt)
    s_w = synth.draw_scales(fmt, N, cfg=92, layer=M + fmt)
    x = synth.activations_fp16(92, M, 0, M, K, 7, 30.0)
    pk = pack_dev(Q, L, s_w, fmt)
    act = Q.rotate_quant_act(dev(x), b)
    q_ref, sx_ref = check_act(act, x, b)
    rows = None if N <= 1000 else np.unique(np.concatenate([np.arange(8), np.random.default_rng(N).choice(N, 150),
                                                            np.arange(N - 40, N)]))
    need = Q.workspace_bytes(pk, M)
    cold = torch.empty(512 << 20, dtype=torch.uint8, device="cuda")
    first = None
    for ws in (None, torch.empty(need, dtype=torch.uint8, device="cuda") if need else None):
        for use_sum in (False, True):
            y, acc = run_linear(Q, pk, act, M, N, use_sum=use_sum, workspace=ws)
            if first is None:
                first = y
                check_linear(y, acc, L, q_ref, sx_ref, s_w, rows=rows)
            cold.fill_(1)
            y2 = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
            Q.linear(pk, act, out=y2, use_sum=use_sum, workspace=ws)
            torch.cuda.synchronize()
            assert torch.equal(y.view(torch.int16), first.view(torch.int16))
            assert torch.equal(y2.view(torch.int16), first.view(torch.int16))
