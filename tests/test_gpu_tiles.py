"""Edges of the split-K tile kernel and of the many-token tiles: K split over
more waves than it has 128-column steps, last steps of 32 and 96 columns, ragged
token and row tiles, ranks around the 16- and 64-rank tiles, runs of 17 row
tiles, int4 factors read packed, and LoRA sums on both sides of the 32-bit
range.  Integers bit-exact and y bit-exact in the pinned fp32 order, against
the oracle; the automatic path gives the same bits."""
import numpy as np
import pytest

import dfssm_synth as S
import oracle
from gpu_util import assert_y, dev, dev_weights, forced_switch, host, say, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch = torch_cuda()
    import paper_2606_10932_amd as D
    oracle.build()
    return torch, D, oracle.get()


def _check(env, path, M, K, N, r, ws, q, s, rows=None):
    torch, D, o = env
    d = dev_weights(ws)
    qd, sd = dev(q), dev(s)
    args = (qd, sd, d["w_bits"], d["alpha"], d["A"], d["B"], d["beta"])
    y, acc_s, acc_a, acc_b = D.scaffold_lora_linear(*args, path=path, acc=True)
    y2 = D.scaffold_lora_linear(*args, path=path)
    ya = D.scaffold_lora_linear(*args)
    torch.cuda.synchronize()
    rows = np.arange(M) if rows is None else rows
    ref = o.linear(q[rows], s[rows], **ws)
    assert np.array_equal(host(acc_s)[rows], ref["acc_s"]), "acc_s"
    if r:
        assert np.array_equal(host(acc_a)[rows], ref["acc_a"]), "acc_a"
    assert np.array_equal(host(acc_b)[rows], ref["acc_b"]), "acc_b"
    assert_y(host(y)[rows], ref, what=f"{M}x{K}x{N} r{r}")
    assert torch.equal(y, y2) and torch.equal(y, ya), "y without accumulator outputs, automatic path"


# (M, K, N, r): the split-K kernel at the form that its cost model picks (every
# form by itself below)
MID_SHAPES = [
    (3, 768, 3352, 16), (5, 1536, 768, 16), (9, 4096, 2048, 64), (16, 2048, 8512, 64),
    (17, 32, 40, 3), (20, 96, 33, 1), (31, 224, 100, 17), (47, 1152, 129, 33),
    (64, 2560, 1000, 48), (97, 640, 2050, 64), (150, 4128, 70, 16), (256, 4096, 2048, 64),
    (301, 160, 513, 0), (511, 128, 65, 64), (700, 1536, 768, 16), (40, 288, 90, 72),
]


@pytest.mark.parametrize("M,K,N,r", MID_SHAPES)
def test_split_k_tiles(env, M, K, N, r):
    torch, D, o = env
    say(f"split-K tiles {M}x{K}x{N} r{r}")
    ws = S.weights(K, N, r, key=(61, M, K, N, r))
    q, s = o.quantize_act(S.activations(M, K, key=(61, M, K)))
    _check(env, D.PATH_MFMA_FEW if M <= 512 else D.PATH_MFMA, M, K, N, r, ws, q, s)


def _check_int4(env, path, M, K, N, r, key):
    """int4 factors against the int8 linear on the unpacked values."""
    torch, D, o = env
    g = np.random.default_rng([key, M, K, N, r])
    A4 = g.integers(0, 256, (r, K // 2), dtype=np.uint8)
    B4 = g.integers(0, 256, (N, r // 2), dtype=np.uint8)
    ws = S.weights(K, N, r, key=(key, M, K, N, r))
    ws["A"] = o.unpack_int4(A4, r * K).reshape(r, K)
    ws["B"] = o.unpack_int4(B4, N * r).reshape(N, r)
    q, s = o.quantize_act(S.activations(M, K, key=(key, M, K)))
    ref = o.linear(q, s, **ws)
    d = dev_weights(ws)
    y, acc_s, acc_a, acc_b = D.scaffold_lora_linear_i4(dev(q), dev(s), d["w_bits"], d["alpha"], dev(A4), dev(B4),
                                                       d["beta"], path=path, acc=True)
    torch.cuda.synchronize()
    assert np.array_equal(host(acc_s), ref["acc_s"]) and np.array_equal(host(acc_a), ref["acc_a"])
    assert np.array_equal(host(acc_b), ref["acc_b"])
    assert_y(host(y), ref, what="int4 tiles")


# the forms of the split-K kernel (tokens x rows x waves of a workgroup); M, N
# and K at remainders of each, fewer 128-column steps than waves, ranks of one,
# two and five 16-rank tiles, one and three 64-rank chunks
FORMS = ["64x64x8", "64x64x4", "32x64x8", "32x64x4", "16x64x4", "16x32x8", "16x16x8"]


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("form", range(len(FORMS)), ids=FORMS)
@pytest.mark.parametrize("M,K,N,r", [(5, 32, 20, 2), (37, 160, 78, 18), (129, 1056, 200, 64), (50, 224, 70, 130)])
def test_split_k_forms(env, form, bits, M, K, N, r):
    torch, D, o = env
    say(f"split-K form {FORMS[form]} int{bits} {M}x{K}x{N} r{r}")
    with forced_switch(D, D.TEST_LINEAR_KERNEL, form + 2):
        if bits == 4:
            _check_int4(env, D.PATH_AUTO, M, K, N, r, 65)
        else:
            ws = S.weights(K, N, r, key=(66, M, K, N, r))
            q, s = o.quantize_act(S.activations(M, K, key=(66, M, K)))
            _check(env, D.PATH_AUTO, M, K, N, r, ws, q, s)


@pytest.mark.parametrize("M,K,N,r", [(2500, 64, 40, 0), (7680, 32, 24, 14), (2030, 96, 33, 50)])
def test_split_k_words_of_small_ranks(env, M, K, N, r):
    """More tokens than the words of rank 64 leave room for."""
    torch, D, o = env
    say(f"split-K words {M}x{K}x{N} r{r}")
    ws = S.weights(K, N, r, key=(69, M, K, N, r))
    q, s = o.quantize_act(S.activations(M, K, key=(69, M, K)))
    with forced_switch(D, D.TEST_LINEAR_KERNEL, 5):
        _check(env, D.PATH_MFMA, M, K, N, r, ws, q, s)


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,K,N,r", [(1, 768, 3352, 16), (2, 160, 77, 6), (1, 32, 1, 2), (2, 256, 31, 256),
                                     (2, 4128, 50, 72), (1, 12288, 70, 32), (2, 2048, 1000, 64), (1, 2048, 8512, 64)])
def test_few_token_kernel(env, bits, M, K, N, r):
    """The few-token kernel by itself: one copy of the LoRA words (r <= 32) and
    one per XCD, one and several 64-rank chunks, K below one wave's columns and
    above all waves', sign rows of odd words, packed B rows of 3 bytes."""
    torch, D, o = env
    say(f"few-token kernel int{bits} {M}x{K}x{N} r{r}")
    with forced_switch(D, D.TEST_LINEAR_KERNEL, 1):
        if bits == 4:
            _check_int4(env, D.PATH_AUTO, M, K, N, r, 67)
        else:
            ws = S.weights(K, N, r, key=(68, M, K, N, r))
            q, s = o.quantize_act(S.activations(M, K, key=(68, M, K)))
            _check(env, D.PATH_AUTO, M, K, N, r, ws, q, s)


@pytest.mark.parametrize("form", [4, 8])
@pytest.mark.parametrize("M,K,N,r", [(128, 128, 256, 64), (127, 96, 255, 16), (129, 160, 272, 17), (257, 1056, 273, 64),
                                     (140, 256, 2180, 65), (2048, 96, 8512, 8),
                                     # the down-projection's 32-rank workgroups, some past the rank; 64 again
                                     (40, 96, 130, 17), (200, 160, 70, 97), (2049, 96, 40, 33),
                                     # ranks of three and four 64-rank chunks
                                     (300, 128, 400, 256), (150, 160, 130, 190)])
def test_many_token_tiles(env, form, M, K, N, r):
    torch, D, o = env
    say(f"many-token tiles form={form} {M}x{K}x{N} r{r}")
    ws = S.weights(K, N, r, key=(62, M, K, N, r))
    q, s = o.quantize_act(S.activations(M, K, key=(62, M, K)))
    rows = np.unique(np.r_[0, 15, 16, 127, M // 2, M - 1]) if M > 1000 else None
    with forced_switch(D, D.TEST_PREFILL_KERNEL, form):
        _check(env, D.PATH_MFMA, M, K, N, r, ws, q, s, rows)


@pytest.mark.parametrize("form", [4, 8])
@pytest.mark.parametrize("scale", ["below", "above", "mixed"])
def test_lora_sum_range(env, form, scale):
    """LoRA sums that fit 32 bits, that do not, and both in one launch: the
    whole-tile epilogue takes them by different arithmetic, with one result.
    Codes and factors of one sign reach 127 * 127 * K per acc_a."""
    torch, D, o = env
    M, K, N, r = 256, 4096, 512, 64
    say(f"lora sum range form={form} {scale}")
    ws = S.weights(K, N, r, key=(63,))
    q, s = o.quantize_act(S.activations(M, K, key=(63,)))
    if scale != "below":
        rows = slice(None) if scale == "above" else slice(70, 72)
        q[rows] = 127
        ws["A"][:] = np.abs(ws["A"])
        ws["B"][::3] = 127
    ref = o.linear(q, s, **ws)
    big = np.abs(ref["acc_b"]).max() >= 2 ** 31
    assert big == (scale != "below")
    with forced_switch(D, D.TEST_PREFILL_KERNEL, form):
        _check(env, D.PATH_MFMA, M, K, N, r, ws, q, s)


@pytest.mark.parametrize("path", ["few", "tile4", "tile8"])
@pytest.mark.parametrize("M,K,N,r", [(19, 96, 70, 2), (130, 2048, 300, 64), (200, 4096, 512, 16), (150, 160, 272, 66)])
def test_packed_int4_tiles(env, path, M, K, N, r):
    """int4 factors, which both tile kernels read packed, against the int8
    linear on the unpacked values."""
    torch, D, o = env
    say(f"int4 tiles {path} {M}x{K}x{N} r{r}")
    p = D.PATH_MFMA_FEW if path == "few" else D.PATH_MFMA
    with forced_switch(D, D.TEST_PREFILL_KERNEL, {"tile4": 4, "tile8": 8}.get(path, 0)):
        _check_int4(env, p, M, K, N, r, 64)
