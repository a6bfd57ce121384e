"""Every form of the row-scoring kernel (1, 4, 8 or 16 wavefronts per row, by the row's 16-byte
words and the number of rows) on both sides of its borders, against float64: ragged tails, rows
whose last chunk is partial, -inf entries, a row of only -inf and one with a NaN."""
import math

import pytest

pytestmark = pytest.mark.gpu

# 16-byte words per row at and around the borders, and the chunk counts of the pipelined form
FEW = [1, 63, 65, 255, 256, 257, 1023, 1024, 1025, 2047, 3071, 3072, 3073, 4095, 7937, 8191, 8192, 8193,
       8447, 8448, 9500, 10243, 12365, 14336, 16383, 16384, 18992, 24576]
MANY = [8192, 8703, 16384, 16999, 20480, 24575, 24576]


PAIR_WORDS = [1, 127, 129, 1000, 1023, 1024, 1279, 2500, 5119, 5120, 7000]


def _check_pairs(words, n, dtype, pad):
    import torch
    import paper_2609_14636_amd as P
    per = 8 if dtype is torch.bfloat16 else 4
    vocab = words * per + pad
    ld = vocab + (-vocab) % per
    g = torch.Generator(device="cuda").manual_seed(words + n)
    t, s = (torch.empty((n, ld), dtype=dtype, device="cuda").normal_(0, 3, generator=g) for _ in range(2))
    ids = torch.randint(0, vocab, (n,), dtype=torch.int32, device="cuda", generator=g)
    ids[0] = vocab - 1
    t[:, vocab:] = 900.0
    s[:, vocab:] = 1000.0
    if vocab > 4:
        t[2, 2::3] = s[2, 2::3] = -math.inf     # no mass on either side
        s[3, 2::3] = -math.inf                  # the teacher alone has some
        t[1, 2::3] = -math.inf                  # the student alone: the divergence is infinite
        ids[1:4] = 0
    s[4, vocab // 2] = math.nan
    ids[6] = vocab
    lay = P.Layout(torch.tensor([0, 1], dtype=torch.int32, device="cuda"),
                   torch.tensor([0, n], dtype=torch.int64, device="cuda"), n)
    path = P.Path(lay, P.STRIDE_UNIT_TURN, exact_kl=True)
    path.score(vocab, [t], s, ids)
    assert torch.isnan(path.kl_full[4]) and torch.isnan(path.logp_s[4])
    assert torch.isnan(path.logp_t[6]) and torch.isfinite(path.kl_full[6])
    at = torch.tensor([0, 2, 3] + list(range(8, n, max(1, n // 64))) + [n - 1], device="cuda")
    lt, ls = (x[at][:, :vocab].double().log_softmax(1) for x in (t, s))
    pick = ids[at].long().unsqueeze(1)
    kl = torch.where(ls > -math.inf, ls.exp() * (ls - lt), torch.zeros_like(ls)).sum(1)
    for got, want in ((path.logp_t, lt.gather(1, pick).squeeze(1)), (path.logp_s, ls.gather(1, pick).squeeze(1))):
        assert float((got[at].double() - want).abs().max()) <= 2e-5
    # a sum of p (s - t) of size about 10 and two logarithms, in fp32
    assert float((path.kl_full[at].double() - kl).abs().max()) <= 1e-4
    assert vocab <= 4 or float(path.kl_full[1]) == math.inf


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_pairs(dtype):
    import torch
    for n in (24, 16384 + 3):
        for words in PAIR_WORDS:
            print("words", words, "tokens", n, flush=True)
            _check_pairs(words, n, torch.bfloat16 if dtype == "bf16" else torch.float32, 3)


def _check(words, n, dtype, pad):
    import torch
    import paper_2609_14636_amd as P
    per = 8 if dtype is torch.bfloat16 else 4
    vocab = words * per + pad
    ld = vocab + (-vocab) % per
    g = torch.Generator(device="cuda").manual_seed(words + n)
    x = torch.empty((n, ld), dtype=dtype, device="cuda").normal_(0, 3, generator=g)
    ids = torch.randint(0, vocab, (n,), dtype=torch.int32, device="cuda", generator=g)
    ids[0], ids[1] = vocab - 1, 0
    x[:, vocab:] = 1000.0                       # padding columns are not logits
    if vocab > 4:
        x[2, :vocab - 1] = -math.inf            # only the last entry has mass
        ids[2] = vocab - 1
        x[3, ::3] = -math.inf
        ids[3] = 1
    x[4, :vocab] = -math.inf
    x[5, vocab // 2] = math.nan
    ids[6], ids[7] = vocab, -1
    lay = P.Layout(torch.tensor([0, 1], dtype=torch.int32, device="cuda"),
                   torch.tensor([0, n], dtype=torch.int64, device="cuda"), n)
    path = P.Path(lay, P.STRIDE_UNIT_TURN, with_student=False)
    path.score(vocab, [x], None, ids)
    got = path.logp_t
    assert torch.isnan(got[4:8]).all()
    assert int(path.flags.item()) & (P.STRIDE_FLAG_NONFINITE | P.STRIDE_FLAG_TOKEN_OOB) == \
        P.STRIDE_FLAG_NONFINITE | P.STRIDE_FLAG_TOKEN_OOB
    at = torch.tensor([0, 1, 2, 3] + list(range(8, n, max(1, n // 64))) + [n - 1], device="cuda")
    z = x[at][:, :vocab].double()
    want = z.gather(1, ids[at].long().unsqueeze(1)).squeeze(1) - torch.logsumexp(z, 1)
    # fp32 sums of at most a few hundred terms per lane and their merges, and the rounding of
    # a logarithm and two differences of numbers below 64: a few units of 2^-18
    assert float((got[at].double() - want).abs().max()) <= 2e-5
    # one term, exp2 of the rounding residual of m log2(e): within 5e-7 of its exact value 0
    assert vocab <= 4 or -5e-7 <= float(got[2]) <= 0.0


@pytest.mark.parametrize("pad", [0, 3])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_few_rows(dtype, pad):
    import torch
    for words in FEW:
        print("words", words, flush=True)
        _check(words, 40, torch.bfloat16 if dtype == "bf16" else torch.float32, pad)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_many_rows(dtype):
    import torch
    for words in MANY:
        print("words", words, flush=True)
        _check(words, 16384 + 5, torch.bfloat16 if dtype == "bf16" else torch.float32, 1)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_grad_forms(dtype):
    """The OPD gradient at the borders of its forms: retained rows against float64, the others zero,
    padding columns and rows past the last untouched."""
    import torch
    import paper_2609_14636_amd as P
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    per = 8 if dtype == "bf16" else 4
    for words in (1, 63, 255, 256, 257, 1024, 1535, 1536, 2047, 3071, 3072, 4095, 4097, 9000):
        for pad in (0, 3):
            vocab, n = words * per + pad, 27
            print("words", words, "pad", pad, flush=True)
            ld = vocab + (-vocab) % per
            g = torch.Generator(device="cuda").manual_seed(words)
            s = torch.empty((n, ld), dtype=td, device="cuda").normal_(0, 3, generator=g)
            ids = torch.randint(0, vocab, (n,), dtype=torch.int32, device="cuda", generator=g)
            ids[0], ids[1] = vocab - 1, 0
            lay = P.Layout(torch.tensor([0, 1, 2], dtype=torch.int32, device="cuda"),
                           torch.tensor([0, 11, n], dtype=torch.int64, device="cuda"), n)
            path = P.Path(lay, P.STRIDE_UNIT_TOKEN)
            path.score(vocab, [s], s, ids)
            path.logp_t.add_(torch.linspace(-1, 1, n, device="cuda"))
            path.stop_unit.copy_(torch.tensor([6, -1], dtype=torch.int32))
            start = torch.tensor([2, 5], dtype=torch.int32, device="cuda")
            buf = torch.full((n + 1, ld), 7.0, dtype=td, device="cuda")
            path.grad(vocab, s, ids, buf[:n], None, start, scale=0.5)
            assert int(path.flags.item()) == 0
            keep = torch.zeros(n, dtype=torch.bool, device="cuda")
            keep[2:7] = keep[16:] = True
            c = 0.5 * (path.logp_t - path.logp_s).double().unsqueeze(1)
            want = c * s[:, :vocab].double().softmax(1)
            want[torch.arange(n, device="cuda"), ids.long()] -= c.squeeze(1)
            got = buf[:n, :vocab].double()
            assert (got[~keep] == 0).all() and (buf[n] == 7.0).all() and (buf[:, vocab:] == 7.0).all()
            # one rounding to the logits' type, and fp32's exp2 argument of a logit below 32
            tol = (2.0 ** -8 if dtype == "bf16" else 4e-6) * want[keep].abs() + 4e-6 * c[keep].abs()
            assert ((got[keep] - want[keep]).abs() <= tol).all()


def _masked(words, n, dtype, masked, exact_kl):
    """Rows whose entries [masked) hold the type's lowest value: they carry no mass, so the rest of the
    row gives the log-probability, the divergence and no flag."""
    import torch
    import paper_2609_14636_amd as P
    per = 8 if dtype is torch.bfloat16 else 4
    vocab = words * per
    g = torch.Generator(device="cuda").manual_seed(words)
    t, s = (torch.empty((n, vocab), dtype=dtype, device="cuda").normal_(0, 3, generator=g) for _ in range(2))
    lo, hi = masked
    t[:, lo * per:hi * per] = s[:, lo * per:hi * per] = torch.finfo(dtype).min
    keep = torch.cat([torch.arange(lo * per), torch.arange(hi * per, vocab)]).cuda()
    ids = keep[torch.randint(0, keep.numel(), (n,), device="cuda", generator=g)].int()
    lay = P.Layout(torch.tensor([0, 1], dtype=torch.int32, device="cuda"),
                   torch.tensor([0, n], dtype=torch.int64, device="cuda"), n)
    path = P.Path(lay, P.STRIDE_UNIT_TURN, exact_kl=exact_kl)
    path.score(vocab, [t], s, ids)
    assert int(path.flags.item()) == 0
    at = torch.arange(0, n, max(1, n // 64), device="cuda")
    lt, ls = (x[at][:, keep].double().log_softmax(1) for x in (t, s))
    col = torch.searchsorted(keep, ids[at].long()).unsqueeze(1)
    # the bounds of _check and _check_pairs
    for got, want in ((path.logp_t, lt), (path.logp_s, ls)):
        assert float((got[at].double() - want.gather(1, col).squeeze(1)).abs().max()) <= 2e-5
    if exact_kl:
        want = (ls.exp() * (ls - lt)).sum(1)
        assert float((path.kl_full[at].double() - want).abs().max()) <= 1e-4


# words of the row, rows, masked words: whole loads of a lane, or all that a wavefront reads
MASKED = [(1280, 16384, (1152, 1280)), (256, 16384, (0, 192)), (512, 40, (0, 256)), (8192, 40, (512, 1024)),
          (2048, 40, (1024, 1536)), (16384, 16384, (512, 1024)), (6400, 40, (2048, 4096))]


@pytest.mark.parametrize("exact_kl", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_masks_of_the_lowest_value(dtype, exact_kl):
    import torch
    for words, n, masked in MASKED:
        print("words", words, "rows", n, "masked", masked, flush=True)
        _masked(words, n, torch.bfloat16 if dtype == "bf16" else torch.float32, masked, exact_kl)


# words, rows: both sides of the borders by the number of rows (1,024 or 2,048, 128) and by the words (1,408,
# 12,288)
BORDERS = [(511, 1024), (511, 1025), (512, 1024), (512, 2048), (512, 2049), (1023, 2048), (1023, 2049),
           (1024, 40), (1407, 300), (1408, 300), (3, 1024), (3, 1025),
           (12287, 128), (12288, 128), (12288, 129), (12289, 128), (18992, 9), (24577, 128),
           (65537, 12)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_borders_by_the_number_of_rows(dtype):
    import torch
    for words, n in BORDERS:
        print("words", words, "rows", n, flush=True)
        _check(words, n, torch.bfloat16 if dtype == "bf16" else torch.float32, 3)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_many_rows_on_lines_and_off_them(dtype):
    """16,384 rows and more whose length is a whole number of 128-byte lines, and not."""
    import torch
    for words, pad in ((8447, 1), (8448, 0), (16383, 1), (16384, 0), (16384, 1), (20001, 0), (24575, 1)):
        print("words", words, "pad", pad, flush=True)
        _check(words, 16384 + 5, torch.bfloat16 if dtype == "bf16" else torch.float32, pad)


@pytest.mark.parametrize("pad", [0, 3])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_pipelined_form(dtype, pad):
    """4,096 rows and more: every number of chunks left over when the pipeline's loop ends."""
    import torch
    for words in [w for w in FEW if w >= 8192]:
        print("words", words, flush=True)
        _check(words, 4096 + 5, torch.bfloat16 if dtype == "bf16" else torch.float32, pad)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_pairs_borders(dtype):
    """Both sides of the paired form's borders by the number of tokens (256 or 1,024) and the words."""
    import torch
    for words, n in ((255, 256), (255, 257), (256, 1024), (256, 1025), (1023, 1024), (1023, 1025), (2559, 24),
                     (2560, 24), (3583, 24), (3584, 24), (3584, 16384)):
        print("words", words, "tokens", n, flush=True)
        _check_pairs(words, n, torch.bfloat16 if dtype == "bf16" else torch.float32, 3)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_grad_borders(dtype):
    """Both sides of the gradient's borders by the number of rows (256 or 1,024), and 1,024 words."""
    import torch
    import paper_2609_14636_amd as P
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    per = 8 if dtype == "bf16" else 4
    for words, n in ((63, 256), (63, 257), (64, 1024), (64, 1025), (255, 1024), (255, 1025), (1024, 40), (1025, 40)):
        print("words", words, "rows", n, flush=True)
        vocab = words * per + 3
        g = torch.Generator(device="cuda").manual_seed(words + n)
        s = torch.empty((n, (words + 1) * per), dtype=td, device="cuda").normal_(0, 3, generator=g)
        ids = torch.randint(0, vocab, (n,), dtype=torch.int32, device="cuda", generator=g)
        ids[0] = vocab - 1
        lay = P.Layout(torch.tensor([0, 1], dtype=torch.int32, device="cuda"),
                       torch.tensor([0, n], dtype=torch.int64, device="cuda"), n)
        path = P.Path(lay, P.STRIDE_UNIT_TOKEN)
        path.score(vocab, [s], s, ids)
        path.logp_t.add_(torch.linspace(-1, 1, n, device="cuda"))
        path.stop_unit.fill_(n - 2)
        grad = torch.full_like(s, 7.0)
        path.grad(vocab, s, ids, grad, None, torch.tensor([1], dtype=torch.int32, device="cuda"), scale=0.5)
        assert int(path.flags.item()) == 0
        c = 0.5 * (path.logp_t - path.logp_s).double().unsqueeze(1)
        want = c * s[:, :vocab].double().softmax(1)
        want[torch.arange(n, device="cuda"), ids.long()] -= c.squeeze(1)
        want[0] = want[n - 1] = 0
        got = grad[:, :vocab].double()
        assert (got[0] == 0).all() and (got[n - 1] == 0).all() and (grad[:, vocab:] == 7.0).all()
        # one rounding to the logits' type, and fp32's exp2 argument of a logit below 32
        tol = (2.0 ** -8 if dtype == "bf16" else 4e-6) * want.abs() + 4e-6 * c.abs()
        assert ((got - want).abs() <= tol).all()
