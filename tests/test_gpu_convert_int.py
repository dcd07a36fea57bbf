"""The row and column kernels of the 64-bit integer key switch and rescale at the edges of their ranges, bit for bit against
the oracle: every ring degree, digits with more limbs than one chunk of conversion inputs, more digits than one chunk of the
inner product (and than the fp64 path takes), ragged last digits, one limb, mixed prime sizes up to 60 bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# (log_n, q_bits, dnum, special_bits, limbs of the ciphertexts, batch)
POINTS = [
    (10, [60, 30, 25], 3, 60, 3, 3),
    (10, [60] * 10, 1, 60, 10, 1),               # ten sources, no levels on the columns
    (11, [60, 59, 58, 57, 56], 2, 60, 4, 9),     # ragged last digit below the top level
    (12, [60] * 9, 9, 60, 9, 2),                 # nine digits of one limb
    (12, [30, 30, 30], 3, 60, 2, 5),
    (12, [50, 40, 45, 50, 36, 50, 44, 50, 41, 40], 10, 50, 10, 2),   # more digits than the fp64 path takes
    (13, [58] * 21, 2, 60, 19, 1),               # chunks of conversion inputs, three rounds of targets
    (14, [55, 51, 51, 51, 51], 4, 60, 5, 4),
    (15, [60, 51], 1, 60, 2, 3),
    (15, [58] * 8, 1, 60, 8, 1),
    (16, [60] * 6, 1, 60, 6, 1),                 # more sources than fit the LDS at once
    (16, [52, 51, 30], 3, 60, 3, 2),
    (10, [60, 59, 58], 3, 60, 3, 70),            # inner products: few limbs shared out over eight XCDs, one row
    (11, [60, 59, 58, 57], 2, 60, 4, 42),        # rows by four waves: 504 inner products of two digits, then more than 512
    (11, [60, 59, 58, 57], 2, 60, 4, 43),
    (12, [60, 45, 30], 3, 60, 3, 16),            # 256 of three digits, then more
    (12, [60, 45, 30], 3, 60, 3, 17),
    (14, [55, 51, 60, 30], 4, 60, 4, 3),         # four digits: sixteen waves
    (10, [60, 59, 58, 57], 2, 60, 4, 21),        # a workgroup a polynomial: 126 inner products of two digits, then more than 128
    (10, [60, 59, 58, 57], 2, 60, 4, 22),
    (12, [60, 45, 30], 1, 60, 3, 1),
    (10, [55, 51, 60, 30], 4, 60, 4, 25),        # four digits: no waves to spare
    (15, [58] * 8, 3, 60, 8, 10),                # columns: 960 workgroups of five waves, then 1056 of three
    (15, [58] * 8, 3, 60, 8, 11),
    (16, [55, 52, 51, 30], 2, 60, 4, 8),         # 512 workgroups and more
    (13, [58] * 5, 5, 60, 5, 24),                # one source, one digit more than targets of a round
    (15, [58] * 8, 3, 60, 8, 17),                # more than 8192 rows of a division
]


@pytest.mark.parametrize("log_n,q_bits,dnum,special,l,batch", POINTS)
def test_key_switch_and_rescale(log_n, q_bits, dnum, special, l, batch):
    from oracle import Oracle
    from paper_1810_00845_amd import hisa, synth
    print("[case]", log_n, len(q_bits), dnum, l, batch, flush=True)
    g, o = hisa.Context(log_n, q_bits, dnum, special, 5), Oracle(log_n, q_bits, dnum, special, 5)
    g.keygen(); o.keygen()
    g.gen_rot_keys([3]); o.gen_rot_keys([3])
    coeff = synth.uniform_residues(log_n + l + batch, (batch, 2, l, g.N), g.primes[:l])
    coeff[0, :, :, :3] = 0
    for i in range(l):
        coeff[0, :, i, 3:6] = g.primes[i] - 1
    cts = g.ct_import_batch(coeff, 2.0 ** 50)
    sample = sorted({0, batch - 1})
    ref = {i: o.import_ct(coeff[i], 2.0 ** 50) for i in sample}
    assert np.array_equal(g.ct_export(cts[0]), coeff[0])
    out = g.rot_left_batch(cts, 3)
    prod = g.mul_no_relin_batch(cts, cts)
    g.relinearize_batch(prod)
    g.rescale_batch(prod)
    for i in sample:
        assert np.array_equal(g.ct_export(out[i]), o.export(o.rot_left(ref[i], 3)))
        assert np.array_equal(g.ct_export(prod[i]), o.export(o.rescale(o.mul(ref[i], ref[i]))))
    g.close()


def test_tables_of_every_level_made_once_and_found_again():
    """Rotation, relinearisation and rescale at every level, downwards and again upwards: the first call at a level makes its
    tables, the later ones find them."""
    from oracle import Oracle
    from paper_1810_00845_amd import hisa, synth
    print("[case] levels of N = 2^11, 5 limbs, dnum 2", flush=True)
    args = (11, [60, 59, 58, 57, 56], 2, 60, 5)
    g, o = hisa.Context(*args), Oracle(*args)
    g.keygen(); o.keygen()
    g.gen_rot_keys([3]); o.gen_rot_keys([3])
    for l in (5, 4, 3, 2, 1, 2, 3, 4, 5):
        coeff = synth.uniform_residues(l, (1, 2, l, g.N), g.primes[:l])
        ct, ref = g.ct_import_batch(coeff, 2.0 ** 50)[0], o.import_ct(coeff[0], 2.0 ** 50)
        assert np.array_equal(g.ct_export(g.rot_left(ct, 3)), o.export(o.rot_left(ref, 3)))
        prod, want = g.mul_no_relin(ct, ct), o.mul(ref, ref)
        g.relinearize(prod)
        assert np.array_equal(g.ct_export(prod), o.export(want))
        if l > 1:
            g.rescale(prod)
            assert np.array_equal(g.ct_export(prod), o.export(o.rescale(want)))
    g.close()


@pytest.mark.parametrize("log_n", [10, 11, 13, 15, 16])
def test_inverse_rows_by_four_waves_and_by_one(log_n):
    """32768 rows go by four waves each, one polynomial more by one wave a row: the same values, and back to what they were."""
    import torch
    from oracle import Oracle
    from paper_1810_00845_amd import hisa
    print("[case] inverse rows, N = 2^%d" % log_n, flush=True)
    g, o = hisa.Context(log_n, [60], 1, 60, 5), Oracle(log_n, [60], 1, 60, 5)
    few = 1 << (25 - log_n)
    torch.manual_seed(log_n)
    a = torch.randint(0, g.primes[0], (few + 1, g.N), dtype=torch.int64, device="cuda")
    a[0, :3], a[few, -3:] = 0, g.primes[0] - 1
    many = a.clone()
    g.ntt_raw(many, 0)
    for r in (0, few):
        assert np.array_equal(many[r].cpu().numpy().view(np.uint64), o.ntt(a[r].cpu().numpy().view(np.uint64), 0))
    some = many[:few].clone()
    for t, rows in ((some, "ntt_int_wide_kernel<%d, 0>"), (many, "ntt_int_kernel<%d, 0, false>")):
        g.profile_enable(True)
        g.ntt_raw(t, 0, inverse=True)
        names = set(g.profile_read())
        g.profile_enable(False)
        assert {n for n in names if not n.endswith("true>")} == {rows % (log_n - 10)}, names
    assert torch.equal(some, a[:few]) and torch.equal(many, a)
    g.close()


def test_more_ciphertexts_than_one_set_of_launches_takes():
    """Key switches of 32769 ciphertexts and a rescale of their 65538 polynomials are two sets of launches each (32767
    ciphertexts, 65535 polynomials): the first ciphertexts, those on both sides of the lines and the last equal single calls."""
    from paper_1810_00845_amd import hisa
    print("[case] 32769 ciphertexts, N = 2^10, 2 limbs", flush=True)
    g = hisa.Context(10, [60, 51], 1, 60, 5)
    g.keygen()
    g.gen_rot_keys([3])
    two = g.ct_random_batch(2, 2, 2.0 ** 40, 9)
    n = 32769
    batch = [two[i % 2] for i in range(n)]
    single = [g.rot_left(ct, 3) for ct in two]
    out = g.rot_left_batch(batch, 3)
    for i in (0, 1, 32766, 32767, 32768):
        assert np.array_equal(g.ct_export(out[i]), g.ct_export(single[i % 2]))
    g.rescale_batch(out)
    for ct in single:
        g.rescale(ct)
    for i in (0, 1, 32766, 32767, 32768):
        assert np.array_equal(g.ct_export(out[i]), g.ct_export(single[i % 2]))
    # relinearisation, whose addends have two polynomials and stand three polynomials apart
    want = [g.mul_no_relin(ct, ct) for ct in two]
    prod = g.mul_no_relin_batch(batch, batch)
    g.relinearize_batch(prod)
    for ct in want:
        g.relinearize(ct)
    for i in (0, 1, 32766, 32767, 32768):
        assert np.array_equal(g.ct_export(prod[i]), g.ct_export(want[i % 2]))
    g.close()
