"""The row and column kernels of the fp64 key switch at the edges of their ranges, bit for bit against the oracle: more source
limbs than the conversion's LDS holds at once, eight digits (running sums normalised on the way), one source limb, a
ragged last digit, batches on both sides of the line between stored and register-held accumulators."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# (log_n, q_bits, dnum, special_bits, limbs of the ciphertexts, batch)
POINTS = [
    (14, [50] * 21, 1, 50, 21, 1),                     # 21 sources in chunks of 20, 21 targets
    (15, [50] * 22, 1, 50, 22, 1),
    (12, [50, 40, 45, 50, 36, 50, 44, 50], 8, 50, 8, 3),
    (12, [50, 49, 48, 47, 46, 45, 44], 6, 50, 6, 80),  # digits of two limbs and an empty one, register-held accumulators
    (13, [50, 45, 45, 45, 45, 45, 45], 4, 49, 5, 5),   # ragged last digit below the top level
    (13, [50, 50], 1, 50, 2, 33),
    (15, [50, 50, 50, 50], 4, 50, 3, 9),
    (13, [50] * 9, 1, 50, 9, 2),                       # conversion sums of eight terms and one more
    (12, [50] * 16, 1, 50, 16, 1),                     # twice eight
    (12, [50, 45, 44, 50, 40, 49], 3, 50, 6, 8),       # rows by four waves: 256 inner products of three digits, then more
    (12, [50, 45, 44, 50, 40, 49], 3, 50, 6, 9),
    (12, [50, 45, 44, 50], 1, 50, 4, 32),              # 512 of one digit in both launches, then more
    (12, [50, 45, 44, 50], 1, 50, 4, 33),
    (15, [50, 45, 44, 50], 4, 50, 4, 1),               # four digits: sixteen waves
    (12, [50, 45, 44], 1, 50, 3, 5),                   # a workgroup a polynomial: 120 inner products of one digit, then more than 128
    (12, [50, 45, 44], 1, 50, 3, 6),
    (12, [50, 45, 44, 50, 40, 49], 3, 50, 6, 4),       # 128 of three digits, then more
    (12, [50, 45, 44, 50, 40, 49], 3, 50, 6, 5),
    (12, [50, 45, 44, 50], 4, 50, 4, 6),               # four digits: no waves to spare
    (12, [50] * 16, 1, 50, 2, 15),                     # behind columns of the division
]


@pytest.mark.parametrize("log_n,q_bits,dnum,special,l,batch", POINTS)
def test_key_switch_and_rescale(log_n, q_bits, dnum, special, l, batch):
    from oracle import Oracle
    from paper_1810_00845_amd import hisa, synth
    print("[case]", log_n, len(q_bits), dnum, l, batch, flush=True)
    g, o = hisa.Context(log_n, q_bits, dnum, special, 5), Oracle(log_n, q_bits, dnum, special, 5)
    g.keygen(); o.keygen()
    steps = [3, g.slots - 1]
    g.gen_rot_keys(steps); o.gen_rot_keys(steps)
    coeff = synth.uniform_residues(log_n + l + batch, (batch, 2, l, g.N), g.primes[:l])
    coeff[0, :, :, :3] = 0
    for i in range(l):
        coeff[0, :, i, 3:6] = g.primes[i] - 1
    cts = g.ct_import_batch(coeff, 2.0 ** 50)
    sample = sorted({0, batch - 1})
    ref = {i: o.import_ct(coeff[i], 2.0 ** 50) for i in sample}
    out = g.rot_left_batch(cts, 3)
    hoisted = g.rot_left_hoisted_batch(cts, steps)
    prod = g.mul_no_relin_batch(cts, cts)
    g.relinearize_batch(prod)
    g.rescale_batch(prod)
    summed = g.rot_left_sum_batch([cts, cts], steps)
    for i in sample:
        want = o.export(o.rot_left(ref[i], 3))
        assert np.array_equal(g.ct_export(out[i]), want)
        assert np.array_equal(g.ct_export(hoisted[0][i]), want)
        assert np.array_equal(g.ct_export(hoisted[1][i]), o.export(o.rot_left(ref[i], steps[1])))
        assert np.array_equal(g.ct_export(prod[i]), o.export(o.rescale(o.mul(ref[i], ref[i]))))
    from oracle.layers import SharedModDown
    want = SharedModDown(o, [ref[0]]).total([(0, r, 1, None) for r in steps], ref[0].scale)
    assert np.array_equal(g.ct_export(summed[0]), o.export(want))
    g.close()


@pytest.mark.parametrize("log_n,sources,chunks", [(13, 21, False), (14, 20, False), (14, 21, True), (15, 20, False), (15, 21, True)])
def test_columns_of_more_sources_than_the_lds_holds(log_n, sources, chunks):
    """20 sources at N = 2^14 and 2^15 (40 at 2^13) are in LDS together; more come in chunks, in a kernel of their own."""
    from oracle import Oracle
    from paper_1810_00845_amd import hisa, synth
    print("[case]", log_n, sources, flush=True)
    g, o = hisa.Context(log_n, [50] * sources, 1, 50, 5), Oracle(log_n, [50] * sources, 1, 50, 5)
    g.gen_rot_keys([3]); o.gen_rot_keys([3])
    coeff = synth.uniform_residues(log_n + sources, (1, 2, sources, g.N), g.primes[:sources])
    ct = g.ct_import(coeff[0], 2.0 ** 50)
    g.profile_enable(True)
    out = g.rot_left(ct, 3)
    names = set(g.profile_read())
    g.profile_enable(False)
    form = "ntt_fp_chunks_kernel<%d, %%d>" if chunks else "ntt_fp_kernel<%d, %%d, true>"
    columns = {n for n in names if n.endswith("true>") or "chunks" in n}
    assert columns == {form % (log_n - 10) % mode for mode in (3, 6)}, names
    assert np.array_equal(g.ct_export(out), o.export(o.rot_left(o.import_ct(coeff[0], 2.0 ** 50), 3)))
    g.close()


def test_more_entries_than_a_grid_has_rows():
    """The ModDown's columns of 32769 ciphertexts are 65538 entries, three more than one launch takes: the first ciphertexts, those
    on both sides of the line and the last equal single calls."""
    from paper_1810_00845_amd import hisa
    print("[case] 32769 ciphertexts, N = 2^12, 2 limbs", flush=True)
    g = hisa.Context(12, [50, 45], 1, 50, 5)
    g.gen_rot_keys([3])
    two = g.ct_random_batch(2, 2, 2.0 ** 40, 9)
    n = 32769
    out = g.rot_left_batch([two[i % 2] for i in range(n)], 3)
    want = [g.ct_export(g.rot_left(ct, 3)) for ct in two]
    for i in (0, 1, 32766, 32767, 32768):
        assert np.array_equal(g.ct_export(out[i]), want[i % 2])
    g.rescale_batch(out)
    single = [g.rot_left(ct, 3) for ct in two]
    for ct in single:
        g.rescale_batch([ct])
    for i in (0, 1, 32766, 32767, 32768):
        assert np.array_equal(g.ct_export(out[i]), g.ct_export(single[i % 2]))
    g.close()


# (log_n, q_bits, dnum, outputs, rotations): digits known to the kernel (1, 2, 3) and more, rotations in one wave and over four
# (few outputs), primes that let sums run through and 50-bit ones that are reduced after every eight products
SUMS = [
    (12, [50, 50, 50], 3, 5, 32),
    (12, [50, 40, 40], 1, 1, 31),
    (13, [50] * 8, 8, 2, 17),
    (12, [50, 46, 45, 36], 2, 4, 3),
    (14, [50] * 6, 2, 17, 14),
    (14, [50, 40, 40, 49, 49, 48], 3, 18, 13),
    (14, [50, 40, 40, 49], 4, 33, 5),
    (12, [50, 46, 45, 44, 43], 5, 3, 9),            # five digits over four waves
    (13, [50] * 8, 8, 30, 3),                       # eight in one
]


@pytest.mark.parametrize("log_n,q_bits,dnum,outputs,rotations", SUMS)
def test_sums_of_many_rotations(log_n, q_bits, dnum, outputs, rotations):
    from oracle import Oracle
    from oracle.layers import SharedModDown
    from paper_1810_00845_amd import hisa, synth
    print("[case]", log_n, len(q_bits), dnum, outputs, rotations, flush=True)
    g, o = hisa.Context(log_n, q_bits, dnum, 50, 5), Oracle(log_n, q_bits, dnum, 50, 5)
    steps = list(range(1, rotations + 1))
    g.gen_rot_keys(steps); o.gen_rot_keys(steps)
    l, n = len(q_bits), outputs + 2
    coeff = synth.uniform_residues(log_n + l + n, (n, 2, l, g.N), g.primes[:l])
    for i in range(l):
        coeff[0, :, i, :] = g.primes[i] - 1           # the largest residues: every coefficient of these transforms alike
        coeff[1, 0, i, ::2] = g.primes[i] // 2
    cts = g.ct_import_batch(coeff, 2.0 ** 50)
    ref = [o.import_ct(c, 2.0 ** 50) for c in coeff[:3]] + [None] * (n - 3)
    for terms_of, sample in ((lambda s, b: b + (s % 3 if b < outputs - 1 else 0), 0), (lambda s, b: b, min(2, outputs - 1))):
        out = g.rot_left_sum_batch([[cts[terms_of(s, b)] for b in range(outputs)] for s in [0] + steps], [0] + steps)
        want = SharedModDown(o, ref[:3]).total([(terms_of(s, sample), s, 1, None) for s in [0] + steps], 2.0 ** 50)
        assert np.array_equal(g.ct_export(out[sample]), o.export(want))
        single = g.rot_left_sum_batch([[cts[terms_of(s, outputs - 1)]] for s in [0] + steps], [0] + steps)
        assert np.array_equal(g.ct_export(out[-1]), g.ct_export(single[0]))
    g.close()


# keys beyond the last-level cache, read once (STREAMED_KEY_BYTES, 208 MB a call) and just below it, by one ciphertext and by two
@pytest.mark.parametrize("log_n,q_bits,dnum,rotations,batch",
                         [(14, [50] * 8, 8, 12, 1), (14, [50] * 8, 8, 11, 1), (15, [50, 45, 45, 45, 45, 45], 3, 18, 1), (14, [50] * 8, 8, 12, 2)])
def test_rotations_with_keys_beyond_the_caches(log_n, q_bits, dnum, rotations, batch):
    from paper_1810_00845_amd import hisa
    print("[case]", log_n, len(q_bits), dnum, rotations, batch, flush=True)
    g = hisa.Context(log_n, q_bits, dnum, 50, 5)
    steps = list(range(1, rotations + 1))
    g.gen_rot_keys(steps)
    l = len(q_bits)
    cts = g.ct_random_batch(batch, l, 2.0 ** 50, 11)
    hoisted = g.rot_left_hoisted_batch(cts, steps)
    for s, row in zip(steps, hoisted):
        for ct, out in zip(cts, row):
            assert np.array_equal(g.ct_export(out), g.ct_export(g.rot_left(ct, s)))
    # the sum of the rotations, from their sums over a group of outputs that keeps the keys and over one that does not
    many = g.rot_left_sum_batch([[cts[0]] * 5 for _ in steps], steps)
    one = g.rot_left_sum_batch([[cts[0]] for _ in steps], steps)
    assert np.array_equal(g.ct_export(one[0]), g.ct_export(many[4]))
    g.close()
