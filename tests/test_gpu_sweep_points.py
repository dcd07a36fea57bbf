"""Parity at the other points of the primitive sweep, in the launch configuration bench.py times there: batches of 64
ciphertexts at N = 2^14 and 2^13 with 16 and 8 limbs, dnum 3 and 1.  The per-kernel timing records say which launches ran,
and they must be exactly those that the host's rules choose: accumulators in registers or, where the rows of a call fill less
than half of the chip, in memory; rows by one wave each or, where a launch has few of them, by four; whole polynomials by
columns and rows or, above 2^22 coefficients, a workgroup each.
Sampled outputs are compared bit for bit with the oracle."""
import re

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# (log_n, limbs, dnum, the largest batch whose accumulators are stored: batch (limbs + K) N / 1024 < 1024)
POINTS = [
    (14, 16, 3, 2),
    (14, 16, 1, 1),
    (13, 16, 1, 3),
    (14, 8, 3, 5),
    (13, 8, 1, 7),
]
# the launches of a rotation, (mode, over columns): inverse rows, ModUp's columns, inner product of the special limbs,
# division's columns, and the inner product of the limbs of q with the difference or the difference alone
IN_REGISTERS = {(2, False), (3, True), (5, False), (6, True), (6, False)}
STORED = {(2, False), (3, True), (5, False), (6, True), (7, False)}


def by_four_waves(launch, g, batch):
    """Whether the rows of a launch over `batch` ciphertexts at the top level go by four waves each: up to 2048 rows, or as
    many inner products as are resident at once (512 of one or two digits, 256 of three or four)."""
    mode, columns = launch
    if columns:
        return False
    rows, l, K, digits = g.N // 1024, g.L, g.K, -(-g.L // g.alpha)
    stored = batch * (l + K) * rows < 1024
    inner = 512 if digits <= 2 else 256 if digits <= 4 else 0
    limbs = {2: l, 5: l + K if stored else K, 6: l, 7: 2 * l}[mode]
    return batch * limbs * rows <= (inner if mode in (5, 6) else 2048)


def launches(g, batch, call):
    """call's result and the launches it made: "ntt_fp_kernel<log2 N - 10, mode, over columns>", or
    "ntt_fp_wide_kernel<log2 N - 10, mode>" where the rows must go by four waves, as (mode, columns)."""
    g.profile_enable(True)
    out = call()
    names = g.profile_read()
    g.profile_enable(False)
    ran = []
    for n, (count, _) in names.items():
        m = re.fullmatch(r"ntt_fp_(wide_)?kernel<(\d+), (\d+)(?:, (true|false))?>", n)
        assert m and int(m.group(2)) == g.log_n - 10 and (m.group(1) is None) == (m.group(4) is not None), names
        launch = int(m.group(3)), m.group(4) == "true"
        assert (m.group(1) is not None) == by_four_waves(launch, g, batch), names
        ran += [launch] * count
    assert len(set(ran)) == len(ran), names
    return out, set(ran)


@pytest.mark.parametrize("log_n,L,dnum,most_stored", POINTS)
def test_rot_left_batch_at_sweep_point(log_n, L, dnum, most_stored):
    from oracle import Oracle
    from paper_1810_00845_amd import hisa, synth
    bits, B, seed = 50, 64, 3
    print("[case] N=2^%d L=%d dnum=%d batch %d" % (log_n, L, dnum, B), flush=True)
    g = hisa.Context(log_n, [bits] * L, dnum, bits, seed)
    o = Oracle(log_n, [bits] * L, dnum, bits, seed)
    try:
        assert g.primes == o.primes
        g.keygen(); o.keygen()
        g.gen_rot_keys([7]); o.gen_rot_keys([7])
        coeff = synth.uniform_residues(40 + log_n + L + dnum, (B, 2, L, g.N), g.primes[:L])
        gcts = g.ct_import_batch(coeff, 2.0 ** 50)
        gout, ran = launches(g, B, lambda: g.rot_left_batch(gcts, 7))
        assert ran == IN_REGISTERS
        for i in (0, 41):
            want = o.export(o.rot_left(o.import_ct(coeff[i], 2.0 ** 50), 7))
            assert np.array_equal(g.ct_export(gout[i]), want), "ciphertext %d differs" % i
        # one ciphertext, and both sides of the line between stored accumulators and those in registers
        for batch, rule in ((1, STORED), (most_stored, STORED), (most_stored + 1, IN_REGISTERS)):
            few, ran = launches(g, batch, lambda: g.rot_left_batch(gcts[:batch], 7))
            assert ran == rule, batch
            for i in (0, batch - 1):
                assert np.array_equal(g.ct_export(few[i]), g.ct_export(gout[i]))
        # relinearize + rescale through the same kernels (mode 4: the rescale)
        prod = g.mul_no_relin_batch(gcts, gcts[1:] + gcts[:1])
        g.relinearize_batch(prod)
        g.rescale_batch(prod)
        a, b = o.import_ct(coeff[5], 2.0 ** 50), o.import_ct(coeff[6], 2.0 ** 50)
        want = o.rescale(o.mul(a, b))
        assert np.array_equal(g.ct_export(prod[5]), o.export(want))
    finally:
        g.close()


@pytest.mark.parametrize("log_n", [12, 13, 14, 15])
def test_transforms_of_few_and_of_many_polynomials(log_n):
    """2^21 coefficients go by columns and rows of four waves, 2^22 by columns and rows of one wave, one polynomial more goes
    through whole-polynomial workgroups: the same values every way, and the oracle's."""
    import torch
    from oracle import Oracle
    from paper_1810_00845_amd import hisa, synth
    print("[case] transforms, N = 2^%d" % log_n, flush=True)
    g, o = hisa.Context(log_n, [50], 1, 50, 3), Oracle(log_n, [50], 1, 50, 3)
    try:
        few = (1 << 22) >> log_n
        a = synth.uniform_residues(log_n, (1, few + 1, 1, g.N), [g.primes[0]])[0, :, 0, :]
        many = torch.from_numpy(a.view(np.int64)).cuda()
        some, fewer = many[:few].clone(), many[:few // 2].clone()
        for inverse, mode in ((False, 0), (True, 1)):
            columns = "ntt_fp_split_kernel<%d, %d, true>" % (log_n - 10, mode)
            for t, want in ((fewer, {columns, "ntt_fp_split_wide_kernel<%d, %d>" % (log_n - 10, mode)}),
                            (some, {columns, "ntt_fp_split_kernel<%d, %d, false>" % (log_n - 10, mode)}),
                            (many, {"ntt_fp_kernel<%d, %d>" % (log_n - 10, mode)})):
                g.profile_enable(True)
                g.ntt_raw(t, 0, inverse=inverse)
                names = set(g.profile_read())
                g.profile_enable(False)
                assert names == want, names
            assert torch.equal(some, many[:few]) and torch.equal(fewer, many[:few // 2])
            if not inverse:
                for r in (0, few):
                    assert np.array_equal(many[r].cpu().numpy().view(np.uint64), o.ntt(a[r], 0))
        assert np.array_equal(many.cpu().numpy().view(np.uint64), a)
    finally:
        g.close()
