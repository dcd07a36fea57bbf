"""GPU parity: every HISA primitive through the C ABI against the CPU oracle.

Integer work is compared bit for bit in coefficient form on identical seeded
inputs; encode/decode (fp64) within tolerances derived from the arithmetic (stated where they are used).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

PARAMS = {
    # name: (log_n, q_bits, dnum, special_bits, seed)
    "n10_a1": (10, [30, 30, 30], 3, 60, 11),          # single-launch NTT, alpha = 1, mixed prime sizes
    "n12_a2": (12, [50, 40, 45, 50, 36], 3, 55, 12),  # two-launch NTT, alpha = 2, ragged last digit
    "n13_d1": (13, [55, 50, 50, 50], 1, 58, 13),      # dnum = 1: alpha = 4 special primes
    "n15_int": (15, [58, 55, 56], 3, 60, 18),         # the integer (Shoup / Barrett) kernels at the benchmark's ring degree
    # all primes below 2^50: the fp64 single-launch transforms and the fused key-switch pipeline
    "n12_fp": (12, [50, 40, 45, 50, 36], 3, 50, 14),  # alpha = 2, ragged last digit, mixed sizes
    "n13_fp": (13, [50, 50, 50, 50], 1, 50, 15),      # dnum = 1
    "n14_fp": (14, [50, 48, 45], 2, 49, 16),
    "n15_fp": (15, [50, 50, 50], 3, 50, 17),          # the benchmark's ring degree
    # the optional initialisation parameters: another error distribution, a secret of fixed Hamming weight
    "n12_sigma_fp": (12, [50, 40, 45], 3, 50, 20, dict(sigma=1.5)),
    "n12_hwt": (12, [50, 40, 45], 2, 55, 21, dict(secret_kind=1, hamming_weight=64, sigma=6.0)),
}


@pytest.fixture(scope="module", params=list(PARAMS))
def pair(request):
    from oracle import Oracle
    from paper_1810_00845_amd import hisa
    log_n, q_bits, dnum, sb, seed = PARAMS[request.param][:5]
    extra = PARAMS[request.param][5] if len(PARAMS[request.param]) > 5 else {}
    print("[case]", request.param, flush=True)
    g = hisa.Context(log_n, q_bits, dnum, sb, seed, **extra)
    o = Oracle(log_n, q_bits, dnum, sb, seed, **extra)
    g.keygen(); o.keygen()
    steps = [1, 7, g.slots - 3, 64]
    g.gen_rot_keys(steps); o.gen_rot_keys(steps)
    yield g, o
    g.close()


def fresh_pair(g, o, seed, limbs, bits=40, scale=2.0 ** 40):
    from paper_1810_00845_amd import synth
    co = synth.plaintext_coeffs(seed, g.N, bits)
    gp, op = g.pt_from_coeffs(co, scale, limbs), o.pt_from_coeffs(co, scale, limbs)
    ctr = 1000 + seed
    g.set_enc_counter(ctr); o.enc_counter = ctr
    return g.encrypt(gp), o.encrypt(op), gp, op


def same(g, o, gct, oct_):
    got = g.ct_export(gct)
    want = o.export(oct_)
    assert got.shape == want.shape
    assert np.array_equal(got, want), "mismatch at %s" % (np.argwhere(got != want)[:4],)
    assert abs(gct.scale - oct_.scale) <= 1e-12 * abs(oct_.scale)


def test_primes_match(pair):
    g, o = pair
    assert g.primes == o.primes and g.alpha == o.alpha


def test_ntt_raw_forward_inverse(pair):
    import torch
    from paper_1810_00845_amd import synth
    g, o = pair
    for prime in range(g.L + g.K):
        q = g.primes[prime]
        a = synth.uniform_residues(prime, (3, 1, g.N), [q])[:, 0, :]
        a[0, :4] = [0, q - 1, 1, q // 2]
        t = torch.from_numpy(a.view(np.int64)).cuda()
        g.ntt_raw(t, prime)
        got = t.cpu().numpy().view(np.uint64)
        for r in range(3):
            assert np.array_equal(got[r], o.ntt(a[r], prime))
        g.ntt_raw(t, prime, inverse=True)
        assert np.array_equal(t.cpu().numpy().view(np.uint64), a)


def test_secret_and_keys_match(pair):
    g, o = pair
    assert np.array_equal(g.secret_export(), o.secret_coeffs())
    assert np.array_equal(g.key_export(0), o.keys[0])
    for r in (1, 64):
        ge = g.galois_elt(r)
        assert ge == o.galois_elt(r)
        assert np.array_equal(g.key_export(ge), o.keys[ge])


def test_plaintext_and_encrypt_decrypt(pair):
    g, o = pair
    for limbs in (g.L, 1):
        gct, oct_, gp, op = fresh_pair(g, o, 3 + limbs, limbs)
        assert np.array_equal(g.pt_export(gp), o.pt_export(op))
        same(g, o, gct, oct_)
        assert np.array_equal(g.pt_export(g.decrypt(gct)), o.pt_export(o.decrypt(oct_)))
    # batch encryption uses consecutive counters
    from paper_1810_00845_amd import synth
    cos = [synth.plaintext_coeffs(50 + i, g.N, 30) for i in range(3)]
    g.set_enc_counter(77); o.enc_counter = 77
    gcts = g.encrypt_batch([g.pt_from_coeffs(c, 2.0 ** 30, g.L) for c in cos])
    for c, gc in zip(cos, gcts):
        same(g, o, gc, o.encrypt(o.pt_from_coeffs(c, 2.0 ** 30, g.L)))


def test_add_sub_mul_family(pair):
    g, o = pair
    ga, oa, gp, op = fresh_pair(g, o, 1, g.L)
    gb, ob, _, _ = fresh_pair(g, o, 2, g.L)
    same(g, o, g.add(ga, gb), o.add(oa, ob))
    same(g, o, g.sub(ga, gb), o.sub(oa, ob))
    same(g, o, g.add_plain(ga, gp), o.add_plain(oa, op))
    same(g, o, g.sub_plain(ga, gp), o.sub_plain(oa, op))
    same(g, o, g.mul_plain(ga, gp), o.mul_plain(oa, op))
    for x in (0.625, -1.75, 3.0e-7):
        same(g, o, g.add_scalar(ga, x), o.add_scalar(oa, x))
        same(g, o, g.sub_scalar(ga, x), o.sub_scalar(oa, x))
        same(g, o, g.mul_scalar(ga, x, 2.0 ** 33), o.mul_scalar(oa, x, 2.0 ** 33))
    same(g, o, g.mul_scalar(ga, -0.37, float(g.primes[g.L - 1])), o.mul_scalar(oa, -0.37, float(o.primes[o.L - 1])))
    g3, o3 = g.mul_no_relin(ga, gb), o.mul_no_relin(oa, ob)
    same(g, o, g3, o3)
    same(g, o, g.add_scalar(g3, 0.3), o.add_scalar(o3, 0.3))      # scale 2^80: beyond 64-bit integers
    same(g, o, g.add(g3, g.mul_plain(ga, gp)), o.add(o3, o.mul_plain(oa, op)))  # 3 + 2 polynomials
    # assign forms
    gc = g.copy(ga); g.add_assign(gc, gb); same(g, o, gc, o.add(oa, ob))
    gc = g.copy(ga); g.sub_assign(gc, gb); same(g, o, gc, o.sub(oa, ob))
    gc = g.copy(ga); g.mul_plain_assign(gc, gp); same(g, o, gc, o.mul_plain(oa, op))
    gc = g.copy(ga); g.mul_scalar_assign(gc, 0.5, 1024.0); same(g, o, gc, o.mul_scalar(oa, 0.5, 1024.0))
    gc = g.copy(ga); g.add_plain_assign(gc, gp); same(g, o, gc, o.add_plain(oa, op))
    gc = g.copy(ga); g.sub_scalar_assign(gc, 0.25); same(g, o, gc, o.sub_scalar(oa, 0.25))


def test_rescale_every_level(pair):
    g, o = pair
    gct, oct_, _, _ = fresh_pair(g, o, 4, g.L)
    g3, o3 = g.mul_no_relin(gct, gct), o.mul_no_relin(oct_, oct_)
    g.rescale(g3); o3 = o.rescale(o3)
    same(g, o, g3, o3)
    while gct.limbs > 1:
        d = g.max_scalar_div(gct, float("inf"))
        assert d == o.max_scalar_div(oct_, float("inf")) == g.primes[gct.limbs - 1]
        g.div_scalar(gct, d); oct_ = o.div_scalar(oct_, d)
        same(g, o, gct, oct_)
    assert g.max_scalar_div(gct, float("inf")) == 1


def test_rotations_every_level(pair):
    g, o = pair
    gct, oct_, _, _ = fresh_pair(g, o, 5, g.L)
    while True:
        for r in (1, 7, 64):
            same(g, o, g.rot_left(gct, r), o.rot_left(oct_, r))
        same(g, o, g.rot_right(gct, 3), o.rot_right(oct_, 3))
        same(g, o, g.rot_left(gct, 0), oct_)
        same(g, o, g.rot_left(gct, g.slots), oct_)
        if gct.limbs == 1:
            break
        g.rescale(gct); oct_ = o.rescale(oct_)
    gc = g.copy(gct); g.rot_left_assign(gc, 7); same(g, o, gc, o.rot_left(oct_, 7))
    gc = g.copy(gct); g.rot_right_assign(gc, 3); same(g, o, gc, o.rot_right(oct_, 3))


def test_relinearize_and_mul_every_level(pair):
    g, o = pair
    ga, oa, _, _ = fresh_pair(g, o, 6, g.L)
    gb, ob, _, _ = fresh_pair(g, o, 7, g.L)
    while True:
        g3, o3 = g.mul_no_relin(ga, gb), o.mul_no_relin(oa, ob)
        g.relinearize(g3)
        same(g, o, g3, o.relinearize(o3))
        same(g, o, g.mul(ga, gb), o.mul(oa, ob))
        if ga.limbs == 1:
            break
        g.rescale(ga); oa = o.rescale(oa)
        g.rescale(gb); ob = o.rescale(ob)
    gc = g.copy(ga); g.mul_assign(gc, gb); same(g, o, gc, o.mul(oa, ob))


def test_batched_forms_match_single_calls(pair):
    g, o = pair
    cts = [fresh_pair(g, o, 20 + i, g.L) for i in range(5)]
    gs, os_ = [c[0] for c in cts], [c[1] for c in cts]
    gp, op = cts[0][2], cts[0][3]
    for gr, oc in zip(g.rot_left_batch(gs, 7), os_):
        same(g, o, gr, o.rot_left(oc, 7))
    # handles that are not views of one allocation (gathered internally), ragged batch of 3
    mixed = [gs[4], gs[0], gs[2]]
    for gr, oc in zip(g.rot_left_batch(mixed, 1), [os_[4], os_[0], os_[2]]):
        same(g, o, gr, o.rot_left(oc, 1))
    for gr, oa, ob in zip(g.add_batch(gs[:4], gs[1:]), os_[:4], os_[1:]):
        same(g, o, gr, o.add(oa, ob))
    for gr, oc in zip(g.mul_plain_batch(gs, gp), os_):
        same(g, o, gr, o.mul_plain(oc, op))
    g3 = g.mul_no_relin_batch(gs[:4], gs[1:])
    o3 = [o.mul_no_relin(a, b) for a, b in zip(os_[:4], os_[1:])]
    for a, b in zip(g3, o3):
        same(g, o, a, b)
    g.relinearize_batch(g3)
    o2 = [o.relinearize(x) for x in o3]
    for a, b in zip(g3, o2):
        same(g, o, a, b)
    g.rescale_batch(g3)
    for a, b in zip(g3, o2):
        same(g, o, a, o.rescale(b))


@pytest.mark.parametrize("log_n,limbs", [(10, 3), (13, 8), (15, 5)])
def test_products_and_sums_beyond_the_last_level_cache(log_n, limbs):
    """The largest products and sums of 256 MB, operands and result together, and one ciphertext more, which go another way (squares
    do not): single calls' values, and the launches that ran."""
    from paper_1810_00845_amd import hisa
    print("[case]", log_n, limbs, flush=True)
    g = hisa.Context(log_n, [50] * limbs, 1, 50, 5)

    def both_sides(polys, fn):
        few = (256 << 20) // (polys * limbs * 8 * g.N)
        for n in (few, few + 1):
            a, b = g.ct_random_batch(n, limbs, 1.0, 1000), g.ct_random_batch(n, limbs, 1.0, 500000)
            g.profile_enable(True)
            got, x, y = fn(a, b)
            names = set(g.profile_read())
            g.profile_enable(False)
            for i in (0, 1, n // 2, n - 1):
                assert np.array_equal(g.ct_export(got[i]), g.ct_export(fn([x[i]], [y[i]], True)))
            yield names

    def product(a, b, one=False):
        return g.mul_no_relin(a[0], b[0]) if one else (g.mul_no_relin_batch(a, b), a, b)

    def square(a, b, one=False):
        return g.mul_no_relin(a[0], a[0]) if one else (g.mul_no_relin_batch(a, a), a, a)

    def total(a, b, one=False):
        return g.add(a[0], b[0]) if one else (g.add_batch(a, b), a, b)

    def of_products(a, b, one=False):                   # three polynomials each
        x, y = (a, b) if one else (g.mul_no_relin_batch(a, a), g.mul_no_relin_batch(a, b))
        return g.add(x[0], y[0]) if one else (g.add_batch(x, y), x, y)

    assert list(both_sides(7, product)) == [{"mul_no_relin_kernel"}, {"mul_no_relin_stream_kernel"}]
    assert list(both_sides(7, square)) == [{"mul_no_relin_kernel"}] * 2
    for names in list(both_sides(6, total)) + list(both_sides(9, of_products)):
        assert "addsub_kernel" in names
    g.close()


def test_hoisted_rotations_equal_single_rotations(pair):
    """Several rotations sharing one decomposition of c1 give, bit for bit, what the oracle's rotLeft gives, at the
    top level and two levels down, with a step that is a plain copy and handles from different allocations."""
    g, o = pair
    cts = [fresh_pair(g, o, 40 + i, g.L) for i in range(3)]
    gs, os_ = [c[0] for c in cts], [c[1] for c in cts]
    steps = [1, 0, 7, 64, g.slots - 3]
    for _ in range(2):
        out = g.rot_left_hoisted_batch([gs[2], gs[0], gs[1]], steps)
        assert len(out) == len(steps) and all(len(row) == 3 for row in out)
        for row, r in zip(out, steps):
            for gr, oc in zip(row, [os_[2], os_[0], os_[1]]):
                same(g, o, gr, o.rot_left(oc, r))
        if gs[0].limbs <= 2:
            break
        for i in range(3):
            g.rescale(gs[i]); os_[i] = o.rescale(os_[i])
            if gs[i].limbs > 2:
                g.rescale(gs[i]); os_[i] = o.rescale(os_[i])
    from paper_1810_00845_amd import hisa
    with pytest.raises(hisa.HisaError) as e:
        g.rot_left_hoisted_batch(gs, [1, 5])          # no key for 5
    assert e.value.code == -4


def test_rotation_sums_match_oracle(pair, request):
    """Sums of rotated ciphertexts with one division by P per output: bit for bit the oracle's sum of key-switch
    accumulators (SharedModDown with unit weights), at the top level and one level down, with and without an unrotated
    term, terms from different allocations; contexts without the fused key switch refuse the call."""
    from oracle.layers import SharedModDown
    from paper_1810_00845_amd import hisa
    g, o = pair
    fused = request.node.callspec.id.endswith("_fp")
    n_out = 3
    cts = [fresh_pair(g, o, 60 + i, g.L) for i in range(4 * n_out)]
    gs, os_ = [c[0] for c in cts], [c[1] for c in cts]
    if not fused:
        with pytest.raises(hisa.HisaError) as e:
            g.rot_left_sum_batch([gs[:n_out], gs[n_out:2 * n_out]], [1, 7])
        assert e.value.code == -1
        return
    for level in range(2):
        for steps in ([1, 0, 7, g.slots - 3], [64, 7], [0]):
            terms = [[gs[(s * n_out + b + level) % len(gs)] for b in range(n_out)] for s in range(len(steps))]
            oterms = [[os_[(s * n_out + b + level) % len(gs)] for b in range(n_out)] for s in range(len(steps))]
            out = g.rot_left_sum_batch(terms, steps)
            assert len(out) == n_out
            for b in range(n_out):
                ins = [oterms[s][b] for s in range(len(steps))]
                want = SharedModDown(o, ins).total([(s, steps[s], 1, None) for s in range(len(steps))], ins[0].scale)
                same(g, o, out[b], want)
        # all rotated terms the same ciphertext (one decomposition per output): the same bits as with copies of it
        steps = [7, 0, 1, 64]
        out = g.rot_left_sum_batch([gs[:n_out]] * 4, steps)
        for b in range(n_out):
            want = SharedModDown(o, [os_[b]] * 4).total([(s, steps[s], 1, None) for s in range(4)], os_[b].scale)
            same(g, o, out[b], want)
        out2 = g.rot_left_sum_batch([gs[:n_out], gs[n_out:2 * n_out], gs[:n_out]], [7, 0, 1])
        for b in range(n_out):
            ins = [os_[b], os_[n_out + b], os_[b]]
            same(g, o, out2[b], SharedModDown(o, ins).total([(0, 7, 1, None), (1, 0, 1, None), (2, 1, 1, None)], ins[0].scale))
        if level == 0:
            # the decrypted sum is the sum of the decrypted rotations (top level only: the rescaling below leaves
            # these 40-bit test messages only a few bits above its rounding)
            steps = [1, 0, 7]
            out = g.rot_left_sum_batch([[gs[s]] for s in range(3)], steps)
            z = g.decode(g.decrypt(out[0]), g.slots)
            ref = sum(np.roll(g.decode(g.decrypt(gs[s]), g.slots), -steps[s]) for s in range(3))
            assert np.abs(z - ref).max() <= 1e-6 * max(1.0, np.abs(ref).max())
        if gs[0].limbs <= 2:
            break
        for i in range(len(gs)):
            g.rescale(gs[i]); os_[i] = o.rescale(os_[i])
    if request.node.callspec.id in ("n12_fp", "n13_fp"):
        # more than 32 outputs: the launch that keeps a rotation's key rows across sixteen outputs, ragged last block
        many = [fresh_pair(g, o, 100 + i, g.L) for i in range(35)]
        mg, mo = [c[0] for c in many], [c[1] for c in many]
        shifted = mg[1:] + mg[:1]
        out = g.rot_left_sum_batch([mg, shifted, mg], [7, 1, 0])
        for b in range(35):
            ins = [mo[b], mo[(b + 1) % 35], mo[b]]
            same(g, o, out[b], SharedModDown(o, ins).total([(0, 7, 1, None), (1, 1, 1, None), (2, 0, 1, None)], ins[0].scale))
    with pytest.raises(hisa.HisaError) as e:
        g.rot_left_sum_batch([gs[:1], gs[1:2]], [1, 5])                  # no key for 5
    assert e.value.code == -4
    with pytest.raises(hisa.HisaError) as e:
        g.rot_left_sum_batch([gs[:1], gs[1:2], gs[2:3]], [0, 1, 0])      # two unrotated terms
    assert e.value.code == -1


def test_import_export_roundtrip(pair):
    from paper_1810_00845_amd import synth
    g, o = pair
    co = synth.uniform_residues(9, (2, 2, g.L, g.N), g.primes[:g.L])
    for gc, c in zip(g.ct_import_batch(co, 4.0), co):
        assert np.array_equal(g.ct_export(gc), c)
        same(g, o, gc, o.import_ct(c, 4.0))


def centred_coeffs(o, coeff_form, limbs):
    """Centred integers from coefficient-form residues (CRT with Python integers)."""
    import math
    qs = o.primes[:limbs]
    Q = math.prod(qs)
    out = []
    for k in range(coeff_form.shape[1]):
        x = 0
        for i, q in enumerate(qs):
            hat = Q // q
            x += int(coeff_form[i, k]) * pow(hat, -1, q) * hat
        x %= Q
        out.append(x - Q if x > Q // 2 else x)
    return out


def test_encode_decode_within_tolerance(pair):
    """fp64 on the GPU against long double in the oracle: coefficients agree to the fp64 rounding of a
    sum of N/2 terms, |delta| <= max(1, 2^-45 * scale * sqrt(N)); decoded slots to 2^-20 and to the
    encoding error bound N/(2*scale)."""
    from paper_1810_00845_amd import synth
    g, o = pair
    z = synth.slot_vector(1, g.slots, complex_values=True)
    for scale, count in ((2.0 ** 25, g.slots), (2.0 ** 45, g.slots), (2.0 ** 30, 37)):
        gp = g.encode(z[:count], scale, g.L)
        assert gp.limbs == g.L and gp.scale == scale
        got = centred_coeffs(o, g.pt_export(gp), g.L)
        want = o.encode_coeffs(z[:count], scale)
        tol = max(1.0, 2.0 ** -45 * scale * g.N ** 0.5)
        assert max(abs(a - int(b)) for a, b in zip(got, want)) <= tol
        dec = g.decode(gp)
        ref = np.zeros(g.slots, dtype=complex); ref[:count] = z[:count]
        assert np.abs(dec - ref).max() <= g.N / (2 * scale) + 2.0 ** -20
        # GPU decode of the oracle's plaintext against the oracle's decode
        op = o.encode(z[:count], scale, g.L)
        gp2 = g.pt_from_coeffs(want, scale, g.L)
        assert np.abs(g.decode(gp2) - o.decode(op)).max() <= 2.0 ** -20
    # end to end through encryption
    gct = g.encrypt(g.encode(z.real, 2.0 ** 40, g.L))
    assert np.abs(g.decode(g.decrypt(gct)) - z.real).max() < 1e-6


def test_error_codes(pair):
    from paper_1810_00845_amd import hisa
    g, o = pair
    gct, oct_, gp, _ = fresh_pair(g, o, 30, g.L)
    def code(fn, *a):
        with pytest.raises(hisa.HisaError) as e:
            fn(*a)
        return e.value.code
    assert code(g.rot_left, gct, 5) == -4                      # no key for this amount
    assert code(g.add, gct, g.mul_scalar(gct, 1.0, 2.0)) == -3  # scale mismatch
    if g.L > 1:
        low = g.copy(gct); g.rescale(low)
        assert code(g.add, gct, low) == -2                     # level mismatch
        assert code(g.mul_plain, low, gp) == -2
        assert code(g.div_scalar, gct, g.primes[0]) == -5      # not the last modulus
        g.div_scalar(gct, 1)                                   # d = 1: no-op
        same(g, o, gct, oct_)
        while low.limbs > 1:
            g.rescale(low)
        assert code(g.rescale, low) == -6                      # depth exhausted
    assert code(g.mul_no_relin, g.mul_no_relin(gct, gct), gct) == -9


def test_bad_initialisation_parameters_are_refused():
    from paper_1810_00845_amd import hisa
    for kw in (dict(sigma=0.1), dict(sigma=11.0), dict(secret_kind=2), dict(secret_kind=1, hamming_weight=0),
               dict(secret_kind=1, hamming_weight=(1 << 10) + 1)):
        with pytest.raises(hisa.HisaError) as e:
            hisa.Context(10, [40, 40], 2, 45, 1, **kw)
        assert e.value.code == -1


def test_fixed_weight_secret_has_its_weight():
    from paper_1810_00845_amd import hisa
    g = hisa.Context(10, [40, 40], 2, 45, 5, secret_kind=1, hamming_weight=1 << 10)
    s = g.secret_export()
    assert np.count_nonzero(s) == 1 << 10 and set(np.unique(s)) == {-1, 1}
    g.close()


def test_largest_ring_degree_on_the_integer_kernels():
    """N = 2^16 (the largest the library accepts; beyond the fp64 transforms' range) with primes above 2^50: the
    strided two-launch transforms, one rotation and one multiply / relinearise / rescale, bit for bit."""
    import torch
    from oracle import Oracle
    from paper_1810_00845_amd import hisa, synth
    log_n, q_bits, dnum, sb, seed = 16, [58, 55], 2, 60, 19
    print("[case] n16_int", flush=True)
    g, o = hisa.Context(log_n, q_bits, dnum, sb, seed), Oracle(log_n, q_bits, dnum, sb, seed)
    try:
        assert g.primes == o.primes
        for prime in range(g.L + g.K):
            q = g.primes[prime]
            a = synth.uniform_residues(40 + prime, (2, 1, g.N), [q])[:, 0, :]
            a[0, :4] = [0, q - 1, 1, q // 2]
            t = torch.from_numpy(a.view(np.int64)).cuda()
            g.ntt_raw(t, prime)
            got = t.cpu().numpy().view(np.uint64)
            for r in range(2):
                assert np.array_equal(got[r], o.ntt(a[r], prime))
            g.ntt_raw(t, prime, inverse=True)
            assert np.array_equal(t.cpu().numpy().view(np.uint64), a)
        g.keygen(); o.keygen()
        g.gen_rot_keys([3]); o.gen_rot_keys([3])
        ga, oa, _, _ = fresh_pair(g, o, 41, g.L)
        gb, ob, _, _ = fresh_pair(g, o, 42, g.L)
        same(g, o, g.rot_left(ga, 3), o.rot_left(oa, 3))
        gm, om = g.mul_no_relin(ga, gb), o.mul_no_relin(oa, ob)
        g.relinearize(gm)
        om = o.relinearize(om)
        same(g, o, gm, om)
        g.rescale(gm)
        same(g, o, gm, o.rescale(om))
    finally:
        g.close()
