"""Encode, encrypt, decrypt and decode over ring degrees, limb counts and slot counts: the edges of the transforms over the
slot order (one chunk, one to five long stages, a prefix of the slots), of the digit recurrence's register forms, of the
encryption's plaintext table, and of the line between transforms by columns and rows and the single-launch ones."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# (log_n, q_bits, special_bits, vectors, slots)
POINTS = [
    (10, [30, 25], 30, 3, 512),
    (11, [40, 30, 30], 45, 2, 17),
    (12, [50], 50, 65, 2048),                   # one limb; one vector more than an encryption launch takes
    (12, [50, 40, 40, 40, 40], 50, 1, 16),
    (13, [50] + [40] * 8, 50, 2, 1),
    (14, [50] + [40] * 16, 50, 17, 8191),       # above the line: the single-launch transforms
    (15, [50] + [38] * 24, 50, 1, 16384),
    (16, [58, 50], 60, 1, 32768),
]


@pytest.mark.parametrize("log_n,q_bits,special,vectors,count", POINTS)
def test_round_trip(log_n, q_bits, special, vectors, count):
    from oracle import Oracle
    from paper_1810_00845_amd import hisa
    print("[case]", log_n, len(q_bits), vectors, count, flush=True)
    g, o = hisa.Context(log_n, q_bits, 1, special, 5), Oracle(log_n, q_bits, 1, special, 5)
    g.keygen(); o.keygen()
    rng = np.random.default_rng(log_n + count)
    limbs, scale = len(q_bits), 2.0 ** 20
    x = rng.uniform(-1, 1, (vectors, count)) + 1j * rng.uniform(-1, 1, (vectors, count))
    pts = [g.encode(v, scale, limbs) for v in x]
    cts = g.encrypt_batch(pts)
    for i in sorted({0, vectors - 1}):
        coeffs = g.pt_export(pts[i])[0].astype(np.int64)          # coefficients are far below the first prime
        coeffs[coeffs > g.primes[0] // 2] -= g.primes[0]
        e = np.asarray(coeffs, dtype=np.float64)
        z = np.zeros(g.slots, dtype=np.complex128)
        z[:count] = x[i]
        full = np.zeros(2 * g.N, dtype=np.complex128)             # slot j at exp(i pi 5^j / N), conjugates opposite
        p = np.array([pow(5, j, 2 * g.N) for j in range(g.slots)])
        full[p], full[2 * g.N - p] = z, z.conj()
        want = np.fft.fft(full)[:g.N].real * scale / g.N
        assert np.abs(e - want).max() <= 0.5 + 1e-6 * scale / 2 ** 20
        assert np.array_equal(g.pt_export(pts[i]), o.pt_export(o.pt_from_coeffs(coeffs, scale, limbs)))
        got = g.decode(pts[i], count)
        assert np.abs(got - x[i]).max() < 1e-3
        wide = g.decode(pts[i])
        assert np.allclose(wide[:count], got, rtol=0, atol=1e-12) and np.abs(wide[count:]).max(initial=0.0) < 1e-3
    for i in range(vectors):                                      # streams in order, whatever the batch
        if i in (0, vectors - 1):
            ct = o.encrypt(o.pt_from_coeffs(np.where((c := g.pt_export(pts[i])[0].astype(np.int64)) > g.primes[0] // 2,
                                                     c - g.primes[0], c), scale, limbs))
            assert np.array_equal(g.ct_export(cts[i]), o.export(ct))
        else:
            o.enc_counter += 1
    for i in sorted({0, vectors - 1}):
        assert np.abs(g.decode(g.decrypt(cts[i]), count) - x[i]).max() < 1e-1
    g.close()


@pytest.mark.parametrize("log_n,q_bits,special,batch,side", [
    (12, [50], 50, 65537, 1),                    # more ciphertexts than a grid has rows of entries
    (13, [50] + [40] * 7, 50, 1000, 2),          # sixteen groups, the last one ragged
    (13, [58] * 8, 60, 130, 2),                  # integer arithmetic, two full groups and two ciphertexts
])
def test_tensor_decrypt_in_groups(log_n, q_bits, special, batch, side):
    """Tensors of many ciphertexts of a few slots each, made of three ciphertexts used over and over: every image equals its
    ciphertext's, and the scratch memory does not grow with the tensor."""
    import torch
    from paper_1810_00845_amd import hisa
    print("[case] decrypt", log_n, len(q_bits), batch, side, flush=True)
    g = hisa.Context(log_n, q_bits, 1, special, 5)
    g.keygen()
    x = np.random.default_rng(batch).uniform(-1, 1, (3, 1, side, side))
    three = g.tensor_encrypt(x, 2.0 ** 30, len(q_bits))
    want = g.tensor_decrypt(three)
    assert np.abs(want - x).max() < 1e-4         # fresh noise: 3.2 sqrt(N) / scale a slot, 30 times that
    many = hisa.CipherTensor(g, [three.cts[i % 3] for i in range(batch)], batch, 1, side, side, three.h_stride, three.w_stride,
                             three.offset, 1, three.c_inner, three.c_stride)
    g.sync()
    free = torch.cuda.mem_get_info()[0]
    got = g.tensor_decrypt(many)
    grown = free - torch.cuda.mem_get_info()[0]
    assert np.array_equal(got, want[np.arange(batch) % 3])
    # plaintexts and coefficient forms of 2^22 coefficients, the lifted values and the transform's work: 32 MB each, and a
    # copy of the group's ciphertexts side by side, 64 MB; a ragged last group takes blocks of its own size
    assert grown <= 2 * (4 * 32 + 64) << 20, grown
    g.close()


@pytest.mark.parametrize("log_n,q_bits,special,batch,height,width", [
    (12, [50], 50, 65537, 1, 1),                 # more ciphertexts than a grid has rows of entries
    (13, [50] + [40] * 7, 50, 150, 2, 3),        # three groups, the last one ragged
    (11, [58, 50], 60, 64, 16, 64),              # integer arithmetic
    (12, [50], 50, 64, 32, 64),                  # 2^17 slot values: the most that are laid out in pinned memory
    (12, [50], 50, 65, 32, 64),                  # one ciphertext more: values scattered on the device
])
def test_tensor_encrypt_in_groups(log_n, q_bits, special, batch, height, width):
    """Every image of a tensor decrypts to itself, on both sides of the lines between one group of plaintexts and several and
    between slot vectors laid out on the host and on the device."""
    from paper_1810_00845_amd import hisa
    print("[case] encrypt", log_n, len(q_bits), batch, height, width, flush=True)
    g = hisa.Context(log_n, q_bits, 1, special, 5)
    g.keygen()
    x = np.random.default_rng(batch).uniform(-1, 1, (batch, 1, height, width))
    got = g.tensor_decrypt(g.tensor_encrypt(x, 2.0 ** 30, len(q_bits)))
    # a slot's noise is a sum of N coefficients of 3.2 and of N roundings: 3.3 sqrt(N) / scale = 2.8e-7 at most, of 65537
    # slots the largest below seven times that
    assert np.abs(got - x).max() < 2e-6
    g.close()


def test_vectors_handed_over_faster_than_they_are_read():
    """100 vectors of 128 KB, encoded without a wait in between, and decoded at the end: three times round the pinned memory
    that they pass through."""
    from paper_1810_00845_amd import hisa
    print("[case] 100 vectors, N = 2^14", flush=True)
    g = hisa.Context(14, [50, 40], 1, 50, 5)
    rng = np.random.default_rng(7)
    x = rng.uniform(-1, 1, (100, g.slots)) + 1j * rng.uniform(-1, 1, (100, g.slots))
    pts = [g.encode(v, 2.0 ** 30, 2) for v in x]
    # a slot's error is a sum of N roundings of at most 1/2: sqrt(N / 12) / scale = 3.5e-8, of 819200 slots the largest below
    # seven times that
    for v, pt in zip(x, pts):
        assert np.abs(g.decode(pt) - v).max() < 2.5e-7
    g.close()
