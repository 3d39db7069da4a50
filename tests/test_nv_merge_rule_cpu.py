"""The rule by which the NVFP4 prefill kernel adds the two activation operands
before the MFMA: for every pair of E4M3 scales that passes it, and every pair
of E2M1 codes, the sum of the two dequantized values is exact in fp16."""

import numpy as np

E2M1 = np.array([0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0])


def e4m3(code):
    e, m = (code >> 3) & 15, code & 7
    return m * 2.0 ** -9 if e == 0 else 2.0 ** (e - 7) * (1 + m / 8)


def passes(d1, d2):
    """The kernel's test, in fp32: the smaller scale's power of two by its exponent bits, at least 2^-6."""
    d1, d2 = np.float32(d1), np.float32(d2)
    pe = (np.minimum(d1, d2).view(np.uint32) & np.uint32(0x7F800000)).view(np.float32)
    return d1 + d2 <= np.maximum(pe, np.float32(2.0 ** -6)) * np.float32(21.25)


def test_merged_sums_are_exact_in_fp16():
    q = np.concatenate([E2M1, -E2M1])
    q1, q2 = q[:, None], q[None, :]
    merged = 0
    for c1 in range(127):       # every finite non-negative E4M3 code
        for c2 in range(127):
            d1, d2 = e4m3(c1), e4m3(c2)
            if not passes(d1, d2):
                continue
            merged += 1
            s = q1 * d1 + q2 * d2                    # fp64: exact
            assert np.array_equal(s.astype(np.float16).astype(np.float64), s), (c1, c2)
    # equal scales always merge, and so does any pair within a factor of 8 of each other
    assert all(passes(e4m3(c), e4m3(c)) for c in range(127))
    assert all(passes(e4m3(a), e4m3(b)) for a in range(8, 127) for b in range(a, min(a + 25, 127)))
    assert 127 * 127 // 4 < merged < 127 * 127
