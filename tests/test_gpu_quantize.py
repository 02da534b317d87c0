"""ffd_quantize_keys on the GPU: bit-exact against the oracle's decomposition and packing."""
import numpy as np
import pytest
import torch

import ffd_inputs as I
from oracle import ffd_oracle as O
from tests.gpu_util import Uploaded, bits_to_bf16

pytestmark = pytest.mark.gpu


def _gpu_quantize(k_bits, t_begin=0, t_end=None, fill=None, bits=2):
    from paper_2609_00097_amd import ffd
    k = bits_to_bf16(k_bits)
    B, Hkv, Lcap, _ = k.shape
    codes, absmax, resid = ffd.empty_quantized(B, Hkv, Lcap, "cuda", bits)
    for t in (codes, absmax, resid):
        t.view(torch.uint8).fill_(0 if fill is None else fill)
    ffd.quantize_keys(k, t_begin, t_end, out=(codes, absmax, resid))
    torch.cuda.synchronize()
    return (codes.cpu().numpy().view(np.uint32), absmax.cpu().view(torch.int16).numpy().view(np.uint16),
            resid.cpu().numpy())


def _assert_equal_packed(gpu, ref, name):
    for g, r, what in zip(gpu, ref, ("codes", "absmax", "resid")):
        assert np.array_equal(g, r), f"{name}: {what} differ at {np.argwhere(g != r)[:5].tolist()}"


@pytest.mark.parametrize("bits", [2, 4, 8])
def test_workload1_bit_exact(bits):
    c = I.workload(1)
    print(f"case {c.name} seed {c.seed} bits {bits}", flush=True)
    _assert_equal_packed(_gpu_quantize(c.k, bits=bits), O.quantize_cache(c.k, bits=bits), c.name)


@pytest.mark.parametrize("bits", [2, 4, 8])
def test_ragged_small_batch_bit_exact(bits):
    c = I.small_case(seed=7, B=3, Hq=8, Hkv=4, seq_lens=(100, 257, 64), Lcap=320)
    _assert_equal_packed(_gpu_quantize(c.k, bits=bits), O.quantize_cache(c.k, bits=bits), "small")


@pytest.mark.parametrize("bits", [2, 4, 8])
@pytest.mark.parametrize("M", [1.5, 3.140625, 0.0078125, 117.0, 1.0e-30, 2.0e30, 3.0e38, 1.0e-38])
def test_every_bf16_value_against_an_absmax(M, bits):
    """All finite bf16 values x with |x| <= M, 127 per token next to the absmax M (App. A edges;
    the bin edges of the 4- and 8-bit codebooks; absmaxes near the top and bottom of the range)."""
    Mb = O.bf16_to_f64(O.f64_to_bf16_bits(np.array([M])))[0]
    x = O.bf16_to_f64(np.arange(65536, dtype=np.uint32).astype(np.uint16))
    x = x[np.isfinite(x) & (np.abs(x) <= Mb)]
    ntok = -(-x.size // 127)
    Lcap = -(-ntok // 64) * 64
    vals = np.zeros((Lcap, 128))
    vals[:, 0] = Mb
    flat = np.zeros(Lcap * 127)
    flat[:x.size] = x
    vals[:, 1:] = flat.reshape(Lcap, 127)
    vals[ntok:] = 0.0                               # zero tokens: M = 0 case
    vals[1::2, 0] = -Mb                             # the absmax element negative on odd tokens
    k_bits = O.f64_to_bf16_bits(vals).reshape(1, 1, Lcap, 128)
    print(f"case every-bf16 M={M} bits={bits}", flush=True)
    _assert_equal_packed(_gpu_quantize(k_bits, bits=bits), O.quantize_cache(k_bits, bits=bits),
                         f"M={M} bits={bits}")


@pytest.mark.parametrize("bits", [2, 4, 8])
def test_partial_range_leaves_other_tokens_untouched(bits):
    c = I.small_case(seed=9, B=1, Hq=4, Hkv=2, seq_lens=(256,))
    got = _gpu_quantize(c.k, 70, 133, fill=0xA5, bits=bits)
    ref = O.quantize_cache(c.k, 70, 133, bits=bits)
    codes = O.unpack_codes(got[0][0, 0], 256, bits)
    ref_codes = O.unpack_codes(ref[0][0, 0], 256, bits)
    assert np.array_equal(codes[70:133], ref_codes[70:133])
    full_sentinel = np.full_like(got[0], 0xA5A5A5A5)
    untouched = O.unpack_codes(full_sentinel[0, 0], 256, bits)
    assert np.array_equal(codes[:70], untouched[:70]) and np.array_equal(codes[133:], untouched[133:])
    # a single appended token (decode-step append)
    got1 = _gpu_quantize(c.k, 200, 201, fill=0, bits=bits)
    ref1 = O.quantize_cache(c.k, 200, 201, bits=bits)
    _assert_equal_packed(got1, ref1, "append one token")


@pytest.mark.parametrize("bits", [2, 4, 8])
def test_ties_and_edges_of_every_absmax_mantissa(bits):
    """Each of the 128 bf16 mantissas of M as a token of its own, at exponents on both sides of the
    fp32 path's range (so that a tile mixes both paths) and in a range that starts and ends inside a
    block: values nearest to rounding ties (h + 1/2) M / (254 Lv) and bin edges j M / Lv, +-M/2 (always
    a tie), +-M, tiny values and zeros of either sign. Bit-exact."""
    rng = np.random.default_rng(17 + bits)
    Lv, Lcap, t0, t1 = (2 ** bits - 1) / 2, 192, 7, 7 + 128
    vals = np.zeros((Lcap, 128))
    for i, mant in enumerate(range(128, 256)):
        M = mant / 128 * 2.0 ** (0, 3, -20, 99, 101, -99, -101)[i % 7]
        h = rng.integers(0, int(254 * Lv), size=60)
        edges = rng.integers(-int(Lv), int(Lv) + 1, size=40) * M / Lv
        ties = (h + 0.5) * M / (254 * Lv) * rng.choice([-1.0, 1.0], size=60)
        fixed = [M, -M, M / 2, -M / 2, M * 2.0 ** -24, -M * 2.0 ** -24, 0.0, -0.0]
        row = np.concatenate([fixed, ties, edges, rng.uniform(-M, M, 20)])
        row = O.bf16_to_f64(O.f64_to_bf16_bits(row))
        vals[t0 + i] = rng.permutation(np.where(np.abs(row) > M, M, row))
    k_bits = O.f64_to_bf16_bits(vals).reshape(1, 1, Lcap, 128)
    print(f"case ties and edges bits={bits}", flush=True)
    _assert_equal_packed(_gpu_quantize(k_bits, t0, t1, bits=bits), O.quantize_cache(k_bits, t0, t1, bits=bits),
                         f"ties bits={bits}")


@pytest.mark.parametrize("bits", [2, 4, 8])
def test_smallest_values_next_to_every_absmax_exponent(bits):
    """Three mantissas of M at every bf16 exponent, next to values down to the smallest subnormal of
    either sign: the sign of a value far below M still decides its level (a negative one lies in the bin
    below 0), also where its quotient by M is no fp32 number. The quantizer, and append_kv with one token
    per sequence, bit-exact."""
    from paper_2609_00097_amd import ffd
    rng = np.random.default_rng(29 + bits)
    rows = []
    for e in range(-133, 128):
        for mant in (1.0, 129 / 128, 255 / 128):
            M = O.bf16_to_f64(O.f64_to_bf16_bits(np.array([mant * 2.0 ** e])))[0]
            gaps = np.concatenate([np.arange(140, 166), rng.integers(0, 261, 35)])
            low = np.maximum(2.0 ** (e - gaps.astype(np.float64)), 2.0 ** -133)
            low = np.concatenate([low, [2.0 ** -133, 2.0 ** -126]])
            row = np.minimum(np.concatenate([low, low * 1.9921875]), M)
            row = O.bf16_to_f64(O.f64_to_bf16_bits(row)) * rng.choice([-1.0, -1.0, 1.0], size=126)
            rows.append(np.concatenate([[M, -M], row]))
    vals = np.array(rows)
    ntok = len(vals)
    Lcap = -(-ntok // 64) * 64
    k_bits = np.zeros((1, 1, Lcap, 128), dtype=np.uint16)
    k_bits[0, 0, :ntok] = O.f64_to_bf16_bits(vals)
    print(f"case smallest values bits={bits}", flush=True)
    _assert_equal_packed(_gpu_quantize(k_bits, bits=bits), O.quantize_cache(k_bits, bits=bits), f"bits={bits}")
    one = np.zeros((ntok, 1, 64, 128), dtype=np.uint16)              # a sequence per token
    one[:, 0, 0] = k_bits[0, 0, :ntok]
    qk = ffd.quantize_keys(bits_to_bf16(np.zeros_like(one)), bits=bits)
    k_new = bits_to_bf16(one[:, :, 0])
    lens = torch.zeros(ntok, dtype=torch.int32, device="cuda")
    ffd.append_kv(k_new, k_new, qk, lens)
    torch.cuda.synchronize()
    got = (qk[0].cpu().numpy().view(np.uint32), qk[1].cpu().view(torch.int16).numpy().view(np.uint16), qk[2].cpu().numpy())
    _assert_equal_packed(got, O.quantize_cache(one, bits=bits), f"append bits={bits}")
