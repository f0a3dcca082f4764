"""The decoder's waves per SIMD: a stream on each side of the lines of its rule
(chunks per CU, block size, mean code length against the table's index width),
decoded bit-exactly in the launch it gets.  The rule's "hold" only delays a
wave, so the decoded weights show that its branch is taken without harm."""
import numpy as np
import pytest

from paper_2504_11651_amd import codec, synth

from conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs an MI355X")]


def random_bits(n):
    """Uniform 16-bit patterns: every exponent equally likely, codes of 8 bits."""
    return np.random.default_rng(9).integers(0, 65536, n, dtype=np.uint16)


def gaussian(n):
    return synth.gaussian(n, 0.02, 6)


def two_sigmas(n):
    """One code book for two standard deviations: a mean code of 2.67 bits."""
    w = synth.gaussian(n, 0.02, 6)
    w[:n // 2] = synth.gaussian(n // 2, 0.011, 7)
    return w


def exponents(n, sd):
    """Normally distributed exponents, random signs and mantissas."""
    rng = np.random.default_rng(12)
    e = np.clip(np.round(rng.normal(115, sd, 1 << 22)), 1, 254).astype(np.uint16)
    return np.resize((e << 7) | rng.integers(0, 128, e.size, dtype=np.uint16), n)


def short_codes(n):
    return exponents(n, 0.6)  # a mean code of 1.63 bits


def long_codes(n):
    return exponents(n, 2.2)  # 3.24 bits


def longer_codes(n):
    return exponents(n, 3.8)  # 4.0 bits


def one_symbol(n):
    return np.full(n, 0x3C12, np.uint16)


@pytest.mark.parametrize("T,K,make,n,per_simd", [
    (64, 11, gaussian, 34_000_003, 5), (64, 11, gaussian, 38_000_001, 3),
    (64, 11, long_codes, 27_000_005, 5), (64, 11, long_codes, 30_000_005, 3),
    (64, 11, longer_codes, 22_000_005, 7), (64, 11, longer_codes, 30_000_005, 4), (64, 11, random_bits, 25_800_009, 7),
    (64, 11, one_symbol, 100_000_007, 6), (64, 9, two_sigmas, 34_000_003, 7),
    (64, 9, two_sigmas, 38_000_001, 4), (64, 9, gaussian, 38_000_001, 3), (64, 9, short_codes, 60_000_005, 3),
    (64, 12, gaussian, 20_000_003, 6), (64, 12, gaussian, 24_000_001, 4),
    (64, 12, gaussian, 38_000_001, 3),
    (128, 11, gaussian, 75_000_001, 4), (128, 11, gaussian, 80_000_001, 2),
    (128, 11, two_sigmas, 80_000_001, 3),
    (128, 11, two_sigmas, 260_000_001, 2), (128, 11, long_codes, 64_000_003, 3),
    (128, 11, longer_codes, 60_000_005, 4), (128, 11, random_bits, 25_800_009, 4),
    (128, 11, short_codes, 126_000_001, 4), (128, 10, gaussian, 80_000_001, 3),
    (128, 9, gaussian, 80_000_001, 3), (128, 9, two_sigmas, 80_000_001, 4), (128, 12, gaussian, 80_000_001, 2),
    (256, 11, gaussian, 75_000_001, 6), (256, 11, two_sigmas, 80_000_001, 3),
    (256, 11, long_codes, 64_000_003, 4), (256, 9, gaussian, 80_000_001, 4),
    (256, 11, random_bits, 25_800_009, 7),
    (512, 11, gaussian, 75_000_001, 6), (512, 11, gaussian, 80_000_001, 4),
    (512, 9, two_sigmas, 80_000_001, 6), (512, 11, random_bits, 25_800_009, 6),
    (1024, 11, gaussian, 75_000_001, 4), (1024, 11, gaussian, 80_000_001, 4)],
    ids=lambda v: getattr(v, "__name__", str(v)))
def test_waves_per_simd(T, K, make, n, per_simd):
    import torch
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are those of 256 CUs")
    assert decoded_shape(T, K, make(n))[:2] == (per_simd * 4 * 256, per_simd)


def test_workgroups_fit_the_lds_they_are_given():
    """Blocks of 20,300 weights with 12-bit tables: three workgroups fit a CU's
    LDS by plain bytes, two by the 1280-byte pieces it is given out in.  A
    launch has as many workgroups as run at once."""
    import torch
    _, _, grid, lds = decoded_shape(512, 12, short_codes(50_000_003))
    assert 160 * 1024 // lds == 3 and 160 * 1024 // (1280 * -(-lds // 1280)) == 2
    assert grid == 2 * torch.cuda.get_device_properties(0).multi_processor_count


def decoded_shape(T, K, w):
    """Waves, waves per SIMD, workgroups and LDS of the launch, after decoding."""
    import torch
    ds = codec.to_device(codec.encode(w, layout=codec.make_layout(8, T, K)))
    grid, block, lds = codec.launch_shape(ds)
    out = torch.full((w.size,), 0x5555, dtype=torch.int16, device="cuda")
    codec.decode_block(ds, out.view(torch.bfloat16))
    torch.cuda.synchronize()
    assert torch.equal(out, torch.from_numpy(w.view(np.int16)).cuda())
    waves = grid * (block // 64)
    return waves, waves / (4 * torch.cuda.get_device_properties(0).multi_processor_count), grid, lds
