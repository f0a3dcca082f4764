"""The decoder's waves per SIMD: one stream on each side of every line of its
rule (which depends on chunks per CU, block size and mean code length), decoded
bit-exactly in the launch it gets.  The rule's "hold" only delays a wave, so
the decoded weights show that its branch is taken without harm."""
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


@pytest.mark.parametrize("T,make,n,per_simd", [
    (64, gaussian, 20_000_003, 5), (64, gaussian, 26_000_001, 4), (64, gaussian, 32_000_005, 3),
    (64, random_bits, 6_900_007, 5), (64, random_bits, 8_000_001, 4),
    (64, random_bits, 25_800_009, 3), (128, gaussian, 80_000_001, 2),
    (128, two_sigmas, 80_000_001, 3), (128, random_bits, 25_800_009, 3),
    (256, gaussian, 80_000_001, 3), (256, two_sigmas, 80_000_001, 4)],
    ids=lambda v: getattr(v, "__name__", str(v)))
def test_waves_per_simd(T, make, n, per_simd):
    check(T, 11, make, n, per_simd)


@pytest.mark.parametrize("T,make,n,per_simd", [
    (64, gaussian, 26_000_001, 6), (64, gaussian, 32_000_005, 3), (128, gaussian, 80_000_001, 2),
    (128, two_sigmas, 80_000_001, 3)], ids=lambda v: getattr(v, "__name__", str(v)))
def test_waves_per_simd_with_large_tables(T, make, n, per_simd):
    """12-bit tables: fewer workgroups fit a CU, and the rule's waves still do."""
    check(T, 12, make, n, per_simd)


def test_workgroups_fit_the_lds_they_are_given():
    """Blocks of about 5,100 weights with 12-bit tables: three 4-wave workgroups
    fit a CU's LDS by plain bytes, two by the 1280-byte pieces it is given out
    in.  A launch has as many workgroups as run at once."""
    import torch
    rng = np.random.default_rng(12)
    e = np.clip(np.round(rng.normal(115, 0.6, 1 << 22)), 1, 254).astype(np.uint16)
    w = np.resize((e << 7) | rng.integers(0, 128, e.size, dtype=np.uint16), 126_000_001)
    ds = codec.to_device(codec.encode(w, layout=codec.make_layout(8, 128, 12)))
    grid, _, lds = codec.launch_shape(ds)
    p = torch.cuda.get_device_properties(0)
    pieces = -(-lds // 1280)
    assert grid <= p.multi_processor_count * (160 * 1024 // (1280 * pieces))
    out = torch.full((w.size,), 0x5555, dtype=torch.int16, device="cuda")
    codec.decode_block(ds, out.view(torch.bfloat16))
    torch.cuda.synchronize()
    assert torch.equal(out, torch.from_numpy(w.view(np.int16)).cuda())


def check(T, K, make, n, per_simd):
    import torch
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are those of 256 CUs")
    w = make(n)
    ds = codec.to_device(codec.encode(w, layout=codec.make_layout(8, T, K)))
    grid, block, _ = codec.launch_shape(ds)
    assert grid * (block // 64) == per_simd * 4 * 256
    out = torch.full((n,), 0x5555, dtype=torch.int16, device="cuda")
    codec.decode_block(ds, out.view(torch.bfloat16))
    torch.cuda.synchronize()
    assert torch.equal(out, torch.from_numpy(w.view(np.int16)).cuda())
