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
    import torch
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are those of 256 CUs")
    w = make(n)
    ds = codec.to_device(codec.encode(w, layout=codec.make_layout(8, T, 11)))
    grid, block, _ = codec.launch_shape(ds)
    assert grid * (block // 64) == per_simd * 4 * 256
    out = torch.full((n,), 0x5555, dtype=torch.int16, device="cuda")
    codec.decode_block(ds, out.view(torch.bfloat16))
    torch.cuda.synchronize()
    assert torch.equal(out, torch.from_numpy(w.view(np.int16)).cuda())
