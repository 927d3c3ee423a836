"""Values at the ends of the storage types through the exact-logits kernels; the wide one holds bf16 operands as the upper halves of fp64 values."""
import pytest
import torch


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("M,E,wide", [(8, 72, 0), (8, 120, 120), (40, 128, 128), (40, 232, 232), (24, 136, 128)])
def test_wide_logits_of_extreme_values(ffn_rules, dtype, M, E, wide):
    """`wide` of the experts on the wide kernel (blocks of 64, the last one partly filled; part of a chunk of 32 k), the others on the narrow one.  Zeros of both signs, subnormals, the largest values, infinities and NaN against fp64: not-a-number and infinite where that is, else within one
    rounding (2^-23: the sums themselves err by M 2^-53 of the largest term, and no two large terms cancel.  A large weight beside the large tokens does
    not belong here: products of 4e38 of either sign leave what the others sum to within 8 * 2^-53 * 4e38, any order being as good)."""
    from paper_2206_03382_amd import moe
    T = 2 ** 22 // E + 33
    assert ffn_rules.wide_logits(T, E, 1) == wide
    gen = torch.Generator(device="cuda").manual_seed(E)
    x, Wg = (torch.rand(s, generator=gen, device="cuda") + 0.5 for s in ((T, M), (M, E)))
    big, tiny = float(torch.finfo(dtype).max), float(torch.finfo(dtype).smallest_normal)
    for i, v in enumerate((0.0, -0.0, tiny / 4, -tiny / 8, tiny, big, -big, float("inf"), float("-inf"), float("nan"))):
        x[i::50, i % M] = v
        x[i + 20::50] = v
    Wg[:, 3], Wg[:, 5] = tiny / 4, -0.0
    x, Wg = x.to(dtype), Wg.to(dtype)
    got, want = moe.gate_logits(x, Wg), (x.double() @ Wg.double()).float()
    assert torch.equal(got.isnan(), want.isnan()) and torch.equal(got.isinf(), want.isinf())
    on = want.isfinite()
    assert bool((got[on] - want[on]).abs().le(2.0 ** -23 * want[on].abs() + 2.0 ** -149).all()) and bool((got[want.isinf()] == want[want.isinf()]).all())
