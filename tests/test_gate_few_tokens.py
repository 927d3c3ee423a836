"""The gate of up to 16 tokens, whose logits and decisions are one launch (gate_few_tokens_kernel in csrc/gate.hip)."""
import ctypes
import os
import subprocess

import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_rule(tmp_path):
    """One tile of tokens, and everything that decisions in one block ask for."""
    (tmp_path / "r.cpp").write_text('#include "paper_2206_03382_amd/csrc/gate_rules.h"\n'
                                    'extern "C" int few(int64_t T, int64_t E, int k, int64_t C) { return moe::gate_of_few_tokens(T, E, k, C); }\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", ROOT, str(tmp_path / "r.cpp"), "-o", str(tmp_path / "r.so")], check=True)
    few = ctypes.CDLL(str(tmp_path / "r.so")).few
    few.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int64]
    assert all(few(*a) for a in ((1, 3, 1, 1), (16, 4, 4, 16), (16, 8, 4, 32), (13, 16, 2, 0), (5, 5, 5, 1000)))
    assert not any(few(*a) for a in ((17, 8, 2, 8), (16, 17, 1, 8), (16, 2, 1, 8), (16, 1, 1, 8), (16, 16, 3, 8), (16, 8, 2, 4096)))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("T,M,E,k,C", [(1, 8, 3, 1, 1), (16, 2048, 8, 2, 8), (15, 40, 4, 4, 3), (16, 1032, 5, 5, 16), (9, 256, 9, 3, 2), (16, 520, 16, 2, 4), (2, 4096, 16, 1, 900),
                                       (17, 256, 8, 2, 8), (16, 256, 2, 2, 16)])
def test_same_as_logits_and_decisions_apart(dtype, T, M, E, k, C):
    """Bit for bit, with equal tokens and equal gate columns among them (ties), a token of zeros, with a gate bias and without."""
    from paper_2206_03382_amd import moe
    gen = torch.Generator(device="cuda").manual_seed(T * M + E)
    for bias in (None, torch.randn(E, generator=gen, device="cuda")):
        for normalize in (0, 1):
            x = torch.randn(T, M, generator=gen, device="cuda").to(dtype)
            Wg = (torch.randn(M, E, generator=gen, device="cuda") / M ** 0.5).to(dtype)
            x[T // 2] = 0
            x[-1] = x[0]
            Wg[:, -1] = Wg[:, 0]
            got = moe.gate_route(x, Wg, bias, k, C, normalize)
            logits = moe.gate_logits(x, Wg, bias)
            want = moe.gate_topk(logits.clone(), k, C, normalize)
            for name in ("idx", "loc", "gate_w", "counts", "slot_src"):
                assert torch.equal(got[name], want[name]), name
            if "logits" in got:
                assert torch.equal(got["logits"], logits)
