"""Descriptors that the library refuses reach it, or a Python error, through the native binding: no call may end the
process."""
import ctypes

import pytest
import torch

from paper_2105_13120_amd import rsa


def desc(N, L=64):
    d = rsa.make_desc(torch.empty(1, 1, 64, 64, dtype=torch.bfloat16), 1)
    d.N, d.L = N, L
    return d


def test_no_ranks():
    X, W = torch.empty(1, 64, 64, dtype=torch.bfloat16), torch.empty(64, 192, dtype=torch.bfloat16)
    with pytest.raises(ZeroDivisionError):
        rsa.qkv_proj(desc(0), X, W)


@pytest.mark.parametrize("N,L", [(-1, 64), (-1, -2 ** 63), (-3, 64), (3, -64)])
def test_negative_sizes(N, L):
    X, W = torch.empty(1, 64, 64, dtype=torch.bfloat16), torch.empty(64, 192, dtype=torch.bfloat16)
    d = desc(N, L)
    d.rank_begin, d.rank_end = 0, 1
    with pytest.raises((rsa.RSAError, RuntimeError)):
        rsa.qkv_proj(d, X, W)


def test_not_a_descriptor():
    X = torch.empty(1, 64, 64, dtype=torch.bfloat16)
    with pytest.raises((TypeError, ctypes.ArgumentError, AttributeError)):
        rsa.qkv_proj(b"no descriptor", X, X)


def test_the_library_alone_needs_hipcc_alone(monkeypatch):
    from paper_2105_13120_amd import build
    ran = []
    monkeypatch.setattr(build, "_run", lambda cmd, verbose: ran.append(cmd))
    assert build.build_library() == build.LIB_PATH
    assert len(ran) == 1 and not any("torch" in word or word.endswith("binding.cpp") for word in ran[0])
