"""The native entry points of the binding: names, defaults, and what they refuse before the library is called (no GPU)."""
import inspect

import pytest
import torch

sq = pytest.importorskip("paper_2105_11010_amd")

D = sq.conv_desc(1, 4, 4, 16, 8)
M = sq.mode()
X = torch.zeros(256, dtype=torch.uint8)
OPTIONAL = {"acc": None, "scale": None, "out": None, "workspace": None}


@pytest.mark.parametrize("name,required,optional", [
    ("sparq_trim", "x y m", {}), ("sparq_dequant", "acc scale out", {}), ("sparq_requant", "acc factor y", {}),
    ("sparq_conv_gemm", "x packed d m", OPTIONAL), ("sparq_conv_gemm_sparse24", "x packed d m", OPTIONAL),
    ("sparq_conv_gemm_packed", "packed_x group packed_w d m", OPTIONAL),
    ("sparq_conv_gemm_u8", "x packed d m factor y", {"workspace": None, "out_mode": None}),
    ("sparq_pack_act", "x packed m", {"group": 1}), ("sparq_unpack_act", "packed y m", {"group": 1})])
def test_signatures(name, required, optional):
    parameters = inspect.signature(getattr(sq, name)).parameters
    assert list(parameters) == required.split() + list(optional)
    assert {k: p.default for k, p in parameters.items() if p.default is not p.empty} == optional


@pytest.mark.parametrize("error,text,call", [
    (TypeError, "missing", lambda: sq.sparq_trim(X, X)),
    (TypeError, "unexpected keyword", lambda: sq.sparq_trim(X, X, M, z=1)),
    (TypeError, "multiple values", lambda: sq.sparq_trim(X, X, M, x=X)),
    (TypeError, "at most", lambda: sq.sparq_trim(X, X, M, 1)),
    (TypeError, "must be a tensor", lambda: sq.sparq_trim(3, X, M)),
    (TypeError, "SparqConvDesc", lambda: sq.sparq_conv_gemm(X, X, M, M)),
    (TypeError, "x must be a contiguous device tensor of dtype torch.uint8", lambda: sq.sparq_conv_gemm(X, X, D, M, acc=None)),
    (TypeError, "workspace must be a contiguous device tensor", lambda: sq.sparq_conv_gemm(X, X, D, M, workspace=X)),
    (ValueError, "activation size", lambda: sq.sparq_conv_gemm(X[1:], X, D, M)),
    (ValueError, "out must hold M\\*N = 128", lambda: sq.sparq_conv_gemm(X, X, D, M, out=X)),
    (ValueError, "scale must hold N", lambda: sq.sparq_conv_gemm(X, X, D, M, scale=X)),
    (ValueError, "factor must hold N", lambda: sq.sparq_conv_gemm_u8(X, X, D, M, X, X[:128])),
    (ValueError, "y must hold M\\*N", lambda: sq.sparq_conv_gemm_u8(X, X, D, M, X[:8], X)),
    (ValueError, "same shape", lambda: sq.sparq_trim(X, X[1:], M)),
    (ValueError, "two dimensions", lambda: sq.sparq_dequant(X, X, X)),
    (ZeroDivisionError, "division", lambda: sq.sparq_conv_gemm(X, X, sq.conv_desc(1, 4, 4, 16, 8, stride=(0, 1)), M)),
], ids=lambda v: v.__name__ if isinstance(v, type) else None)
def test_refused_before_the_library_is_called(error, text, call):
    with pytest.raises(error, match=text):
        call()
