"""The native argument marshalling of the per-layer calls (csrc/qoq_py.cpp): what it refuses, and on which stream it launches."""
import numpy as np
import pytest
import torch

from paper_2405_04532_amd import api
from paper_2405_04532_amd import workloads as wl

gpu = pytest.mark.gpu
DEV = "cuda:0"
M, K, N = 16, 256, 256
B, T, HKV, H, S, D = 2, 3, 2, 4, 64, 128


@pytest.fixture(scope="module", autouse=True)
def built():
    import os
    if not (os.path.exists(api.LIB_PATH) and os.path.exists(api.NATIVE_PATH)):
        from paper_2405_04532_amd import build
        build.build()


class NoTruth:
    """A flag without a truth value, as an array of several elements has none."""
    def __bool__(self):
        raise ValueError("no truth value")


@gpu
def test_a_flag_without_a_truth_value_raises_its_own_error():
    x, gamma = torch.ones((M, K), dtype=torch.float16, device=DEV), torch.ones(K, dtype=torch.float16, device=DEV)
    perm = torch.arange(K, dtype=torch.int32, device=DEV)
    for call in (lambda f: api.quant_act_per_token(x, f), lambda f: api.quant_act_per_token(x, True, f),
                 lambda f: api.quant_act_per_token_reordered(x, perm, f), lambda f: api.quant_act_per_token_reordered(x, perm, True, f),
                 lambda f: api.rmsnorm_quant(x, gamma, 1e-5, f), lambda f: api.rmsnorm_quant(x, gamma, 1e-5, True, f),
                 lambda f: api.rmsnorm_quant(x, gamma, 1e-5, True, True, f),
                 lambda f: api.silu_mul_quant(x, f), lambda f: api.silu_mul_quant(x, True, f), lambda f: api.silu_mul_quant(x, True, True, f)):
        with pytest.raises(ValueError, match="no truth value"):
            call(NoTruth())
        assert len(call(np.bool_(True))) in (4, 5)
    with pytest.raises(ValueError):
        api.rmsnorm_quant(x, gamma, "small")
    for eps in ("1e-5", np.float32(1e-5), torch.tensor(1e-5)):                   # whatever float() takes
        assert len(api.rmsnorm_quant(x, gamma, eps)) == 5
