"""Test-side glue: move torch tensors to the numpy forms the oracle takes."""
import ctypes

import numpy as np
import torch

from paper_2603_24840_amd.workloads import bits, npy  # noqa: F401  (host views shared with bench.py and smoke())


def f32_to_bf16_bits(x):
    """Round-to-nearest-even float32 -> bf16 bit patterns."""
    u = np.asarray(x, dtype=np.float32).view(np.uint32).astype(np.uint64)
    return ((u + 0x7FFF + ((u >> 16) & 1)) >> 16).astype(np.uint16)


def bf16_tensor_from_bits(b, device):
    return torch.from_numpy(np.ascontiguousarray(b).view(np.int16)).view(torch.bfloat16).to(device)


def to_dev(x, device, dtype=None):
    """numpy array (an input, or an oracle result rounded to the interface dtype) -> device tensor."""
    a = np.ascontiguousarray(x if dtype is None else np.asarray(x).astype(dtype))
    return torch.from_numpy(a).to(device)


def oracle_survivors(O, prob_f32, cfg):
    """Survivors the oracle selects from fp32 probabilities (numpy), as (keep_mask, survivor_idx)."""
    return O.select(np.asarray(prob_f32, dtype=np.float32), cfg.n_prompts, cfg.G, cfg.K, cfg.rho)


def _mlp_query(name, A, n, d, m, delta_terms, gathered, row_stride):
    out = [ctypes.c_int32() for _ in range(3)]
    rc = getattr(A.lib(), name)(n, d, m, row_stride or d, int(gathered), delta_terms, *[ctypes.byref(x) for x in out])
    assert rc == 0
    return tuple(x.value for x in out)


def mlp_kernels(A, n, d, m, delta_terms, gathered=False, row_stride=None):
    """(forward, weight gradient, splits) that the MLP calls take for a batch, numbered as in the header: a test that is
    there for one kernel says so, and fails when a changed choice leads its sizes elsewhere."""
    return _mlp_query("arrol_score_mlp_kernels", A, n, d, m, delta_terms, gathered, row_stride)


def mlp_tiles(A, n, d, m, delta_terms, gathered=False, row_stride=None):
    """(wavefront groups of the forward blocks, units and wavefront groups of a weight gradient block), as above."""
    return _mlp_query("arrol_score_mlp_tiles", A, n, d, m, delta_terms, gathered, row_stride)


def logprob_kernel(A, T, V, d, n_splits=0):
    """(kernel, tile rows, tile tokens, splits) of a log-prob call, as above."""
    out = [ctypes.c_int32() for _ in range(4)]
    assert A.lib().arrol_logprob_kernel(T, V, d, n_splits, *[ctypes.byref(x) for x in out]) == 0
    return tuple(x.value for x in out)


def logprob_streamed(A, T, V, d, n_splits=0):
    """Whether that call loads the LM head past the caches."""
    out = ctypes.c_int32()
    assert A.lib().arrol_logprob_streamed(T, V, d, n_splits, ctypes.byref(out)) == 0
    return bool(out.value)
