"""Helpers shared by the GPU parity tests: host bits -> device tensors, oracle-side views; the plan of a block step."""
import ctypes

import numpy as np
import torch

import oracle
import workloads as wl


def attn_plan(lib, B, Hq, Hkv, Sq, Sk, D, offset=None):
    """(parts of the keys, packed heads) of a block step on these shapes; offset of the causal rule, None: no mask.  Host only."""
    def t(H, S, ptr):
        return lib.TrTensor(ptr, lib.TR_BF16, B, H, S, D, H * S * D, S * D, D)
    packed = ctypes.c_int32(-1)
    off = offset or 0
    parts = lib.raw_lib().tr_block_attn_plan(ctypes.byref(t(Hq, Sq, 0x7F0000000000)), ctypes.byref(t(Hkv, Sk, 0x7F8000000000)),
                                             int(offset is not None), max(off, 0), max(-off, 0), ctypes.byref(packed))
    return parts, packed.value


STEP_BF16, STEP_F32, STEP_MERGE, RING, RING_BF16 = range(5)


def attn_shape(lib, form, B, Hq, Hkv, Sq, Sk, D, offset=None, n=1):
    """(Query rows of a workgroup, key groups) of a call on these shapes; offset as above, n chunks of a ring.  Host only."""
    def t(H, S, ptr):
        return lib.TrTensor(ptr, lib.TR_BF16, B, H, S, D, H * S * D, S * D, D)
    groups = ctypes.c_int32(-1)
    off = offset or 0
    rows = lib.raw_lib().tr_attn_workgroup(ctypes.byref(t(Hq, Sq, 0x7F0000000000)), ctypes.byref(t(Hkv, Sk, 0x7F8000000000)),
                                           int(offset is not None), max(off, 0), max(-off, 0), form, n, ctypes.byref(groups))
    return rows, groups.value


def attn_per_unit(lib, form, B, Hq, Hkv, Sq, Sk, D, offset=None, n=1):
    """How many workgroups of that call share a compute unit: it tells the two launches of 64 rows and two key groups apart.  Host only."""
    def t(H, S, ptr):
        return lib.TrTensor(ptr, lib.TR_BF16, B, H, S, D, H * S * D, S * D, D)
    off = offset or 0
    return lib.raw_lib().tr_attn_workgroups_per_unit(ctypes.byref(t(Hq, Sq, 0x7F0000000000)), ctypes.byref(t(Hkv, Sk, 0x7F8000000000)),
                                                     int(offset is not None), max(off, 0), max(-off, 0), form, n)


def bits_to_dev(bits: np.ndarray) -> torch.Tensor:
    """bf16 bit patterns (uint16 numpy) -> bf16 torch tensor on cuda:0 with the same bits."""
    return torch.from_numpy(bits.view(np.int16)).to("cuda").view(torch.bfloat16)


def rand_bits(shape, seed, std=1.0):
    rng = np.random.Generator(np.random.PCG64(seed))
    return wl.f32_to_bf16_bits(rng.standard_normal(shape, dtype=np.float32) * np.float32(std))


def f64(bits):
    return wl.bf16_bits_to_f64(bits)


def to_np(t: torch.Tensor) -> np.ndarray:
    return t.detach().float().cpu().numpy().astype(np.float64)


def max_abs(a, b):
    a, b = np.asarray(a, dtype=np.float64), np.asarray(b, dtype=np.float64)
    both_ninf = np.isneginf(a) & np.isneginf(b)
    d = np.abs(np.where(both_ninf, 0.0, a) - np.where(both_ninf, 0.0, b))
    return float(np.max(d)) if d.size else 0.0


def check_rows(cfg, out, lse, qb, kb, vb, n_random, heads=None):
    """Compare sampled rows of every head against exact oracle rows."""
    rows = wl.sample_rows(cfg.S, cfg.chunk, n_random, seed=cfg.seed + 1)
    G = cfg.Hq // cfg.Hkv
    worst_o = worst_l = 0.0
    ridx = torch.from_numpy(rows).to("cuda")
    for h in (range(cfg.Hq) if heads is None else heads):
        g = h // G
        ref_o, ref_l = oracle.attention_rows(f64(qb[0, h][rows]), rows, f64(kb[0, g]), f64(vb[0, g]), cfg.scale, cfg.causal)
        worst_o = max(worst_o, max_abs(to_np(out[0, h][ridx]), ref_o))
        worst_l = max(worst_l, max_abs(to_np(lse[0, h][ridx]), ref_l))
    return worst_o, worst_l, len(rows)
