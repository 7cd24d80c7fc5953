"""The C-ABI library loads and exports every entry point include/sd.h declares
(no compute calls: this runs without a GPU)."""
import ctypes
import os
import re
import struct

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    lib_path = os.path.join(ROOT, "paper_2211_17192_amd", "libsd.so")
    if not os.path.exists(lib_path):
        from paper_2211_17192_amd import build
        build.build(verbose=False)
    header = open(os.path.join(ROOT, "include", "sd.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    names = set(re.findall(r"\b(sd_[a-z_]+)\s*\(", header))
    assert {"sd_load_models", "sd_prefill", "sd_step", "sd_reset", "sd_step_baseline", "sd_spec_sample"} <= names
    lib = ctypes.CDLL(lib_path)
    for n in sorted(names):
        assert hasattr(lib, n), n


def kernels_of_the_library():
    """name -> what the compiler notes of each kernel of the built library (its code object's metadata)."""
    msgpack = pytest.importorskip("msgpack")
    with open(os.path.join(ROOT, "paper_2211_17192_amd", "libsd.so"), "rb") as f:
        data = f.read()
    out, at = {}, data.find(b"AMDGPU\0\0")
    while at >= 0:
        namesz, descsz, kind = struct.unpack("<III", data[at - 12:at])
        if (namesz, kind) == (7, 32):
            out.update((k[".name"], k) for k in msgpack.unpackb(data[at + 8:at + 8 + descsz], strict_map_key=False)["amdhsa.kernels"])
        at = data.find(b"AMDGPU\0\0", at + 8)
    assert len(out) > 100
    return out


def test_attention_kernels_keep_their_registers():
    """What the matrix-core attention kernels put into scratch lies outside their key loops: a handful of registers.  (47 with
    position bias, heads of 128 and two row tiles, where two steps' biases were held at once.)"""
    spilled = {n: k[".vgpr_spill_count"] for n, k in kernels_of_the_library().items() if "attn_mma_kernel" in n}
    assert len(spilled) > 20 and max(spilled.values()) <= 8, {n: v for n, v in spilled.items() if v > 8}


def test_no_attention_kernel_is_built_that_nothing_launches():
    """bf16 heads of 64 and 128 have the matrix-core kernel, which merges its key ranges itself; two row tiles of a decoding
    forward need several query heads per KV head, which models with position bias or cross-attention do not have."""
    names = list(kernels_of_the_library())
    assert any("attn_kernelIDF16bLi32E" in n for n in names) and any("attn_kernelIfLi128E" in n for n in names)
    assert not [n for n in names if re.search(r"attn_(merge_)?kernelIDF16bLi(64|128)E", n)]
    assert not [n for n in names if re.search(r"attn_mma_kernelILi\d+ELi2ELi\dELi[12]ELi0E", n)]


def test_workspace_sizing_needs_no_gpu():
    from paper_2211_17192_amd import binding, synth
    cfg_p, _, cfg_q, _ = synth.tiny_pair()
    cp, cq = binding._cfg_struct(cfg_p), binding._cfg_struct(cfg_q)
    rt = binding._RuntimeCfg(batch=1, max_gamma=4, page_size=16)
    n = binding.lib.sd_workspace_bytes(ctypes.byref(cp), ctypes.byref(cq), ctypes.byref(rt))
    assert 100_000 < n < 50_000_000
    rt.batch = 4                                    # four sequences: four times the KV pages and activations,
    n4 = binding.lib.sd_workspace_bytes(ctypes.byref(cp), ctypes.byref(cq), ctypes.byref(rt))   # plus the batched GEMMs' scratch
    assert n < n4 < 6 * n
    rt.batch = 65
    assert binding.lib.sd_workspace_bytes(ctypes.byref(cp), ctypes.byref(cq), ctypes.byref(rt)) == 0
    rt.batch, rt.max_gamma = 1, 16
    assert binding.lib.sd_workspace_bytes(ctypes.byref(cp), ctypes.byref(cq), ctypes.byref(rt)) == 0


def test_choose_gamma_matches_brute_force_and_the_papers_rule():
    """Section 3.5 host logic through the C ABI: the chosen gamma maximises Theorem 3.8
    (checked against the oracle's search and a direct evaluation), gamma never shrinks as
    alpha grows or c falls, and Corollary 3.9's condition alpha > c decides whether any
    gamma gives an improvement."""
    import numpy as np
    from oracle import analysis
    from paper_2211_17192_amd import binding
    for c in (0.0, 0.01, 0.02, 0.05, 0.1, 0.2, 0.4):
        prev = 0
        for alpha in np.linspace(0.05, 0.95, 19):
            g, v = binding.choose_gamma(alpha, c, 15)
            assert g == analysis.optimal_gamma(alpha, c, 15)
            direct = (1 - alpha ** (g + 1)) / ((1 - alpha) * (g * c + 1))
            assert abs(v - direct) < 1e-12 * direct
            for other in range(1, 16):
                assert v >= analysis.walltime_improvement(alpha, other, c) - 1e-12
            assert (v > 1.0) == (alpha > c) or abs(alpha - c) < 1e-9
            assert g >= prev
            prev = g
    # c = 0: more guesses always help, the search stops at the cap
    assert binding.choose_gamma(0.5, 0.0, 7)[0] == 7
    g = ctypes.c_int32(0)
    for bad in ((1.0, 0.1, 5), (-0.1, 0.1, 5), (0.5, -1.0, 5), (0.5, 0.1, 0), (float("nan"), 0.1, 5)):
        assert binding.lib.sd_choose_gamma(bad[0], bad[1], bad[2], ctypes.byref(g), None) == binding.SD_EINVAL


def test_bench_refuses_more_than_one_gpu_and_unknown_workloads():
    """bench.py runs on one GPU only and says so; its command line is checked before anything
    touches a GPU."""
    import subprocess, sys, os
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=120)
    assert r.returncode != 0 and "one GPU" in (r.stderr + r.stdout)
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--workload", "nope"], capture_output=True, text=True, timeout=120)
    assert r.returncode != 0 and "invalid choice" in r.stderr


def decoder_without_a_gpu(monkeypatch, pinned):
    """A SpecDecoder that hands out host arrays; pinned(n) stands for the allocation of n values in pinned memory."""
    from paper_2211_17192_amd import binding
    empty = binding.torch.empty
    monkeypatch.setattr(binding.torch, "empty", lambda n, pin_memory=False, **kw: pinned(n) if pin_memory else empty(n, **kw))
    dec = object.__new__(binding.SpecDecoder)
    dec._ctx, dec._pinned = ctypes.c_void_p(), []
    return dec


def test_pinned_host_arrays_are_bounded_in_bytes(monkeypatch):
    import torch
    taken, zeros = [], torch.zeros
    dec = decoder_without_a_gpu(monkeypatch, lambda n: taken.append(n) or zeros(n))
    n = 64 * 8 * 32000                                # 64 sequences' logits at gamma 7: 66 MB
    held = [dec._host_array(n) for _ in range(8)]
    assert all(x.shape == (n,) and x.dtype.name == "float32" for x in held)
    assert taken and 4 * sum(taken) <= 128 << 20
    before = len(taken)
    held.clear()                                      # dead arrays no longer count
    held.append(dec._host_array(n))
    assert len(taken) == before + 1
    assert dec._host_array(8 * n).shape == (8 * n,) and len(taken) == before + 1
    assert dec._host_array(0).shape == (0,)


def test_host_arrays_without_pinned_memory(monkeypatch):
    def none_left(n):
        raise RuntimeError("HIP error: out of memory")
    dec = decoder_without_a_gpu(monkeypatch, none_left)
    a = dec._host_array(1000)
    a[:] = 1.0
    assert a.shape == (1000,) and a.dtype.name == "float32" and not dec._pinned
