"""What the library puts on which stream, seen from the HIP calls it makes (launch_log.cpp stands in for the runtime; no GPU)."""
import os
import subprocess

import pytest

from oracle import transformer as T
from paper_2211_17192_amd import binding, synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    lib = os.path.join(ROOT, "paper_2211_17192_amd")
    exe = str(tmp_path_factory.mktemp("launches") / "launch_log")
    subprocess.run(["g++", "-std=c++17", "-O1", "-rdynamic", "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "launch_log.cpp"),
                    os.path.join(lib, "libsd.so"), "-Wl,-rpath," + lib, "-Wl,--allow-shlib-undefined", "-o", exe], check=True)

    def go(cfg_p, cfg_q, *calls):
        """One list of lines per call."""
        text = []
        for cfg in (cfg_p, cfg_q):
            keys = ("arch", "n_layers", "d_model", "n_heads", "n_kv_heads", "d_head", "d_ff", "vocab", "max_len", "enc_len")
            text.append("model " + " ".join(str(int(cfg[k])) for k in keys) + (" 1" if cfg["dtype"] == "bf16" else " 0"))
            for name, (shape, _) in synth.weight_shapes(cfg).items():
                text.append(f"tensor {name} {shape[0]} {shape[1] if len(shape) > 1 else 0}")
        res = subprocess.run([exe], input="\n".join(text + list(calls)) + "\n", text=True, capture_output=True, timeout=60)
        assert res.returncode == 0, res.stderr
        out, part = [], []
        for line in res.stdout.splitlines():
            if line.startswith("call "):
                out.append(part)
                part = []
            elif line == "loaded":
                part = []
            else:
                part.append(line)
        return out
    return go


def launches(lines):
    """(stream, kernel, grid, notes) of every launch."""
    words = [l.split() for l in lines if l.startswith("launch ")]
    return [(int(w[1]), w[2], tuple(int(v) for v in w[3:6]), tuple(w[6:])) for w in words]


def pair(arch, max_len=200, layers=2, dtype="bf16", **kw):
    cfg = synth.model_cfg(arch, layers, 256, 4, 512, 512, max_len, d_head=64, dtype=dtype, **kw)
    return cfg, dict(cfg, n_layers=1)


@pytest.mark.parametrize("arch,kw", [(T.GPT, {}), (T.T5DEC, dict(enc_len=61)), (T.GQA, dict(n_kv_heads=2))])
def test_a_callers_stream_gets_every_launch(run, arch, kw):
    """sd_runtime_cfg.stream: every call enqueues on it (a caller may have masked its CUs, or time what is on it)."""
    calls = ["load 1 4 1 1 0", "prefill 0 100", "step 4 1.0", "prefill 0 9", "measure", "plain 1.0"]
    for call, lines in zip(calls, run(*pair(arch, **kw), *calls)):
        assert launches(lines) and {l.split()[1] for l in lines if l.split()[0] in ("launch", "copy", "graph", "sync", "record")} == {"0"}, call


def test_the_contexts_own_streams_are_both_waited_for(run):
    """Without a caller's stream Mq's prompt runs beside Mp's; the host waits for both and nothing is enqueued behind."""
    _, lines = run(*pair(T.GQA), "load 1 4 0 0 0", "prefill 0 100")
    assert {l[0] for l in launches(lines)} == {1, 2}
    assert sorted(lines[-2:]) == ["sync 1", "sync 2"]


@pytest.mark.parametrize("least", [0, 1])           # passes of 2048 rows and a last one of 9; of 16 rows
def test_key_ranges_of_both_prompts_are_spread(run, least):
    """Each pass of up to 16 rows over a long context gives Mq's key ranges the workgroups that Mp's, of the same heads, get."""
    cfg, _ = pair(T.GQA, max_len=3000)
    _, lines = run(cfg, cfg, f"load 1 4 0 0 {least}", "prefill 0 2058")
    attn = {s: [(k, g) for s2, k, g, _ in launches(lines) if s2 == s and "attn_mma_kernel" in k] for s in (1, 2)}
    assert len(attn[1]) == (129 if least else 2) and attn[1][-1][1] == (4, 1, 6)           # (the last layer's is left out)
    assert attn[2] == attn[1]


@pytest.mark.parametrize("options", [[], ["filter"]])
@pytest.mark.parametrize("arch,dtype,kw,batch", [(T.GPT, "f32", {}, 1), (T.GPT, "f32", {}, 18), (T.T5DEC, "bf16", dict(enc_len=61), 1),
                                                 (T.GQA, "bf16", dict(n_kv_heads=2), 1), (T.GQA, "bf16", dict(n_kv_heads=2), 18)])
def test_measurements_time_what_an_iteration_runs(run, arch, dtype, kw, batch, options):
    """sd_measure_cost and sd_time_forward: the launches of a draft step that is neither the first nor the last of an iteration, of
    its verify forward and of a plain step; only the fetch of the parameters, once an iteration, is nobody's."""
    prefill = [f"prefill {b} 9" for b in range(batch)]
    calls = [f"load {batch} 4 1 1 0", *options, *prefill, "measure", "time 1 1", "time 0 4", "time 0 1", "step 3 1.0", *prefill, "plain 1.0"]
    out = dict(zip(calls, run(*pair(arch, dtype=dtype, **kw), *calls)))

    def graphs(call):
        got = []
        for line in out[call]:
            if line == "begin":
                got.append([])
            elif line == "end":
                got.append(None)
            elif got and got[-1] is not None:
                got[-1].append(line)
        return [[(k, g, n) for _, k, g, n in launches(part)] for part in got if part is not None]

    (step,), (plain,) = graphs("step 3 1.0"), graphs("plain 1.0")
    draws = [i for i, (k, _, _) in enumerate(step) if "sample_row" in k]
    accept = next(i for i, (k, _, _) in enumerate(step) if "accept" in k or "row_parts" in k or "row_filter_kernelI" in k and i > draws[2])
    assert len(draws) == 3 and [n for _, _, n in step].count(("fetches",)) == 1 and plain[0][2] == ("fetches",)
    again, verify = step[draws[0] + 1: draws[1] + 1], step[draws[2] + 1: accept]
    plain[0] = (*plain[0][:2], ())
    assert again[-1][2] == ("embeds",)
    assert graphs("measure") == [again, plain]
    assert graphs("time 1 1") == [again[:-1]] and graphs("time 0 4") == [verify] and graphs("time 0 1") == [plain[:-1]]


def test_weights_pass_the_l2s_only_where_they_would_not_stay(run):
    """32 sequences: each product of a small draft's step leaves its weights in the L2s for the next step; those of 32 MB and more that one row tile
    of workgroups reads go past them."""
    small = synth.model_cfg(T.GQA, 1, 1024, 8, 4096, 8192, 200, n_kv_heads=8, d_head=128, dtype="bf16")
    large = synth.model_cfg(T.GQA, 1, 4096, 32, 14336, 8192, 200, n_kv_heads=8, d_head=128, dtype="bf16")
    calls = ["load 32 3 1 1 0", *(f"prefill {b} 9" for b in range(32)), "time 1 1", "time 0 2"]
    past = [["Lb1E" in k for _, k, _, _ in launches(lines) if "gemm_rows_kernel" in k or "gemm_slices_kernel" in k]
            for lines in run(large, small, *calls)[-2:]]
    assert past[0] == [False] * 5                              # QKV, O, FFN-in, FFN-out, LM head
    assert past[1] == [True, False, True, True]                # (64 rows: O by two row tiles; FFN-out is gemm_split_kernel's)


# (rows, gamma, vocabulary, beta): three workgroups a sequence; beta's three and two for the draw; beta's three and, where a round has
# room for one more only, the draw's three after all
@pytest.mark.parametrize("case,workgroups", [((85, 3, 9000, 0), 255), ((86, 3, 9000, 0), 258), ((51, 3, 9000, 1), 255), ((52, 3, 9000, 1), 312)])
def test_a_cu_of_its_own_where_the_workgroups_are_no_more_than_the_cus(run, case, workgroups):
    """Which of its two builds an accept call takes (on 256 CUs)."""
    (lines,) = run(*pair(T.GPT), "sample " + " ".join(map(str, case)))
    (_, kernel, grid, _), = [l for l in launches(lines) if "accept_kernel" in l[1]]
    assert grid[0] * grid[1] == workgroups and ("accept_kernelILi0ELb1E" in kernel) == (workgroups <= 256)
