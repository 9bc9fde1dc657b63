"""Host-side checks of bench.py that need no GPU: the multi-GPU refusal and the workloads the default run covers."""
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused_with_a_message():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 2
    assert "single-GPU" in r.stderr and r.stdout.strip() == ""


def test_default_run_covers_both_configurations_the_bandwidth_target_names():
    """The baseline's metric names no configuration; its target sentence names the OLMoE-like and the Mixtral-like
    ones.  The default line is quoted on the OLMoE-like layer (the second baseline configuration) and carries a
    section for a cut of the Mixtral-like stack (the third)."""
    sys.path.insert(0, ROOT)
    import bench
    from workload import get_config
    saved = sys.argv
    sys.argv = ["bench.py"]
    try:
        a = bench.parse()
    finally:
        sys.argv = saved
    assert a.gpus == 1 and a.workload == "olmoe_like" and a.second_layers > 0
    base = json.load(open(os.path.join(ROOT, "BASELINE.json")))
    assert "OLMoE-like and Mixtral-like" in base["north_star"]
    for name, want in (("olmoe_like", base["configs"][1]), ("mixtral_like", base["configs"][2])):
        cfg = get_config(name)
        text = json.dumps(want).lower()
        for value in (cfg.n_experts, cfg.top_k, cfg.d_model, cfg.d_ff, cfg.capacity, cfg.n_layers):
            assert str(value) in text, (name, value)


def test_launch_names_follow_the_rule_of_the_library():
    import re
    sys.path.insert(0, ROOT)
    import bench
    from workload import get_config
    text = open(os.path.join(ROOT, "paper_2602_11192_amd", "csrc", "routed_prologue.hpp")).read()
    assert int(re.search(r"kShareFrags = (\d+)", text).group(1)) == bench.SHARED_LOGITS_KIB      # (fragments of a KiB)
    olmoe, mixtral = get_config("olmoe_like"), get_config("mixtral_like")
    assert bench.single_launch_kernels(olmoe) == ("decode_shared_kernel", "combine_clear_kernel")
    assert bench.single_launch_kernels(olmoe, int4=True)[0] == "decode_shared_q4_kernel"
    assert bench.single_launch_kernels(mixtral, tiles=True) == ("decode_tiles_kernel", "combine_chunks_kernel")
    fp32 = get_config("tiny_fp32")
    assert bench.single_launch_kernels(fp32) == ("token_layer_kernel",)
    files = ("ffn_fused.hip", "ffn_tiles.hip", "ffn_fused_q4.hip", "ffn_rowmajor.hip")
    kernels = "".join(open(os.path.join(ROOT, "paper_2602_11192_amd", "csrc", f)).read() for f in files)
    for cfg in (olmoe, mixtral, fp32):
        for kw in (dict(), dict(tiles=True), dict(int4=True)):
            for name in bench.single_launch_kernels(cfg, **kw):
                assert re.search(r"\b%s\(" % name, kernels), name
