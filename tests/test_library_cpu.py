"""Host-side checks of libcmoe that need no GPU: the library loads, exports every symbol the public
header declares, and its argument checks turn bad input into error codes (never a crash)."""
import os
import re
import subprocess

import numpy as np
import pytest

from paper_2502_04416_amd import binding, synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2502_04416_amd", "csrc")


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(binding.LIB_PATH):
        import __graft_entry__ as g
        g.build()
    return binding.load()


def test_every_declared_symbol_is_exported(lib):
    header = open(os.path.join(ROOT, "include", "cmoe.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(cmoe_[a-z_]+)\s*\(", header))
    assert len(declared) >= 32
    assert declared == set(binding.EXPORTS)
    for name in declared:
        assert hasattr(lib, name), name
    assert "gfx950" in binding.cmoe_version()


def _tiny():
    cfg = synth.scaled(synth.CONFIGS[0], d_model=16, d_ff=32, n_experts=4, n_shared=1, top_k=1)
    return cfg, synth.make_weights(cfg), synth.trivial_partition(cfg)


def test_build_from_partition_roundtrip(lib):
    cfg, w, p = _tiny()
    h = binding.cmoe_build_from_partition(binding.make_config(cfg), *w, p["neuron_order"], p["rep_neuron"])
    e = binding.cmoe_export_partition(h, cfg.d_ff, cfg.n_routed)
    assert np.array_equal(e["neuron_order"], p["neuron_order"]) and np.array_equal(e["rep_neuron"], p["rep_neuron"])
    assert binding.cmoe_packed_bytes(h) > 3 * cfg.d_model * cfg.d_ff * 4
    assert binding.cmoe_workspace_bytes(h, 128) > binding.cmoe_workspace_bytes(h, 1) > 0
    binding.cmoe_destroy(h)


@pytest.mark.parametrize("field,value,msg", [
    ("n_experts", 5, "multiple"),            # d_ff % N != 0
    ("n_shared", 4, "n_shared"),             # N_s >= N
    ("top_k", 4, "top_k"),                   # N_k > N_r
    ("top_k", 0, "top_k"),
    ("dtype", "bad", "dtype"),
])
def test_bad_config_is_rejected(lib, field, value, msg):
    cfg, w, p = _tiny()
    c = binding.make_config(cfg)
    if field == "dtype":
        c.dtype = 7
    else:
        setattr(c, field, value)
    with pytest.raises(binding.CmoeError, match=msg):
        binding.cmoe_build_from_partition(c, *w, p["neuron_order"], p["rep_neuron"])


def test_bad_partition_is_rejected(lib):
    cfg, w, p = _tiny()
    order = p["neuron_order"].copy()
    order[0] = order[1]
    with pytest.raises(binding.CmoeError, match="permutation"):
        binding.cmoe_build_from_partition(binding.make_config(cfg), *w, order, p["rep_neuron"])
    reps = p["rep_neuron"].copy()
    reps[0] = cfg.d_ff
    with pytest.raises(binding.CmoeError, match="rep_neuron"):
        binding.cmoe_build_from_partition(binding.make_config(cfg), *w, p["neuron_order"], reps)


def test_forward_before_upload_is_an_error(lib):
    cfg, w, p = _tiny()
    h = binding.cmoe_build_from_partition(binding.make_config(cfg), *w, p["neuron_order"], p["rep_neuron"])
    with pytest.raises(binding.CmoeError, match="upload"):
        binding.cmoe_forward(h, 1, 1, 1, None, None, None, 1, 1)
    binding.cmoe_destroy(h)


def test_null_handles(lib):
    assert binding.cmoe_packed_bytes(None) == 0
    assert binding.cmoe_workspace_bytes(None, 4) == 0
    with pytest.raises(binding.CmoeError):
        binding.cmoe_set_gate_params(None, None, None)
    binding.cmoe_destroy(None)


def test_generator_rounding_matches_torch():
    """The input generator's bf16 rounding against torch's conversion (a library routine)."""
    import torch
    x = (np.random.default_rng(0).standard_normal(100000) * 3).astype(np.float32)
    assert np.array_equal(synth.round_to_bf16(x), torch.from_numpy(x).bfloat16().float().numpy())


def test_update_bias_matches_the_oracle_on_the_host(lib):
    """cmoe_update_bias is host arithmetic (Sec. 4.3): same result as the oracle's step, fp32 vs fp64."""
    from oracle import cmoe_oracle as O
    cfg = synth.scaled(synth.CONFIGS[0], d_model=16, d_ff=48, n_experts=6, n_shared=1, top_k=2)
    w, p = synth.make_weights(cfg), synth.trivial_partition(cfg)
    h = binding.cmoe_build_from_partition(binding.make_config(cfg), *w, p["neuron_order"], p["rep_neuron"])
    u0 = np.linspace(-0.5, 0.5, cfg.n_routed).astype(np.float32)
    b0 = np.linspace(0.3, -0.3, cfg.n_routed).astype(np.float32)
    binding.cmoe_set_gate_params(h, u0, b0)
    ref = b0.astype(np.float64)
    rng = np.random.Generator(np.random.PCG64(3))
    for _ in range(5):
        counts = rng.integers(0, 50, size=cfg.n_routed)
        binding.cmoe_update_bias(h, counts, 1e-3)
        ref = O.bias_update(ref, counts, 1e-3)
    u, b = binding.cmoe_get_gate_params(h, cfg.n_routed)
    assert np.array_equal(u, u0)
    assert np.abs(b.astype(np.float64) - ref).max() < 1e-6
    binding.cmoe_update_bias(h, np.zeros(cfg.n_routed, dtype=np.int32), 1e-3)        # no routed token: unchanged
    assert np.array_equal(binding.cmoe_get_gate_params(h, cfg.n_routed)[1], b)
    with pytest.raises(binding.CmoeError):
        binding.cmoe_update_bias(h, -np.ones(cfg.n_routed, dtype=np.int32), 1e-3)
    binding.cmoe_destroy(h)


def test_baseline_copy_is_optional(lib):
    """Without the dense baseline the packed weights are about half the size, and the switch is one-way."""
    cfg, w, p = _tiny()
    h = binding.cmoe_build_from_partition(binding.make_config(cfg), *w, p["neuron_order"], p["rep_neuron"])
    both = binding.cmoe_packed_bytes(h)
    binding.cmoe_set_baseline(h, False)
    moe_only = binding.cmoe_packed_bytes(h)
    assert moe_only < both and both - moe_only >= 3 * cfg.d_model * cfg.d_ff * 4
    with pytest.raises(binding.CmoeError, match="released"):
        binding.cmoe_set_baseline(h, True)
    binding.cmoe_destroy(h)


def test_tuning_switches(lib):
    binding.cmoe_set_tuning("CMOE_SPLITK", 0)
    binding.cmoe_set_tuning("CMOE_SPLITK", 1)
    binding.cmoe_set_tuning("CMOE_GEMM1_CFG", -1)
    with pytest.raises(binding.CmoeError, match="unknown"):
        binding.cmoe_set_tuning("CMOE_NO_SUCH_SWITCH", 1)


def test_non_finite_calibration_tokens_are_rejected(lib):
    cfg = synth.scaled(synth.CONFIGS[0], d_model=16, d_ff=32, n_experts=4, n_shared=1, top_k=1, k_act=3)
    w = synth.make_weights(cfg)
    x = synth.make_token_source(cfg).calibration(n=40).copy()
    x[17, 3] = np.nan
    with pytest.raises(binding.CmoeError, match="token 17"):
        binding.cmoe_build(binding.make_config(cfg), *w, x)
    with pytest.raises(binding.CmoeError, match="token 17"):
        binding.cmoe_profile_activations(binding.make_config(cfg), w[0], w[1], x, on_gpu=False)
    x[17, 3] = np.inf
    with pytest.raises(binding.CmoeError, match="token 17"):
        binding.cmoe_build(binding.make_config(cfg), *w, x)


def test_bench_refuses_more_than_one_gpu():
    """This build runs on one GPU: the bench says so and exits instead of launching ranks."""
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 2
    assert "ONE GPU" in r.stderr and r.stdout.strip() == ""


def test_lds_limit_is_raised_on_every_device(tmp_path):
    """The limit of dynamic LDS belongs to a kernel's copy on one device: the first launch on each raises it, one that failed is
    tried again, and host threads may race for it.  (The two runtime calls are stand-ins that record.)"""
    src = tmp_path / "limit.cpp"
    src.write_text(r'''
#include "lds_limit.h"
#include <cassert>
#include <thread>
#include <vector>
static thread_local int device = 0;
static std::atomic<int> calls[80];
static std::atomic<bool> refuse{false};
extern "C" hipError_t hipGetDevice(int* d) { *d = device; return hipSuccess; }
extern "C" hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) {
  ++calls[device];
  return refuse ? hipErrorInvalidValue : hipSuccess;
}
int main() {
  cmoe::LdsLimit a, b;
  int kernel = 0;
  for (int rep = 0; rep < 3; ++rep)
    for (device = 0; device < 70; ++device) assert(a.raise(&kernel, 100000) == hipSuccess);
  for (int d = 0; d < 70; ++d) assert(calls[d] == (d < 64 ? 1 : 3));
  device = 5;
  refuse = true;
  assert(b.raise(&kernel, 100000) != hipSuccess && calls[5] == 2);
  refuse = false;
  assert(b.raise(&kernel, 100000) == hipSuccess && b.raise(&kernel, 100000) == hipSuccess && calls[5] == 3);
  cmoe::LdsLimit c;
  std::vector<std::thread> threads;
  for (int i = 0; i < 16; ++i)
    threads.emplace_back([&, i] { device = i % 4 + 72; c.raise(&kernel, 1); device = i % 4; for (int k = 0; k < 100; ++k) c.raise(&kernel, 1); });
  for (auto& t : threads) t.join();
  for (int d = 0; d < 4; ++d) assert(calls[d] >= 2 && calls[d] <= 5);
  return 0;
}
''')
    exe = tmp_path / "limit"
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC, str(src), "-o", str(exe),
                    "-lpthread"], check=True)
    subprocess.run([str(exe)], check=True)
    callers = {f for f in os.listdir(CSRC) if "hipFuncSetAttribute" in open(os.path.join(CSRC, f)).read()}
    assert callers == {"lds_limit.h", "profile.hip"}             # (the latter sets it before its launch every time)


def test_forward_plan(lib):
    """The query names the kernels of a batch on the host, and follows the switches."""
    cfg = synth.scaled(synth.CONFIGS[1], d_model=512, d_ff=8 * 100, n_experts=8, n_shared=1, top_k=2)
    part = synth.trivial_partition(cfg)
    layer = binding.Layer.from_partition(cfg, *synth.make_weights(cfg), part["neuron_order"], part["rep_neuron"], upload=False)
    try:
        assert layer.forward_plan(1)["down"] == ("combines", 16)
        binding.cmoe_set_tuning("CMOE_GEMM1_CFG", 6)
        for shape, plan in ((8, ("tiles", 8)), (22, ("persistent", 1))):
            binding.cmoe_set_tuning("CMOE_GEMM2_CFG", shape)
            assert layer.forward_plan(300) == {"gate_up": ("tiles", 6), "down": plan}
            assert layer.forward_plan(300, dense=True)["down"][0] == "tiles"      # (no work list: a forced 22 is refused)
    finally:
        binding.cmoe_set_tuning("CMOE_GEMM1_CFG", -1)
        binding.cmoe_set_tuning("CMOE_GEMM2_CFG", -1)
    with pytest.raises(binding.CmoeError):
        layer.forward_plan(0)
    layer.close()


def test_large_slot_outputs_stay_in_the_caches(lib):
    """The persistent down contraction stores past the caches up to 45 MB of slot outputs, and beyond 380 MB."""
    cfg = synth.scaled(synth.CONFIGS[1], d_model=512, d_ff=8 * 100, n_experts=8, n_shared=1, top_k=2)
    part = synth.trivial_partition(cfg)
    layer = binding.Layer.from_partition(cfg, *synth.make_weights(cfg), part["neuron_order"], part["rep_neuron"], upload=False)
    limit = (45 << 20) // (3 * 512 * 2)
    try:
        binding.cmoe_set_tuning("CMOE_GEMM2_CFG", 22)
        assert layer.forward_plan(limit)["down"] == ("persistent", 1)
        assert layer.forward_plan(limit + 1)["down"] == ("persistent", 0)
        limit = (380 << 20) // (3 * 512 * 2)
        assert layer.forward_plan(limit)["down"] == ("persistent", 0)
        assert layer.forward_plan(limit + 1)["down"] == ("persistent", 1)
    finally:
        binding.cmoe_set_tuning("CMOE_GEMM2_CFG", -1)
    layer.close()


@pytest.mark.parametrize("d,d_ff,T,dense,gate_up,down", [
    (256, 1024, 64, True, 16, 16),
    (256, 1024, 4096, True, 64, 16),      # the gate/up contraction fills the chip with large tiles long before the down does
    (256, 1024, 8192, True, 64, 64),
    (64, 1024, 16384, True, 64, 16),
    (1024, 4096, 2048, True, 64, 64),
    (64, 8192, 4096, False, 64, 16),
    (512, 1536, 64, False, 16, 16),
])
def test_fp32_tiles_chosen_per_contraction(lib, d, d_ff, T, dense, gate_up, down):
    cfg = synth.scaled(synth.CONFIGS[0], d_model=d, d_ff=d_ff, n_experts=8, n_shared=2, top_k=2)
    part = synth.trivial_partition(cfg)
    layer = binding.Layer.from_partition(cfg, *synth.make_weights(cfg), part["neuron_order"], part["rep_neuron"], upload=False)
    assert layer.forward_plan(T, dense) == {"gate_up": ("fma", gate_up), "down": ("fma", down)}
    layer.close()


@pytest.mark.parametrize("d,n,n_s,k,T,streamed", [
    (2048, 12, 1, 2, 64, True),           # routed entries per expert times d: 23831
    (4096, 16, 1, 3, 32, True),           # 26214, units of 16 neurons
    (4096, 16, 1, 3, 33, False),          # 27034
    (5632, 16, 1, 2, 31, True),           # 23279, units of 8
    (5632, 16, 1, 2, 32, False),          # 24030
    (4096, 32, 0, 5, 24, True),           # 15360, no always-on group
    (4096, 16, 0, 4, 17, False),          # 17408
    (3072, 16, 0, 3, 46, True),           # 26496, narrow enough for the common line
])
def test_streamed_units_where_they_win(lib, d, n, n_s, k, T, streamed):
    cfg = synth.scaled(synth.CONFIGS[1], d_model=d, d_ff=n * 32, n_experts=n, n_shared=n_s, top_k=k)
    part = synth.trivial_partition(cfg)
    layer = binding.Layer.from_partition(cfg, *synth.make_weights(cfg), part["neuron_order"], part["rep_neuron"], upload=False)
    assert (layer.forward_plan(T)["gate_up"][0] == "streamed") == streamed
    layer.close()


@pytest.mark.parametrize("d,n,m,n_s,k,T,down", [
    (2048, 8, 692, 1, 2, 2048, ("tiles", 0)),         # one round of tall tiles of one depth
    (2048, 8, 692, 0, 2, 3000, ("tiles", 0)),
    (2048, 8, 692, 2, 2, 2048, ("persistent", 1)),    # ... with an always-on group twice as deep
    (2048, 12, 320, 1, 2, 1400, ("tiles", 0)),
    (2048, 16, 256, 1, 3, 1400, ("persistent", 1)),   # K too short for tall tiles
    (2048, 32, 192, 2, 6, 400, ("tiles", 21)),
    (2048, 8, 692, 1, 2, 3000, ("persistent", 1)),
])
def test_persistent_down_contraction_where_it_wins(lib, d, n, m, n_s, k, T, down):
    cfg = synth.scaled(synth.CONFIGS[1], d_model=d, d_ff=n * m, n_experts=n, n_shared=n_s, top_k=k)
    part = synth.trivial_partition(cfg)
    layer = binding.Layer.from_partition(cfg, *synth.make_weights(cfg), part["neuron_order"], part["rep_neuron"], upload=False)
    assert layer.forward_plan(T)["down"] == down
    layer.close()


@pytest.mark.parametrize("d,n_s,T,kernel", [
    (512, 1, 8, "units"), (2048, 1, 16, "units"), (2560, 2, 4, "units"),      # too narrow for a stream
    (3072, 2, 4, "streamed"), (4096, 1, 2, "streamed"), (4096, 0, 2, "units"), (4096, 0, 4, "streamed"), (5120, 0, 2, "streamed"),
])
def test_decode_batches_stream_where_it_wins(lib, d, n_s, T, kernel):
    cfg = synth.scaled(synth.CONFIGS[1], d_model=d, d_ff=16 * 32, n_experts=16, n_shared=n_s, top_k=3)
    part = synth.trivial_partition(cfg)
    layer = binding.Layer.from_partition(cfg, *synth.make_weights(cfg), part["neuron_order"], part["rep_neuron"], upload=False)
    assert layer.forward_plan(T)["gate_up"][0] == kernel
    try:                                                                      # a forced shape counts at every width
        binding.cmoe_set_tuning("CMOE_GEMM1_CFG", 24)
        assert layer.forward_plan(T)["gate_up"][0] == "streamed"
    finally:
        binding.cmoe_set_tuning("CMOE_GEMM1_CFG", -1)
    layer.close()


@pytest.mark.parametrize("d,n,m,n_s,k,T,down", [
    (3072, 16, 704, 0, 4, 64, "tiles"),        # 16 rows per row of weights, 320398 against 312640
    (3072, 16, 704, 0, 4, 62, "combines"),
    (4096, 16, 704, 0, 4, 64, "combines"),     # a wider layer, more workgroups: 180224
    (3072, 16, 96, 0, 4, 64, "combines"),      # narrow experts
    (4096, 4, 96, 1, 2, 40, "tiles"),          # 30 rows per row of weights
])
def test_down_and_combine_where_it_wins(lib, d, n, m, n_s, k, T, down):
    """The fused down + combine launch beyond 32 tokens: hidden activations per workgroup against rows of weights."""
    cfg = synth.scaled(synth.CONFIGS[1], d_model=d, d_ff=n * m, n_experts=n, n_shared=n_s, top_k=k)
    part = synth.trivial_partition(cfg)
    zeros = np.zeros((d, n * m), dtype=np.float32)
    layer = binding.Layer.from_partition(cfg, zeros, zeros, zeros.T, part["neuron_order"], part["rep_neuron"], upload=False)
    assert layer.forward_plan(T)["down"][0] == down
    layer.close()


def test_down_and_combine_of_a_dense_hierarchy(lib):
    """Whole experts, two of eight per token: a quarter of the weights' rows per token, 3072 wide."""
    cfg = synth.scaled(synth.CONFIGS[4], d_model=3072, d_ff=8 * 192, n_experts=8, n_shared=2, top_k=2, n_outer=8, outer_top_k=2)
    part = synth.trivial_partition(cfg)
    zeros = np.zeros((cfg.d_model, cfg.d_ff), dtype=np.float32)
    layers = [binding.Layer.from_partition(cfg, zeros, zeros, zeros.T, part["neuron_order"], part["rep_neuron"], upload=False)
              for _ in range(cfg.n_outer)]
    h = binding.cmoe_hier_create([l.h for l in layers], cfg.outer_top_k, np.zeros((cfg.d_model, cfg.n_outer)), None)
    assert binding.cmoe_forward_plan(h, 33, dense=True, hier=True)["down"][0] == "combines"
    assert binding.cmoe_forward_plan(h, 64, dense=True, hier=True)["down"][0] == "tiles"
    assert binding.cmoe_forward_plan(h, 64, hier=True)["down"][0] == "combines"
    binding.cmoe_hier_destroy(h)
    for l in layers:
        l.close()
