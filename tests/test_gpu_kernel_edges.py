"""GPU parity of the tile shapes, routing kernels and decode kernels at the sizes where their indexing can go wrong,
against the CPU oracle (tolerances of parity_utils: 1e-2 for bf16, indices exact)."""
import numpy as np
import pytest

from paper_2502_04416_amd import synth
from parity_utils import check_dense, check_flat
from test_gpu_hier import _check, _make

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def binding():
    from paper_2502_04416_amd import binding as b
    b.load()
    return b


def _case(binding, d, N, m, n_s, k, T, seed=0, **kw):
    cfg = synth.scaled(synth.CONFIGS[1], d_model=d, d_ff=N * m, n_experts=N, n_shared=n_s, top_k=k, n_centres=16)
    weights = synth.make_weights(cfg, seed=3100 + seed)
    part = synth.trivial_partition(cfg, seed=seed)
    x = synth.make_token_source(cfg).eval_batch(seed, n=T)
    layer = binding.Layer.from_partition(cfg, *weights, part["neuron_order"], part["rep_neuron"], **kw)
    return cfg, weights, part, x, layer


@pytest.mark.parametrize("which", ["CMOE_GEMM1_CFG", "CMOE_GEMM2_CFG"])
@pytest.mark.parametrize("shape", [0, 6, 9, 19, 20, 21])
@pytest.mark.parametrize("d,m,T", [(328, 100, 333), (40, 32, 300), (64, 48, 257), (96, 20, 161)])
def test_deep_ring_shapes(binding, which, shape, d, m, T):
    """The deep-ring tile shapes on K loops shorter than the ring (d = 40: two steps, the second ragged; width 32: one
    step), of odd and even length, with row tiles, column tiles and 16-row blocks that end inside."""
    cfg, weights, part, x, layer = _case(binding, d, 12, m, 2, 3, T)
    try:
        binding.cmoe_set_tuning("CMOE_SPLITK", 0)
        ref = layer.forward(x)
        binding.cmoe_set_tuning(which, shape)
        out, dense = layer.forward(x), layer.dense_forward(x)
    finally:
        binding.cmoe_set_tuning("CMOE_SPLITK", 1)
        binding.cmoe_set_tuning(which, -1)
    check_flat(cfg, weights, part, x, out)
    check_dense(cfg, weights, x, dense)
    assert np.array_equal(out["y"], ref["y"])          # K in the same order: the shape changes no bit
    layer.close()


@pytest.mark.parametrize("which", ["CMOE_GEMM1_CFG", "CMOE_GEMM2_CFG"])
@pytest.mark.parametrize("shape", [0, 6, 20, 21])
def test_deep_ring_k_split(binding, which, shape):
    """Partial sums of a K split whose last part is short: d = 1056 for gate/up (33 steps: parts of 9, the last of 6), the
    dense layer's d_ff = 1088 for down (34: of 9, the last of 7)."""
    cfg, weights, part, x, layer = _case(binding, 1056, 8, 136, 1, 2, 90)
    flat, dense = {}, {}
    try:
        for split in (0, 1):
            binding.cmoe_set_tuning("CMOE_SPLITK", split)
            binding.cmoe_set_tuning(which, shape)
            flat[split], dense[split] = layer.forward(x), layer.dense_forward(x)
            binding.cmoe_set_tuning(which, -1)
    finally:
        binding.cmoe_set_tuning("CMOE_SPLITK", 1)
        binding.cmoe_set_tuning(which, -1)
    check_flat(cfg, weights, part, x, flat[1])
    check_dense(cfg, weights, x, dense[1])
    assert not np.array_equal(dense[0], dense[1])       # another order of the same sum
    layer.close()


def test_gather_across_two_gigabytes(binding):
    """A batch whose rows lie 2 GB and more apart: 64-bit row addresses in the gate/up contraction.  Tokens from its
    beginning, middle and end against the oracle; the same tokens in two smaller batches, and with a forced shape of
    either kind (a ring shape without such addresses gives way to the one that has them), give the same bits."""
    import torch
    T, d = 262144 + 77, 4096
    cfg = synth.scaled(synth.CONFIGS[1], d_model=d, d_ff=8 * 32, n_experts=8, n_shared=1, top_k=1, n_centres=16)
    part, weights = synth.trivial_partition(cfg), synth.make_weights(cfg)
    layer = binding.Layer.from_partition(cfg, *weights, part["neuron_order"], part["rep_neuron"])
    x = torch.randn((T, d), generator=torch.Generator(device="cuda").manual_seed(5), device="cuda", dtype=torch.bfloat16)
    y, half, y2 = torch.empty_like(x), 131072, torch.empty_like(x)
    topk = torch.empty((T, 1), dtype=torch.int32, device="cuda")
    scores = torch.empty((T, 7), dtype=torch.float32, device="cuda")
    layer.forward_device(x, y, topk=topk, scores=scores)
    idx = torch.cat([torch.arange(t, t + 40) for t in (0, half - 20, 262144 - 20, T - 40)]).cuda()
    out = {"y": y[idx].float().cpu().numpy(), "topk": topk[idx].cpu().numpy(), "scores": scores[idx].cpu().numpy()}
    out["counts"] = np.bincount(out["topk"].ravel(), minlength=7)
    check_flat(cfg, weights, part, x[idx].float().cpu().numpy(), out)
    # (a multiple of 16384 tokens per piece keeps the router's K slices, hence its scores, those of the whole batch)
    for lo, hi in ((0, half), (half, T)):
        layer.forward_device(x[lo:hi], y2[lo:hi])
    assert torch.equal(y, y2)
    try:
        for shape in (4, 9):
            binding.cmoe_set_tuning("CMOE_GEMM1_CFG", shape)
            y2.zero_()
            layer.forward_device(x, y2)
            assert torch.equal(y, y2)
    finally:
        binding.cmoe_set_tuning("CMOE_GEMM1_CFG", -1)
    layer.close()


@pytest.mark.parametrize("gate", [False, True])
@pytest.mark.parametrize("d,N,n_s,k,T", [
    (512, 16, 1, 3, 65),        # two K slices of one chunk, 32 tokens per workgroup
    (512, 40, 2, 5, 97),        # more than 32 routed experts: two groups of 64 router rows
    (768, 12, 0, 1, 79),        # three slices: the two launches
    (1536, 12, 1, 4, 130),      # six slices: three units per wave, the last waves short
    (2048, 65, 1, 16, 200),     # 64 routed experts, top-16: eight slices of one chunk
    (2560, 16, 1, 3, 71),       # five slices of two chunks
    (4096, 8, 1, 7, 2081),      # eight slices of two chunks, every routed expert chosen
    (512, 8, 2, 2, 8300),       # two slices of one chunk, 32 tokens per workgroup
    (1024, 8, 1, 2, 8300),      # two slices of two chunks
    (512, 8, 1, 2, 16500),      # one slice of two chunks
])
def test_scoring_and_selection_in_one_launch(binding, d, N, n_s, k, T, gate):
    """Prefill batches of a flat layer: K slices, units per wave, token blocks and histogram rows of every kind."""
    cfg, weights, part, x, layer = _case(binding, d, N, 16, n_s, k, T, seed=1)
    u = b = None
    if gate:
        u, b = synth.make_gate_params(cfg, seed=7300)
        layer.set_gate_params(u, b)
    out = layer.forward(x)
    check_flat(cfg, weights, part, x, out, u=u, b=b)
    counts = np.bincount(out["topk"].ravel(), minlength=cfg.n_routed)
    assert np.array_equal(out["counts"], counts)
    layer.close()


@pytest.mark.parametrize("gate", [False, True])
@pytest.mark.parametrize("d,T", [(512, 1), (512, 2), (512, 20), (512, 64), (512, 65), (512, 200), (768, 200)])
def test_non_finite_tokens_stay_in_their_rows(binding, d, T, gate):
    """A token of NaNs or infinities has no meaningful choice of experts, but it gets valid ones, and the other tokens of
    the batch keep their outputs.  (One token, one tile, scoring and selection in one launch, and in two: d = 768.)"""
    cfg, weights, part, x, layer = _case(binding, d, 16, 32, 1, 3, T, seed=2)
    if gate:
        layer.set_gate_params(*synth.make_gate_params(cfg, seed=7300))
    ref = layer.forward(x)
    bad = x.copy()
    bad[0] = np.nan
    if T > 2:
        bad[1] = np.inf
    out = layer.forward(bad)
    assert ((out["topk"] >= 0) & (out["topk"] < cfg.n_routed)).all()
    assert all(len(set(row)) == cfg.top_k for row in out["topk"].tolist())
    n_bad = 2 if T > 2 else 1
    if T > n_bad:
        assert np.array_equal(out["topk"][n_bad:], ref["topk"][n_bad:])
        assert np.array_equal(out["y"][n_bad:], ref["y"][n_bad:])
    layer.close()


@pytest.mark.parametrize("T", [1, 2, 40, 130])
def test_non_finite_tokens_in_a_hierarchy(binding, T):
    cfg = synth.scaled(synth.CONFIGS[4], d_model=512, d_ff=8 * 40, n_experts=8, n_shared=2, top_k=2, n_outer=4,
                       outer_top_k=2, n_centres=16)
    hier, _, _, _ = _make(binding, cfg, gate=True)
    x = synth.make_token_source(cfg).eval_batch(7, n=T)
    ref = hier.forward(x)
    bad = x.copy()
    bad[0] = np.nan
    out = hier.forward(bad)
    assert all(len(set(row)) == 2 for row in out["outer"].tolist())
    assert ((out["outer"] >= 0) & (out["outer"] < 4)).all() and ((out["sub"] >= 0) & (out["sub"] < 6)).all()
    assert all(len(set(row)) == 2 for row in out["sub"].reshape(-1, 2).tolist())
    if T > 1:
        assert np.array_equal(out["outer"][1:], ref["outer"][1:]) and np.array_equal(out["sub"][1:], ref["sub"][1:])
        assert np.array_equal(out["y"][1:], ref["y"][1:])
    hier.close()


@pytest.mark.parametrize("d", [1536, 2560, 3584, 5120, 8192])
@pytest.mark.parametrize("T,m", [(1, 40), (1, 96), (3, 40), (16, 40)])
def test_decode_kernels_at_other_widths(binding, d, T, m):
    """Model widths whose K slice per wave is not 2, 4, 8 or 16 steps, or two runs of them."""
    cfg, weights, part, x, layer = _case(binding, d, 8, m, 1, 2, T, seed=3)
    out = layer.forward(x)
    check_flat(cfg, weights, part, x, out)
    check_dense(cfg, weights, x, layer.dense_forward(x))
    assert np.array_equal(out["y"], layer.forward(x)["y"])
    layer.close()


@pytest.mark.parametrize("d", list(range(512, 4097, 512)) + [5120, 6144, 7680, 8192, 10240])
def test_every_decode_width(binding, d):
    """Every model width that the weight-streaming kernels serve; the widths above 4096, whose K slice takes several runs,
    up to four tokens (five choose between streamed units and tiles: both)."""
    for T in (1, 4, 5):
        cfg, weights, part, x, layer = _case(binding, d, 8, 40, 1, 2, T, seed=4)
        out = layer.forward(x)
        check_flat(cfg, weights, part, x, out)
        check_dense(cfg, weights, x, layer.dense_forward(x))
        if d > 4096 and T == 5:
            try:
                for shape, kernel in ((7, "tiles"), (24, "streamed")):
                    binding.cmoe_set_tuning("CMOE_GEMM1_CFG", shape)
                    assert layer.forward_plan(T)["gate_up"][0] == kernel
                    check_flat(cfg, weights, part, x, layer.forward(x))
            finally:
                binding.cmoe_set_tuning("CMOE_GEMM1_CFG", -1)
        layer.close()


@pytest.mark.parametrize("d", [1536, 5120, 6144, 7680, 8192, 10240])
def test_hierarchy_at_decode_widths(binding, d):
    """The same for a hierarchy: its router has SwiGLU and linear rows, and the selection a launch of its own."""
    cfg = synth.scaled(synth.CONFIGS[4], d_model=d, d_ff=8 * 40, n_experts=8, n_shared=2, top_k=2, n_outer=4,
                       outer_top_k=2, n_centres=16)
    hier, experts, w_router, offsets = _make(binding, cfg)
    for T in (1, 4):
        x = synth.make_token_source(cfg).eval_batch(6, n=T)
        _check(cfg, experts, w_router, offsets, x, hier.forward(x), hier.dense_forward(x), np.arange(T))
    hier.close()


@pytest.mark.parametrize("gate", [False, True])
@pytest.mark.parametrize("N,n_s,k", [(40, 1, 9), (40, 1, 10), (13, 0, 1), (13, 1, 1), (65, 1, 16), (33, 1, 6), (33, 1, 7)])
@pytest.mark.parametrize("T", [1, 3, 20, 64, 130])
def test_selection_by_rounds_and_by_rank(binding, N, n_s, k, T, gate):
    """Both sides of the line between the two selections of a tile (160 top_k against the square of the routed experts),
    and one token; equal scores go to the lower expert either way."""
    cfg, weights, part, x, layer = _case(binding, 512, N, 8, n_s, k, T, seed=5)
    layer.close()
    reps = part["rep_neuron"].copy()
    reps[7] = reps[2]                                   # routed experts 2 and 7 share their representative
    part = dict(part, rep_neuron=reps)
    layer = binding.Layer.from_partition(cfg, *weights, part["neuron_order"], reps)
    u = b = None
    if gate:
        u, b = synth.make_gate_params(cfg, seed=7300)
        b[7] = b[2]
        layer.set_gate_params(u, b)
    check_flat(cfg, weights, part, x, layer.forward(x), u=u, b=b, exact_ties_strict=True)
    layer.close()


@pytest.mark.parametrize("remap", [1, 0])
@pytest.mark.parametrize("d,N,m,n_s,k,T", [
    (328, 12, 100, 2, 3, 333),     # K of 7 and 4 steps, column tiles and 16-row blocks that end inside
    (40, 12, 96, 0, 4, 1000),      # K as short as the ring is deep, no deep tiles, fewer columns than a wave has
    (1024, 8, 160, 3, 2, 700),     # 15 and 5 steps, deep tiles that do not divide among the workgroups of a die
    (512, 66, 97, 2, 5, 2100),     # more than 64 groups, rows that fill a tile to the last
])
def test_persistent_down_contraction(binding, d, N, m, n_s, k, T, remap):
    """The persistent down kernel against the oracle, and bit for bit against a workgroup per tile."""
    cfg, weights, part, x, layer = _case(binding, d, N, m, n_s, k, T)
    try:
        binding.cmoe_set_tuning("CMOE_SPLITK", 0)
        binding.cmoe_set_tuning("CMOE_XCD_REMAP", remap)
        binding.cmoe_set_tuning("CMOE_GEMM2_CFG", 8)
        assert layer.forward_plan(T)["down"] == ("tiles", 8)
        ref = layer.forward(x)
        binding.cmoe_set_tuning("CMOE_GEMM2_CFG", 22)
        assert layer.forward_plan(T)["down"] == ("persistent", 1)
        out = layer.forward(x)
    finally:
        binding.cmoe_set_tuning("CMOE_GEMM2_CFG", -1)
        binding.cmoe_set_tuning("CMOE_XCD_REMAP", 1)
        binding.cmoe_set_tuning("CMOE_SPLITK", 1)
    check_flat(cfg, weights, part, x, out)
    assert np.array_equal(out["y"], ref["y"])
    layer.close()


@pytest.mark.parametrize("T,past_caches", [(38000, 1), (2100, 0)])
def test_persistent_down_contraction_many_tiles(binding, T, past_caches):
    """More tiles per workgroup (65) than it looks up at a time; few, with results that go through the caches."""
    import torch
    cfg = synth.scaled(synth.CONFIGS[1], d_model=4096, d_ff=8 * 96, n_experts=8, n_shared=1, top_k=6, n_centres=16)
    part, weights = synth.trivial_partition(cfg), synth.make_weights(cfg)
    layer = binding.Layer.from_partition(cfg, *weights, part["neuron_order"], part["rep_neuron"])
    x = torch.randn((T, 4096), generator=torch.Generator(device="cuda").manual_seed(5), device="cuda", dtype=torch.bfloat16)
    y = {}
    try:
        for shape, plan in ((8, ("tiles", 8)), (22, ("persistent", past_caches))):
            binding.cmoe_set_tuning("CMOE_GEMM2_CFG", shape)
            assert layer.forward_plan(T)["down"] == plan
            y[shape] = torch.empty_like(x)
            layer.forward_device(x, y[shape])
    finally:
        binding.cmoe_set_tuning("CMOE_GEMM2_CFG", -1)
    assert torch.equal(y[8], y[22])
    layer.close()


@pytest.mark.parametrize("d,N,m,n_s,k,T", [
    (70, 4, 9, 0, 1, 1),           # rows that are not whole float4s, K ragged in every wave, widths padded to 32
    (64, 8, 40, 1, 2, 17),         # fewer chunks of K than waves; one row past a tile
    (328, 12, 50, 2, 3, 100),      # K = 20.5 chunks, columns that end inside a tile
    (640, 8, 136, 1, 1, 48),       # K of more than one batch of loads
    (512, 12, 64, 1, 2, 1024),     # as many entries as the placement counts by itself, over several tiles of tokens
    (512, 12, 64, 1, 2, 1025),     # one token more: the histogram of a launch of its own
    (512, 12, 64, 1, 3, 1500),     # batches of the large tiles
])
def test_fp32_tiles(binding, d, N, m, n_s, k, T):
    """The fp32 contraction kernels and the scorer at their edges, with and without aligned rows of x."""
    import torch
    cfg = synth.scaled(synth.CONFIGS[0], d_model=d, d_ff=N * m, n_experts=N, n_shared=n_s, top_k=k, n_centres=16)
    weights = synth.make_weights(cfg, seed=3300)
    part = synth.trivial_partition(cfg, seed=1)
    x = synth.make_token_source(cfg).eval_batch(1, n=T)
    layer = binding.Layer.from_partition(cfg, *weights, part["neuron_order"], part["rep_neuron"])
    out = layer.forward(x)
    check_flat(cfg, weights, part, x, out)
    check_dense(cfg, weights, x, layer.dense_forward(x))
    buf = torch.empty(T * d + 1, device="cuda")
    xu = buf[1:].view(T, d).copy_(torch.from_numpy(x))           # rows that start 4 bytes past a 16-byte boundary
    y = torch.empty((T, d), device="cuda")
    layer.forward_device(xu, y)
    assert np.array_equal(y.cpu().numpy(), out["y"])             # the same sums in the same order
    try:                                                         # either kernel for either contraction, whatever the rule takes
        for rows in ((16, 64), (64, 16), (16, 16), (64, 64)):
            binding.cmoe_set_tuning("CMOE_F32_ROWS1", rows[0])
            binding.cmoe_set_tuning("CMOE_F32_ROWS2", rows[1])
            assert layer.forward_plan(T) == {"gate_up": ("fma", rows[0]), "down": ("fma", rows[1])}
            check_flat(cfg, weights, part, x, layer.forward(x))
            check_dense(cfg, weights, x, layer.dense_forward(x))
    finally:
        binding.cmoe_set_tuning("CMOE_F32_ROWS1", -1)
        binding.cmoe_set_tuning("CMOE_F32_ROWS2", -1)
    layer.close()


@pytest.mark.parametrize("d,N,m,n_s,k,T", [
    (512, 8, 100, 1, 2, 2),        # one chunk of K per wave, padded widths, two tokens
    (2560, 8, 64, 1, 2, 16),       # an odd number of chunks; a full token tile
    (1024, 8, 64, 1, 2, 16),       # one chunk of four steps
    (1024, 8, 64, 1, 2, 40),       # ... of four or two with four token tiles
    (1024, 8, 64, 0, 3, 17),       # two chunks of two, no always-on group, one row past a token tile
    (1536, 6, 50, 2, 1, 33),       # three chunks of two; four token tiles, the third with one row
    (2048, 4, 96, 1, 3, 64),       # the largest batch, routed groups of two to four token tiles
    (5632, 8, 40, 1, 2, 5),        # a width without decode kernels
    (8192, 8, 32, 1, 2, 12),       # a width of several runs, past the decode kernels' four tokens
    (4096, 66, 32, 2, 4, 3),       # more than 64 groups
])
def test_streamed_gate_up(binding, d, N, m, n_s, k, T):
    """The streamed gate/up units, with the always-on group inside the selection launch and in the list, in both sizes and
    where the batch's rule takes them or not, against the oracle; all of them bit for bit."""
    cfg, weights, part, x, layer = _case(binding, d, N, m, n_s, k, T)
    outs = []
    try:
        for shared in (1, 0):
            for split, shape in ((16, 23), (8, 24)):
                binding.cmoe_set_tuning("CMOE_FRONT_SHARED", shared)
                binding.cmoe_set_tuning("CMOE_DECODE_SPLIT", split)
                binding.cmoe_set_tuning("CMOE_GEMM1_CFG", shape)
                assert layer.forward_plan(T)["gate_up"] == ("streamed", split)
                outs.append(layer.forward(x))
    finally:
        for name, value in (("CMOE_FRONT_SHARED", 1), ("CMOE_DECODE_SPLIT", -1), ("CMOE_GEMM1_CFG", -1)):
            binding.cmoe_set_tuning(name, value)
    check_flat(cfg, weights, part, x, outs[0])
    check_flat(cfg, weights, part, x, layer.forward(x))
    assert all(np.array_equal(o["y"], outs[0]["y"]) for o in outs)
    layer.close()


@pytest.mark.parametrize("gate", [False, True])
@pytest.mark.parametrize("d,N,n_s,k,T", [
    (768, 17, 1, 3, 65),        # 16 routed experts: two of four row blocks; three slices
    (768, 17, 0, 3, 65),        # 17: all four
    (1024, 17, 1, 16, 70),      # four slices of one chunk
    (2048, 16, 0, 3, 2400),     # four slices of two chunks
    (2560, 8, 1, 2, 2600),      # two slices of five chunks: the two launches
    (512, 9, 1, 2, 8300),       # two slices, 32 tokens per workgroup
])
def test_router_row_blocks_in_use(binding, d, N, n_s, k, T, gate):
    """Scoring and selection in one launch on either side of 16 routed experts, and batches of three and four K slices."""
    cfg, weights, part, x, layer = _case(binding, d, N, 16, n_s, k, T, seed=2)
    u = b = None
    if gate:
        u, b = synth.make_gate_params(cfg, seed=7300)
        layer.set_gate_params(u, b)
    out = layer.forward(x)
    check_flat(cfg, weights, part, x, out, u=u, b=b)
    assert np.array_equal(out["counts"], np.bincount(out["topk"].ravel(), minlength=cfg.n_routed))
    layer.close()


@pytest.mark.parametrize("d,N,n_s,k,T", [
    (512, 17, 1, 3, 1),         # two K steps per slice: two of the four waves; 16 routed experts: two of four row blocks
    (512, 18, 1, 3, 16),        # 17: all four
    (512, 50, 1, 3, 17),        # 49: six of eight
    (768, 12, 1, 2, 33),        # three steps, a third block of tokens with one token
    (2304, 12, 0, 2, 64),       # nine steps: waves of three, the last none
    (4352, 8, 1, 2, 18),        # seventeen: waves of five, in two runs
    (10240, 8, 1, 2, 3),        # forty: waves of ten, in runs of eight and two
])
def test_small_batch_scorer(binding, d, N, n_s, k, T):
    """The scorer of at most 64 tokens: K steps over waves and runs, row blocks in use, blocks of 16 tokens."""
    cfg, weights, part, x, layer = _case(binding, d, N, 16, n_s, k, T, seed=6)
    check_flat(cfg, weights, part, x, layer.forward(x))
    layer.close()


@pytest.mark.parametrize("dtype,N,m,n_s,k,T", [
    ("bf16", 65, 16, 1, 16, 3),       # 65 groups: the last one alone in the second half of the lookup
    ("bf16", 64, 16, 0, 9, 12),       # 64: the first half full
    ("bf16", 65, 40, 1, 12, 21),      # fused down contraction with two token tiles, widths that end inside an item
    ("bf16", 65, 40, 1, 3, 70),       # low tiles
    ("fp32", 65, 16, 1, 2, 40),
])
def test_work_items_of_many_groups(binding, dtype, N, m, n_s, k, T):
    """The group of a work item, looked up for all groups at once: at most 64 groups, and more."""
    cfg = synth.scaled(synth.CONFIGS[0 if dtype == "fp32" else 1], d_model=512, d_ff=N * m, n_experts=N, n_shared=n_s, top_k=k, n_centres=16)
    weights, part = synth.make_weights(cfg, seed=3107), synth.trivial_partition(cfg, seed=7)
    x = synth.make_token_source(cfg).eval_batch(7, n=T)
    layer = binding.Layer.from_partition(cfg, *weights, part["neuron_order"], part["rep_neuron"])
    check_flat(cfg, weights, part, x, layer.forward(x))
    layer.close()


@pytest.mark.parametrize("d,N,m,n_s,k,T,kernel", [
    (3072, 8, 40, 1, 2, 33, "combines"),      # a third token tile of one row; two K steps per group
    (3072, 8, 300, 0, 2, 64, "combines"),     # no always-on group, items of eight and two K steps, at the line
    (4096, 16, 32, 4, 1, 51, "combines"),     # a fourth tile of three rows in the always-on group, one or two in the others
    (4096, 4, 32, 2, 2, 63, "tiles"),         # every token chooses every expert: 63 rows per row of weights
])
def test_down_and_combine_in_one_launch_beyond_32_tokens(binding, d, N, m, n_s, k, T, kernel):
    """Token tiles two at a time through the registers of the fused down + combine launch."""
    cfg, weights, part, x, layer = _case(binding, d, N, m, n_s, k, T, seed=8)
    assert layer.forward_plan(T)["down"][0] == kernel
    check_flat(cfg, weights, part, x, layer.forward(x))
    layer.close()


@pytest.mark.parametrize("m", [32, 128, 129, 384, 385])
@pytest.mark.parametrize("T", [1, 9, 16])
def test_down_and_combine_of_narrow_experts(binding, m, T):
    """Work items of up to four K steps and of more, alone and behind a full one: 1, 4, 5, 8 + 4 and 8 + 5 steps."""
    cfg, weights, part, x, layer = _case(binding, 512, 24, m, 1, 10, T, seed=9)
    assert layer.forward_plan(T)["down"][0] == "combines"
    check_flat(cfg, weights, part, x, layer.forward(x))
    layer.close()


@pytest.mark.parametrize("d,N,m,n_s,k,T", [
    (3072, 16, 40, 1, 3, 48),     # slot weights of Eq. 9
    (4096, 65, 32, 1, 9, 64),     # 65 groups: the last one alone in the second half of the lookup
    (3072, 64, 16, 0, 16, 33),    # 64, no always-on group, as many slots per token as there can be
])
def test_gated_down_and_combine_beyond_32_tokens(binding, d, N, m, n_s, k, T):
    """The fused down + combine launch with four token tiles, slot weights other than one and many groups."""
    cfg, weights, part, x, layer = _case(binding, d, N, m, n_s, k, T, seed=10)
    u, b = synth.make_gate_params(cfg, seed=7300)
    layer.set_gate_params(u, b)
    assert layer.forward_plan(T)["down"][0] == "combines"
    check_flat(cfg, weights, part, x, layer.forward(x), u=u, b=b)
    layer.close()


@pytest.mark.parametrize("n_outer,N,n_s,k", [(4, 8, 2, 2), (16, 5, 1, 1)])       # 28 groups; 80
def test_hierarchical_down_and_combine_beyond_32_tokens(binding, n_outer, N, n_s, k):
    """The same for hierarchies, whose slots carry the outer weight, and for their dense form."""
    cfg = synth.scaled(synth.CONFIGS[4], d_model=3072, d_ff=N * 24, n_experts=N, n_shared=n_s, top_k=k, n_outer=n_outer,
                       outer_top_k=2, n_centres=16)
    hier, experts, w_router, offsets = _make(binding, cfg, gate=True)
    for T in (33, 64):
        assert hier.forward_plan(T)["down"][0] == "combines"
        assert hier.forward_plan(T, dense=True)["down"][0] == ("combines" if T * 2 <= 16 * n_outer else "tiles")
        x = synth.make_token_source(cfg).eval_batch(8, n=T)
        _check(cfg, experts, w_router, offsets, x, hier.forward(x), hier.dense_forward(x), np.arange(0, T, 5))
    hier.close()


@pytest.mark.parametrize("d,N,n_s,k,T,scorer", [
    (328, 8, 1, 2, 70, ("tokens", 0)),         # a width without K slices
    (512, 9, 1, 2, 64, ("small", 8)),
    (8448, 8, 1, 2, 18, ("small", 8)),         # 33 K steps per slice: waves of nine, in runs of eight and one, the last of six
    (768, 17, 1, 3, 65, ("selects", 3)),
    (1024, 17, 1, 16, 70, ("selects", 4)),
    (2048, 16, 0, 3, 2400, ("selects", 4)),
    (2560, 8, 1, 2, 4064, ("selects", 5)),     # slices of two chunks
    (2560, 8, 1, 2, 4065, ("split", 2)),       # two slices of five chunks: one more than the pairs that the one launch takes
    (2304, 8, 1, 2, 200, ("split", 3)),        # three of three
    (512, 9, 1, 2, 8300, ("selects", 2)),      # 32 tokens per workgroup
    (2560, 40, 2, 5, 150, ("split", 5)),       # 128 router rows, more than a workgroup pulls
])
def test_scorer_of_a_batch(binding, d, N, n_s, k, T, scorer):
    cfg, weights, part, x, layer = _case(binding, d, N, 16, n_s, k, T, seed=11)
    assert layer.scorer_plan(T) == scorer
    out = layer.forward(x)
    check_flat(cfg, weights, part, x, out)
    assert np.array_equal(out["counts"], np.bincount(out["topk"].ravel(), minlength=cfg.n_routed))
    layer.close()
