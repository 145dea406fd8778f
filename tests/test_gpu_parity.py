"""GPU parity: the HIP library, called through its C ABI, against the fp64 CPU oracle on the same
seeded stored inputs.

Tolerances (relative Frobenius error of out_grad against the oracle):
  * stated for this path: 1e-2 for 16-bit inputs, 1e-4 for fp32 inputs; per-sample norms 5e-3 relative;
  * derived from the arithmetic and asserted as well, so that a partial bug cannot hide in the slack:
      - two-pass schedule and fp32 inputs: fp32 accumulation only (products of 16-bit inputs are exact in
        fp32), error ~ sqrt(T) * 2^-24, asserted <= 5e-5;
      - scratch schedule, 16-bit inputs: one extra rounding of G_i to 16 bits, rms 2^-9 / sqrt(3) ~ 1.1e-3
        relative for bf16, asserted <= 4e-3;
      - norms: two-pass, ghost, explicit and fp32 paths take them from fp32 sums: asserted <= 1e-4.  The scratch
        schedule with 16-bit inputs takes the norm of the tile as parked in bfloat16 (so that the clip factor bounds
        what is summed): each element moves by at most 2^-8 relative, the norm of many by less than 2^-9 (asserted,
        + 1e-5), and for tiles of 2^16 elements or more the roundings average out (asserted <= 1e-4);
      - noise field: |z_gpu - z_oracle| <= 2e-6 per element (fp32 Box-Muller on exact 24-bit uniforms; the
        host build of the same header measures 6e-7), so out(sigma) - out(0) is compared at 4e-6 * sigma * C
        max-abs (one more fp32 rounding of the sum) and 1e-6 relative Frobenius.
The noisy output alone is never the only check: with sigma = 1 the noise dwarfs the clipped signal.
"""
import numpy as np
import pytest
import torch

from oracle import flashdp_oracle as O
import workloads as W
import paper_2507_01154_amd as F
from gpu_util import DEV, rel_fro, run_layer, to_device, env, oracle_signal_and_bound, elementwise_excess

pytestmark = pytest.mark.gpu

TOL_STATED = {"bf16": 1e-2, "f16": 1e-2, "fp32": 1e-4}
TOL_NORM_STATED = 5e-3


def tight_tol(dtype, schedule):
    if dtype == "fp32" or schedule in ("twopass", "explicit", "ghost"):
        return 5e-5        # (fp32 inputs asked for "fused" take the scratch schedule with an fp32 scratch)
    return 4e-3   # the 16-bit scratch is bfloat16 for bf16 and for fp16 inputs


def check_case(X, dY, C, sigma, seed, layer, dtype, schedule, tile=None, oracle=None):
    """The four-part protocol; returns realised errors for logging."""
    D, P = dY.shape[2], X.shape[2]
    want0, wn = oracle if oracle is not None else O.linear_dp_grad(X, dY, C, 0.0, seed, layer)
    # the same from the oracle's stage functions, with the per-element magnitude sum_i c_i |G_i|
    Xw, dYw = (X.astype(np.float32), dY.astype(np.float32)) if X.dtype == np.float16 else (X, dY)
    want0_b, wn_b, bound = oracle_signal_and_bound(Xw, dYw, C)
    assert np.array_equal(want0_b, want0) and np.array_equal(wn_b, wn)
    got0, gn, used = run_layer(X, dY, C, 0.0, seed, layer, schedule, tile=tile)
    if schedule != "auto":
        assert used == schedule
    assert np.all(np.isfinite(got0)) and np.all(np.isfinite(gn))
    e_sig = rel_fro(got0, want0)
    e_norm = float(np.max(np.abs(gn - wn) / np.maximum(wn, 1e-300))) if np.all(wn > 0) else float(np.max(np.abs(gn - wn)))
    assert e_sig <= TOL_STATED[dtype], (e_sig, used)
    assert e_sig <= tight_tol(dtype, used), (e_sig, used)
    parked = dtype != "fp32" and used in ("scratch", "overlap", "fused")
    worst, k = elementwise_excess(got0, want0, bound, parked)
    assert worst <= 1.0, (f"element {divmod(k, P)}: got {got0.reshape(-1)[k]!r}, want {want0.reshape(-1)[k]!r}, "
                          f"sum_i c_i|G_i| {bound.reshape(-1)[k]!r}, error / allowed = {worst:.3f}", used)
    tol_norm = 2.0 ** -9 + 1e-5 if (parked and D * P < 65536) else 1e-4
    assert e_norm <= TOL_NORM_STATED and e_norm <= tol_norm, e_norm
    e_noise = 0.0
    if sigma > 0:
        got1, gn1, _ = run_layer(X, dY, C, sigma, seed, layer, schedule, tile=tile)
        z = O.noise_field(seed, layer, D * P).reshape(D, P)
        diff = got1.astype(np.float64) - got0.astype(np.float64)
        e_noise = float(np.max(np.abs(diff - sigma * C * z)))
        assert e_noise <= 4e-6 * sigma * C * max(1.0, float(np.max(np.abs(got0))) / (sigma * C)), e_noise
        assert rel_fro(diff, sigma * C * z) <= 1e-6
        assert rel_fro(got1, want0 + sigma * C * z) <= TOL_STATED[dtype]
        assert np.array_equal(gn1, gn)                      # noise never touches the norms
    return e_sig, e_norm, e_noise, used


# ---------------------------------------------------------------------------------------------------
# noise generator on its own
# ---------------------------------------------------------------------------------------------------

@pytest.mark.parametrize("seed,layer,n", [(1, 0, 1 << 20), ((5 << 32) | 77, 6, 1000003), (0, 0xFFFFFFFF, 7), (3, 2, 4096)])
def test_noise_field_matches_oracle(seed, layer, n):
    z = torch.full((n + 8,), float("nan"), device=DEV)
    F.flashdp_noise_field(seed, layer, n, z)
    torch.cuda.synchronize()
    got = z.cpu().numpy()
    assert np.all(np.isnan(got[n:]))                        # nothing written past n
    want = O.noise_field(seed, layer, n)
    assert np.max(np.abs(got[:n] - want)) <= 2e-6


def test_box_muller_edge_words():
    edge = [0, 255, 256, 0xFFFFFFFF, 0xFFFFFF00, 0x80000000, 0x7FFFFFFF, 0x40000000, 0x3FFFFFFF, 0xC0000000,
            0xBFFFFFFF, 0x20000000, 0xE0000000, 0x100, 0x200, 0x5FFFFFFF, 0x60000000, 0x2FFFFFFF, 0x30000000]
    w = np.array([(a, b, b, a) for a in edge for b in edge], dtype=np.uint32)
    rng = np.random.default_rng(3)
    w = np.concatenate([w, rng.integers(0, 1 << 32, size=(1 << 18, 4), dtype=np.uint64).astype(np.uint32)])
    dw = torch.from_numpy(w.view(np.int32)).to(DEV)
    z = torch.empty(w.shape, device=DEV, dtype=torch.float32)
    F.flashdp_box_muller(dw, w.shape[0], z)
    torch.cuda.synchronize()
    want = O.gaussians_from_words(w)
    assert np.max(np.abs(z.cpu().numpy() - want)) <= 2e-6


# ---------------------------------------------------------------------------------------------------
# configuration 1 (tiny, fp32) and its companion
# ---------------------------------------------------------------------------------------------------

@pytest.mark.parametrize("schedule", ["twopass", "scratch"])
@pytest.mark.parametrize("C", [1.0, 20.0])
def test_tiny_fp32(schedule, C):
    w = W.WORKLOADS["tiny_fp32"]
    X, dY = W.make_layer(w, 0)
    e = check_case(X, dY, C, 1.0, w.noise_seed, 0, "fp32", schedule)
    print("tiny_fp32", schedule, C, e)


# ---------------------------------------------------------------------------------------------------
# small shapes spanning several tiles with ragged edges, every kernel variant
# ---------------------------------------------------------------------------------------------------

SMALL = [
    # B, T, d_in, d_out
    (3, 200, 328, 520),      # several 128/256 tiles, ragged in every dimension, T not a multiple of 64
    (2, 64, 256, 256),       # exactly one 256 tile, one k-tile
    (5, 1, 8, 8),            # T = 1, smallest matrix-core shape
    (2, 130, 264, 24),       # thin output
]


@pytest.mark.parametrize("shape", SMALL)
@pytest.mark.parametrize("schedule", ["twopass", "scratch", "explicit"])
@pytest.mark.parametrize("tile", [2, 3, 4, 6])
def test_small_bf16_all_tiles(shape, schedule, tile):
    B, T, P, D = shape
    base = W.WORKLOADS["gpt2_small_mlp_up"]
    w = W.scaled_down(base, B=B, T=T, dims=[(P, D)])
    X, dY = W.make_layer(w, 0)
    e = check_case(X, dY, 1.0, 1.0, 11, 3, "bf16", schedule, tile=tile)
    print(shape, schedule, tile, e)


@pytest.mark.parametrize("schedule", ["twopass", "scratch", "explicit"])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("shape,tile", [((3, 37, 77, 5), None), ((2, 40, 3, 131), None), ((4, 16, 33, 35), None), ((3, 37, 77, 131), -1)])
def test_16_bit_shapes_of_the_generic_kernel(shape, tile, dtype, schedule):
    # rows shorter than 16 bytes, one small tile, and sizes that take the matrix cores unless switched off; the total of
    # the accumulating pass differs from the matrix cores' by the order of fp32 additions only
    B, T, P, D = shape
    w = W.scaled_down(W.WORKLOADS["gpt2_small_mlp_up"], B=B, T=T, dims=[(P, D)])
    X, dY = W.make_layer(w, 0)
    want = None
    if dtype == "f16":
        X, dY = O.widen(X).astype(np.float16), O.widen(dY).astype(np.float16)
        want = O.linear_dp_grad(X.astype(np.float32), dY.astype(np.float32), 1.0, 0.0, 5, 1)
    check_case(X, dY, 1.0, 0.5, 5, 1, dtype, schedule, tile=tile, oracle=want)
    assert F.flashdp_last_kernel() == "gemm_simple_kernel"
    if tile is not None:
        generic, n0, _ = run_layer(X, dY, 1.0, 0.0, 5, 1, schedule, tile=tile)
        cores, n1, _ = run_layer(X, dY, 1.0, 0.0, 5, 1, schedule)
        assert F.flashdp_last_kernel() == "gemm_mfma_kernel"
        tol = 4e-3 if schedule == "scratch" else 1e-5      # parked values may round the other way
        assert rel_fro(generic, cores.astype(np.float64)) <= tol and np.allclose(n0, n1, rtol=1e-4 if schedule == "scratch" else 1e-5, atol=0)


@pytest.mark.parametrize("schedule", ["twopass", "scratch", "explicit"])
def test_odd_dims(schedule):
    base = W.WORKLOADS["gpt2_small_mlp_up"]
    w = W.scaled_down(base, B=3, T=37, dims=[(77, 131)])
    X, dY = W.make_layer(w, 0)
    check_case(X, dY, 1.0, 0.5, 5, 1, "bf16", schedule)


@pytest.mark.parametrize("dtype,B,T,P,D,kernel", [(torch.float32, 52, 37, 509, 255, "gemm_mfma_f32_kernel"), (torch.float32, 1, 9, 3001, 3001, "gemm_mfma_f32_kernel"),
                                                  (torch.float32, 2, 40, 77, 131, "gemm_simple_kernel"), (torch.bfloat16, 3, 70, 129, 257, "gemm_mfma_kernel"),
                                                  (torch.bfloat16, 1, 33, 3001, 3001, "gemm_mfma_kernel")])
@pytest.mark.parametrize("schedule", ["twopass", "scratch", "explicit"])
def test_unaligned_sizes_add_to_an_earlier_micro_batch(dtype, B, T, P, D, kernel, schedule):
    g = torch.Generator(device=DEV).manual_seed(P + D)
    x, y = torch.randn((B, T, P), generator=g, device=DEV).to(dtype), (0.05 * torch.randn((B, T, D), generator=g, device=DEV)).to(dtype)
    out = torch.full((D, P), float("nan"), device=DEV)
    L = [dict(X=x, dY=y, d_in=P, d_out=D, C=1.0, sigma=0.0, seed=1, layer=0, out_grad=out, out_norms=None)]
    F.flashdp_block_dp_grad_micro(L, B, T, F.dtype_code(x), schedule, accumulate=False, add_noise=False)
    assert F.flashdp_last_kernel() == kernel
    once = out.clone()
    assert torch.isfinite(once).all()
    F.flashdp_block_dp_grad_micro(L, B, T, F.dtype_code(x), schedule, accumulate=True, add_noise=False)
    # the same sum added to itself, in one of two orders of at most 45 fp32 additions
    assert float((out.double() - 2.0 * once.double()).norm() / (2.0 * once.double()).norm()) <= 1e-6


@pytest.mark.parametrize("schedule", ["twopass", "scratch", "explicit"])
@pytest.mark.parametrize("dtype,shape", [("bf16", s) for s in [(2, 33, 9, 72), (1, 1, 15, 131), (3, 70, 129, 257), (2, 64, 255, 136),
                                                               (2, 40, 264, 135), (130, 20, 265, 10), (3, 97, 2049, 2303)]]
                         + [("f16", (2, 65, 71, 383)), ("fp32", (10, 37, 509, 255)), ("fp32", (2, 18, 769, 1021)), ("fp32", (52, 37, 509, 255)),
                            ("fp32", (8, 18, 769, 1021))])
def test_sizes_no_vector_width_divides(dtype, shape, schedule):
    # edges of the 128 and 256 tiles, chunks that reach 1..7 columns past a row, one token, single short rows
    B, T, P, D = shape
    rng = np.random.default_rng(B * T + P)
    X = rng.standard_normal((B, T, P)).astype(np.float32)
    dY = (rng.standard_normal((B, T, D)) * 0.05 * (10.0 ** rng.uniform(-1, 1, size=(B, 1, 1)))).astype(np.float32)
    want = None
    if dtype == "f16":
        X, dY = X.astype(np.float16), dY.astype(np.float16)
        want = O.linear_dp_grad(X.astype(np.float32), dY.astype(np.float32), 1.0, 0.0, 9, 2)
    elif dtype == "bf16":
        X, dY = ((a.view(np.uint32) >> 16).astype(np.uint16) for a in (X, dY))
    check_case(X, dY, 1.0, 1.0, 9, 2, dtype, schedule, oracle=want)
    # fp32: the matrix-core kernel where its 256 x 256 tiles occupy enough of the chip (the 52 and the 8 samples)
    assert F.flashdp_last_kernel() == ("gemm_mfma_kernel" if dtype != "fp32" else "gemm_mfma_f32_kernel" if B in (52, 8) else "gemm_simple_kernel")


@pytest.mark.parametrize("B,P,D", [(17, 1999, 2001), (16, 1999, 2001), (17, 1999, 2004)])
def test_fp32_samples_that_no_cache_holds_are_summed_past_the_caches(B, P, D):
    # both forms of the fp32 aggregation, with and without samples that start between two 16-byte groups; fp64 on the GPU
    g = torch.Generator(device=DEV).manual_seed(D)
    X, dY = torch.randn((B, 2, P), generator=g, device=DEV), torch.randn((B, 2, D), generator=g, device=DEV)
    out, norms = torch.full((D, P), float("nan"), device=DEV), torch.empty((B,), device=DEV)
    F.flashdp_block_dp_grad([dict(X=X, dY=dY, d_in=P, d_out=D, C=1.0, sigma=0.0, seed=1, layer=0, out_grad=out, out_norms=norms)],
                            B, 2, F.F32, "scratch")
    want = torch.zeros((D, P), dtype=torch.float64, device=DEV)
    for i in range(B):
        G = dY[i].double().T @ X[i].double()
        want += G / G.norm().clamp(min=1.0)
    assert float((out - want).norm() / want.norm()) <= 5e-5


@pytest.mark.parametrize("schedule", ["twopass", "scratch", "explicit"])
@pytest.mark.parametrize("B,T,P,D,kernel", [(70, 16, 500, 10, "gemm_simple_kernel"), (70, 17, 500, 10, "gemm_mfma_kernel"),
                                            (130, 40, 10, 265, "gemm_mfma_kernel"), (128, 4, 513, 250, "gemm_mfma_kernel")])
def test_thin_layers_of_many_samples(B, T, P, D, kernel, schedule):
    # on both sides of the rules between the generic kernel and the two tilings of unaligned rows
    rng = np.random.default_rng(B + T + P)
    X = W.float32_to_bf16_bits(rng.standard_normal((B, T, P)).astype(np.float32))
    dY = W.float32_to_bf16_bits((rng.standard_normal((B, T, D)) * 0.05 * (10.0 ** rng.uniform(-1, 1, size=(B, 1, 1)))).astype(np.float32))
    check_case(X, dY, 1.0, 0.5, 9, 2, "bf16", schedule)
    assert F.flashdp_last_kernel() == kernel


@pytest.mark.parametrize("B", [1, 3, 70])
@pytest.mark.parametrize("P,D", [(9, d) for d in range(8, 16)] + [(3, 3), (1, 1), (2, 3), (7, 1), (1, 8), (67, 31)])
def test_last_group_of_the_16_bit_aggregation(B, P, D):
    # every remainder of the layer's size by eight, layers of fewer than eight elements, clip factors worked out by the
    # aggregation itself (up to 64 samples) and before it; noise; a second micro-batch added to the first
    rng = np.random.default_rng(B * 100 + P * D)
    X = W.float32_to_bf16_bits(rng.standard_normal((B, 5, P)).astype(np.float32))
    dY = W.float32_to_bf16_bits((rng.standard_normal((B, 5, D)) * 0.3).astype(np.float32))
    sig, wn, bound = oracle_signal_and_bound(X, dY, 1.0)
    z = O.noise_field(9, 2, D * P).reshape(D, P)
    for sigma in (0.0, 0.5):
        got, gn, _ = run_layer(X, dY, 1.0, sigma, 9, 2, "scratch")
        # a value parked as bfloat16 moves by up to 2^-8 of itself, and so does a norm of few values; noise as elsewhere here
        assert np.all(np.abs(gn - wn) <= (2.0 ** -8 + 1e-6) * wn)
        assert np.all(np.abs(got - sig - sigma * z) <= 2.0 ** -7 * bound + 4e-6)
    dX, ddY = to_device(X), to_device(dY)
    out = torch.full((D * P + 8,), float("nan"), device=DEV)
    L = [dict(X=dX, dY=ddY, d_in=P, d_out=D, C=1.0, sigma=0.5, seed=9, layer=2, out_grad=out, out_norms=None)]
    F.flashdp_block_dp_grad_micro(L, B, 5, F.BF16, "scratch", accumulate=False, add_noise=False)
    once = out.clone()
    F.flashdp_block_dp_grad_micro(L, B, 5, F.BF16, "scratch", accumulate=True, add_noise=True)
    assert torch.isnan(out[D * P:]).all()                                      # nothing written past the layer
    want = 2.0 * once[:D * P].double() + 0.5 * torch.from_numpy(z.reshape(-1)).to(DEV)
    # two orders of at most 71 fp32 additions each, and the noise field's 2e-6
    assert float((out[:D * P] - want).abs().max()) <= 4e-6 * max(1.0, float(once[:D * P].abs().max()))


@pytest.mark.parametrize("dtype,B,T,P,D", [(torch.bfloat16, 64, 128, 300, 30), (torch.bfloat16, 8, 1024, 768, 10), (torch.float16, 4, 200, 4001, 2049),
                                           (torch.float32, 52, 37, 509, 255), (torch.float32, 3, 100, 2222, 3333)])
def test_accumulation_of_unaligned_sizes_adds_whole_samples(dtype, B, T, P, D):
    # Each sample is summed by itself and then added to the total.  A sum of T products in steps of 8 to 16 rounds T / 8
    # times at the size it has grown to, 2^-24 / sqrt(3) each: 3e-7 of the result for T = 1024, less for fewer, and B
    # additions add as much for B = 64.  (All B * T products in one running sum: 6e-7 to 7e-7 on these shapes.)
    g = torch.Generator(device=DEV).manual_seed(P)
    x, y = torch.randn((B, T, P), generator=g, device=DEV).to(dtype), (0.05 * torch.randn((B, T, D), generator=g, device=DEV)).to(dtype)
    out = [torch.full((D, P), float("nan"), device=DEV) for _ in range(2)]
    F.flashdp_plain_grad(x, y, B, T, P, D, F.dtype_code(x), out[0])
    F.flashdp_block_dp_grad([dict(X=x, dY=y, d_in=P, d_out=D, C=1.0, sigma=0.0, seed=1, layer=0, out_grad=out[1], out_norms=None)],
                            B, T, F.dtype_code(x), "twopass")
    want = torch.zeros((2, D, P), dtype=torch.float64, device=DEV)
    for i in range(B):
        G = y[i].double().T @ x[i].double()
        want[0] += G
        want[1] += G / G.norm().clamp(min=1.0)
    for o, w in zip(out, want):
        assert float((o - w).norm() / w.norm()) <= 3.5e-7


@pytest.mark.parametrize("schedule,scale,C", [("twopass", 1e13, 1.0), ("twopass", 1e7, 1e-30), ("ghost", 1e7, 1e-30)])
@pytest.mark.parametrize("dtype,B,T,P,D", [(torch.bfloat16, 5, 37, 77, 131), (torch.bfloat16, 4, 70, 136, 257), (torch.bfloat16, 3, 20, 4001, 2049),
                                           (torch.float32, 5, 37, 77, 131), (torch.float32, 52, 37, 509, 255), (torch.float32, 3, 9, 4001, 2049)])
def test_accumulation_of_unaligned_sizes_survives_a_factor_of_zero(dtype, B, T, P, D, schedule, scale, C):
    # one sample's clip factor is 0 (its norm is beyond what fp32 sums of squares hold, or 1e45 times C), its elements are
    # finite: the other samples' sum has to stay what it is, wherever in the batch that sample stands (a total rescaled by
    # c_i / c_(i+1) would not)
    g = torch.Generator(device=DEV).manual_seed(P)
    x0, y0 = torch.randn((B, T, P), generator=g, device=DEV), 0.05 * torch.randn((B, T, D), generator=g, device=DEV)
    for at in (0, 1, B - 1):
        x, y = x0.clone(), y0.clone()
        x[at] *= scale
        y[at] *= scale
        x, y = x.to(dtype), y.to(dtype)
        out, norms = torch.full((D, P), float("nan"), device=DEV), torch.empty((B,), device=DEV)
        F.flashdp_block_dp_grad([dict(X=x, dY=y, d_in=P, d_out=D, C=C, sigma=0.0, seed=1, layer=0, out_grad=out, out_norms=norms)],
                                B, T, F.dtype_code(x), schedule)
        want = torch.zeros((D, P), dtype=torch.float64, device=DEV)
        for i in range(B):
            if i != at:
                G = y[i].double().T @ x[i].double()
                want += G / (G.norm() / C).clamp(min=1.0)
        assert float(norms[at]) / C > 1.5e45
        assert float((out - want).norm() / want.norm()) <= 5e-5, at


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("B,T,dims", [(1, 100, [(136, 264), (8, 8), (768, 128)]), (3, 33, [(256, 384)] * 9), (2, 64, [(130, 257), (128, 64), (264, 72)])])
def test_layers_of_a_call_are_those_of_single_calls(B, T, dims, dtype):
    # layers that share launches (16-bit, small), more of them than one launch takes, one among them that takes another
    # kernel, workspaces that hold all, two or one of them, and one output buffer named twice (the later layer stands)
    rng = np.random.default_rng(B + T)
    tt = torch.bfloat16 if dtype == "bf16" else torch.float32
    layers, want = [], []
    for l, (P, D) in enumerate(dims):
        X = torch.from_numpy(rng.standard_normal((B, T, P)).astype(np.float32)).to(DEV).to(tt)
        dY = torch.from_numpy((rng.standard_normal((B, T, D)) * 0.05).astype(np.float32)).to(DEV).to(tt)
        L = dict(X=X, dY=dY, d_in=P, d_out=D, C=1.0 + l, sigma=0.5, seed=9 + l, layer=l,
                 out_grad=torch.empty((D, P), device=DEV), out_norms=torch.empty((B,), device=DEV))
        F.flashdp_block_dp_grad([L], B, T, F.dtype_code(X), "scratch")
        want.append((L["out_grad"].clone(), L["out_norms"].clone()))
        layers.append(L)
    code = F.dtype_code(layers[0]["X"])
    one = F.flashdp_workspace_bytes(layers, B, T, code, "scratch")
    for ws in (one, 2 * one, 9 * one, None):
        for L in layers:
            L["out_grad"].fill_(float("nan"))
            L["out_norms"].fill_(float("nan"))
        F.flashdp_block_dp_grad(layers, B, T, code, "scratch", None if ws is None else torch.empty((ws,), dtype=torch.uint8, device=DEV))
        for L, (g, n) in zip(layers, want):
            assert torch.equal(L["out_grad"], g) and torch.equal(L["out_norms"], n), ws
    if len(set(dims)) == 1:
        F.flashdp_block_dp_grad([layers[0], dict(layers[1], out_grad=layers[0]["out_grad"])], B, T, code, "scratch",
                                torch.empty((9 * one,), dtype=torch.uint8, device=DEV))
        assert torch.equal(layers[0]["out_grad"], want[1][0])


@pytest.mark.parametrize("dtype", ["bf16", "f16", "fp32"])
@pytest.mark.parametrize("shape", [(17, 1, 1), (3, 63, 130), (2, 65, 67), (2, 66, 3), (2, 3, 65), (33, 64, 64), (65, 130, 61), (256, 257, 10), (17, 2884, 2950), (31, 2816, 3072)])
def test_rows_without_a_sequence(shape, dtype):
    # both tile sizes (2816 x 3072 and 2884 x 2950: 128), edges of tiles and of the batch's steps, features that no vector
    # width divides, a second micro-batch added to the first one's sum, a workspace of the smallest size that is accepted
    B, P, D = shape
    rng = np.random.default_rng(B + P * D)
    X = rng.standard_normal((B, 1, P)).astype(np.float32)
    dY = (rng.standard_normal((B, 1, D)) * 0.05 * (10.0 ** rng.uniform(-1, 1, size=(B, 1, 1)))).astype(np.float32)
    want = None
    if dtype == "f16":
        X, dY = X.astype(np.float16), dY.astype(np.float16)
        want = O.linear_dp_grad(X.astype(np.float32), dY.astype(np.float32), 1.0, 0.0, 9, 2)
    elif dtype == "bf16":
        X, dY = ((a.view(np.uint32) >> 16).astype(np.uint16) for a in (X, dY))
    e_sig, e_norm, _, used = check_case(X, dY, 1.0, 1.0, 9, 2, dtype, "auto", oracle=want)
    assert used == "rows" and e_sig <= 2e-6 and e_norm <= 2e-7     # fp32 sums of at most 256 products; norms rounded once
    dX, ddY = to_device(X), to_device(dY)
    once, twice = (torch.empty((D, P), device=DEV) for _ in range(2))
    L = [dict(X=dX, dY=ddY, d_in=P, d_out=D, C=1.0, sigma=0.0, seed=9, layer=2, out_grad=o, out_norms=None) for o in (once, twice)]
    ws = torch.empty((F.flashdp_workspace_bytes([L[0]], B, 1, F.dtype_code(dX), "twopass"),), dtype=torch.uint8, device=DEV)
    for k in range(3):
        F.flashdp_block_dp_grad_micro([L[min(k, 1)]], B, 1, F.dtype_code(dX), "auto", ws, accumulate=k == 2, add_noise=False)
    assert torch.equal(twice, 2.0 * once)


@pytest.mark.parametrize("B,P,D,dtype,used", [(1, 16388, 12, torch.float32, "scratch"), (2, 11, 20001, torch.bfloat16, "scratch"),
                                              (1, 16384, 12, torch.float32, "rows"), (4, 2048, 2049, torch.float32, "rows"),
                                              (4, 2047, 2051, torch.float16, "rows"), (3, 11, 20001, torch.bfloat16, "rows"),
                                              (2, 17001, 512, torch.float32, "rows")])
def test_rows_without_a_sequence_that_are_long(B, P, D, dtype, used):
    g = torch.Generator(device=DEV).manual_seed(P)
    X, dY = (torch.randn((B, 1, n), generator=g, device=DEV).to(dtype) for n in (P, D))
    out, norms = torch.full((D, P), float("nan"), device=DEV), torch.full((B,), float("nan"), device=DEV)
    F.flashdp_block_dp_grad([dict(X=X, dY=dY, d_in=P, d_out=D, C=1.0, sigma=0.0, seed=1, layer=0, out_grad=out, out_norms=norms)],
                            B, 1, F.dtype_code(X), "auto")
    assert F.flashdp_last_schedule() == used
    x, y = X.double()[:, 0], dY.double()[:, 0]
    n = x.norm(dim=1) * y.norm(dim=1)
    want = (y / n[:, None]).T @ x
    # scratch: norms of fp32 sums or of 2^16 or more values parked as bfloat16, 1e-4 as stated at the head of this file
    assert float(((norms - n) / n).abs().max()) <= (2e-7 if used == "rows" else 1e-4)
    assert float((out - want).norm() / want.norm()) <= (4e-3 if used == "scratch" and dtype != torch.float32 else 2e-6)


def test_rows_without_a_sequence_take_any_workspace_that_holds_a_chunk():
    # many samples of a small layer: a workspace for one parked sample is smaller than the batch's factors and partials
    B, P, D = 2000, 10, 6
    g = torch.Generator(device=DEV).manual_seed(1)
    X, dY = (torch.randn((B, 1, n), generator=g, device=DEV) for n in (P, D))
    out, norms = (torch.empty(s, device=DEV) for s in ((D, P), (B,)))
    L = [dict(X=X, dY=dY, d_in=P, d_out=D, C=1.0, sigma=0.0, seed=1, layer=0, out_grad=out, out_norms=norms)]
    want_n = X.double().norm(dim=2)[:, 0] * dY.double().norm(dim=2)[:, 0]
    want = (dY.double()[:, 0] / want_n.clamp(min=1.0)[:, None]).T @ X.double()[:, 0]
    small = F.flashdp_workspace_bytes(L, B, 1, F.F32, "twopass")
    for n_ws, used in ((F.flashdp_workspace_bytes_chunked(L, B, 1, F.F32, 3, 1), "scratch"), (small, "rows")):
        assert used == "rows" or n_ws < small
        out.fill_(float("nan"))
        F.flashdp_block_dp_grad(L, B, 1, F.F32, "auto", torch.empty((n_ws,), dtype=torch.uint8, device=DEV))
        assert F.flashdp_last_schedule() == used
        assert torch.allclose(norms.double(), want_n, rtol=1e-6)
        assert float((out.double() - want).norm() / want.norm()) <= 5e-5
    with pytest.raises(F.FlashDPError) as ei:
        F.flashdp_block_dp_grad(L, B, 1, F.F32, "auto", torch.empty((512,), dtype=torch.uint8, device=DEV))
    assert ei.value.status == F.WORKSPACE_TOO_SMALL


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_rows_without_a_sequence_that_are_not_finite_or_overflow(dtype):
    # G_i is not formed there, so what its elements would show has to show all the same
    g = torch.Generator(device=DEV).manual_seed(3)
    B, P, D = 5, 72, 40
    x0, y0 = (torch.randn((B, 1, n), generator=g, device=DEV) for n in (P, D))

    def run(x, y, C):
        x, y = x.to(dtype), y.to(dtype)
        out, norms = torch.full((D, P), 7.0, device=DEV), torch.full((B,), 7.0, device=DEV)
        F.flashdp_block_dp_grad([dict(X=x, dY=y, d_in=P, d_out=D, C=C, sigma=0.0, seed=1, layer=0, out_grad=out, out_norms=norms)],
                                B, 1, F.dtype_code(x), "auto")
        assert F.flashdp_last_schedule() == "rows"
        want = x.double().square().sum(2).sqrt() * y.double().square().sum(2).sqrt()
        return out, norms, want[:, 0], x.double()[:, 0], y.double()[:, 0]

    for bad in (float("nan"), float("inf")):
        for operand in (0, 1):
            x, y = x0.clone(), y0.clone()
            (x, y)[operand][2, 0, 11] = bad
            out, norms, want, _, _ = run(x, y, 1.0)
            assert torch.isnan(out).all() and not torch.isfinite(norms[2])
            keep = [0, 1, 3, 4]
            assert torch.allclose(norms[keep].double(), want[keep], rtol=1e-6)
    # finite rows whose outer product overflows fp32
    x, y = x0.clone(), y0.clone()
    x[2] *= 1e30
    y[2] *= 1e30
    out, norms, _, _, _ = run(x, y, 1.0)
    assert torch.isnan(out).all() and torch.isinf(norms[2])
    # clip factors down to and below the smallest normal float: one sample that counts, so the output is its contribution
    for norm, C in ((1e11, 1.0), (1e31, 1.0), (2.5e37, 1.0), (1e21, 1e-19), (1.5e34, 1e-9), (1.2e33, 1e-12), (1e34, 1e-12)):
        x = torch.zeros_like(x0)
        x[2] = x0[2] * (norm / (x0[2].norm() * y0[2].norm()))
        out, norms, want, xd, yd = run(x, y0, C)
        n = float(out.double().norm())
        assert torch.isfinite(norms).all() and n <= C * (1 + 3e-7), (norm, C, n / C)
        if float(want[2]) / C < 1e38:      # the factor is a normal float: the direction and the length are right too
            exact = yd[2][:, None] * xd[2][None, :] * (C / float(want[2]))
            assert float((out.double() - exact).norm()) <= 1e-5 * C, (norm, C)


@pytest.mark.parametrize("schedule", ["twopass", "scratch", "explicit"])
@pytest.mark.parametrize("shape", [(3, 100, 136, 264), (2, 33, 50, 70), (3, 70, 332, 520), (2, 16, 128, 128)])
def test_f16_and_fp32_inputs(schedule, shape):
    B, T, P, D = shape
    rng = np.random.default_rng(B * T)
    X32 = rng.standard_normal((B, T, P)).astype(np.float32)
    dY32 = (rng.standard_normal((B, T, D)) * 0.05 * (10.0 ** rng.uniform(-1, 1, size=(B, 1, 1)))).astype(np.float32)
    check_case(X32, dY32, 1.0, 1.0, 9, 2, "fp32", schedule)
    X16, dY16 = X32.astype(np.float16), dY32.astype(np.float16)
    want = O.linear_dp_grad(X16.astype(np.float32), dY16.astype(np.float32), 1.0, 0.0, 9, 2)
    check_case(X16, dY16, 1.0, 1.0, 9, 2, "f16", schedule, oracle=want)


# ---------------------------------------------------------------------------------------------------
# ghost-norm schedule: norms from the two Gram matrices (never formed in memory), then the clipped accumulation
# ---------------------------------------------------------------------------------------------------

@pytest.mark.parametrize("shape", SMALL + [
    (3, 300, 328, 520),      # 3 x 3 blocks of 128 rows: diagonal and off-diagonal blocks, ragged last block
    (2, 513, 72, 40),        # long sequence, small features: the regime the identity is meant for
    (2, 150, 77, 131),       # odd feature sizes: generic Gram kernel, 64-row blocks, ragged
])
def test_ghost_norm_schedule_bf16(shape):
    B, T, P, D = shape
    base = W.WORKLOADS["gpt2_small_mlp_up"]
    w = W.scaled_down(base, B=B, T=T, dims=[(P, D)])
    X, dY = W.make_layer(w, 0)
    e = check_case(X, dY, 1.0, 1.0, 11, 3, "bf16", "ghost")
    print(shape, "ghost", e)


@pytest.mark.parametrize("shape", [(3, 100, 136, 264), (2, 33, 50, 70), (2, 200, 128, 128)])
def test_ghost_norm_schedule_f16_and_fp32(shape):
    B, T, P, D = shape
    rng = np.random.default_rng(B * T + 1)
    X32 = rng.standard_normal((B, T, P)).astype(np.float32)
    dY32 = (rng.standard_normal((B, T, D)) * 0.05 * (10.0 ** rng.uniform(-1, 1, size=(B, 1, 1)))).astype(np.float32)
    check_case(X32, dY32, 1.0, 1.0, 9, 2, "fp32", "ghost")
    X16, dY16 = X32.astype(np.float16), dY32.astype(np.float16)
    want = O.linear_dp_grad(X16.astype(np.float32), dY16.astype(np.float32), 1.0, 0.0, 9, 2)
    check_case(X16, dY16, 1.0, 1.0, 9, 2, "f16", "ghost", oracle=want)


def test_ghost_norms_equal_contraction_norms_on_zero_and_single_token_samples():
    # a sample of zeros has norm 0 (factor 1) by either route; T = 1 makes the Gram matrices 1 x 1
    rng = np.random.default_rng(4)
    X = W.float32_to_bf16_bits(rng.standard_normal((3, 1, 16)).astype(np.float32))
    dY = W.float32_to_bf16_bits(rng.standard_normal((3, 1, 24)).astype(np.float32))
    X[1] = 0
    g, n, used = run_layer(X, dY, 1.0, 0.0, 1, 0, "ghost")
    t, m, _ = run_layer(X, dY, 1.0, 0.0, 1, 0, "twopass")
    assert used == "ghost" and n[1] == 0.0 and m[1] == 0.0
    assert np.allclose(n, m, rtol=1e-6, atol=0) and rel_fro(g, t.astype(np.float64)) <= 1e-6


def test_clip_branches_and_degenerate_inputs():
    base = W.WORKLOADS["gpt2_small_mlp_up"]
    w = W.scaled_down(base, B=4, T=96, dims=[(128, 136)])
    X, dY = W.make_layer(w, 0)
    _, norms = O.linear_dp_grad(X, dY, 1.0, 0.0, 0)
    C = float(np.sort(norms)[1] * 1.5)          # two samples below the threshold, two above
    assert np.sum(norms < C) == 2
    for schedule in ("twopass", "scratch"):
        check_case(X, dY, C, 0.0, 0, 0, "bf16", schedule)
    # a sample with zero gradient: norm 0, factor 1, no NaN
    dY0 = dY.copy()
    dY0[1] = 0
    for schedule in ("twopass", "scratch"):
        got, gn, _ = run_layer(X, dY0, 1.0, 0.0, 0, 0, schedule)
        want, wn = O.linear_dp_grad(X, dY0, 1.0, 0.0, 0)
        assert gn[1] == 0.0 and np.all(np.isfinite(got)) and rel_fro(got, want) <= 4e-3
    # B = 1
    check_case(X[:1], dY[:1], 1.0, 1.0, 4, 0, "bf16", "scratch")
    check_case(X[:1], dY[:1], 1.0, 1.0, 4, 0, "bf16", "twopass")


@pytest.mark.parametrize("tile", [None, 3, 6])
@pytest.mark.parametrize("schedule", ["scratch", "twopass"])
def test_a_clipped_contribution_never_exceeds_C(schedule, tile):
    """Sensitivity bound of Algorithm 1 on what is actually summed: with one sample and sigma = 0 the output IS that
    sample's clipped contribution, so its norm (taken in fp64 from the returned fp32 values) must not exceed C.  On the
    scratch schedule the summed tile is the one parked as bfloat16, whose norm - not the norm of the fp32 accumulators
    - is therefore the one that has to be clipped."""
    base = W.WORKLOADS["gpt2_small_mlp_up"]
    w = W.scaled_down(base, B=3, T=130, dims=[(520, 776)])
    X, dY = W.make_layer(w, 0)
    for i in range(3):
        for C in (1.0, 0.37):
            got, gn, used = run_layer(X[i:i + 1], dY[i:i + 1], C, 0.0, 1, 0, schedule, tile=tile)
            assert used == schedule and gn[0] > C                     # the sample does clip
            n_out = float(np.sqrt(np.sum(np.square(got.astype(np.float64)))))
            assert n_out <= C * (1 + 2e-7), (i, C, n_out / C - 1)       # fp32 rounding of c_i and of each product only
            assert n_out >= C * (1 - 1e-5)


def test_plain_grad_is_the_unclipped_limit():
    base = W.WORKLOADS["gpt2_small_mlp_up"]
    w = W.scaled_down(base, B=3, T=160, dims=[(264, 392)])
    X, dY = W.make_layer(w, 0)
    B, T, P = X.shape
    D = dY.shape[2]
    dX, ddY = to_device(X), to_device(dY)
    want = O.widen(dY).reshape(B * T, D).T @ O.widen(X).reshape(B * T, P)        # Eq. batched-grad
    for tile in (2, 3, 4):
        out = torch.full((D, P), float("nan"), device=DEV)
        with env(FLASHDP_TILE=tile):
            F.flashdp_plain_grad(dX, ddY, B, T, P, D, F.BF16, out)
        torch.cuda.synchronize()
        assert rel_fro(out.cpu().numpy(), want) <= 5e-6
    got, _, _ = run_layer(X, dY, 1e30, 0.0, 0, 0, "twopass")
    assert rel_fro(got, want) <= 5e-6


def test_repeatable_and_workspace_argument():
    base = W.WORKLOADS["gpt2_small_mlp_up"]
    w = W.scaled_down(base, B=4, T=128, dims=[(384, 520)])
    X, dY = W.make_layer(w, 0)
    a = run_layer(X, dY, 1.0, 1.0, 7, 1, "scratch")
    b = run_layer(X, dY, 1.0, 1.0, 7, 1, "scratch")
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])             # fixed-order reductions: bit-repeatable
    B, T, P = X.shape
    D = dY.shape[2]
    L = [dict(X=None, dY=None, d_in=P, d_out=D, C=1.0, sigma=1.0, seed=7, layer=1, out_grad=None)]
    need = F.flashdp_workspace_bytes(L, B, T, F.BF16, "scratch")
    small = F.flashdp_workspace_bytes(L, B, T, F.BF16, "twopass")
    assert need >= B * D * P * 2 and 0 < small < 65536
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    c = run_layer(X, dY, 1.0, 1.0, 7, 1, "scratch", workspace=ws)
    assert np.array_equal(a[0], c[0])
    d = run_layer(X, dY, 1.0, 1.0, 7, 1, "auto", workspace=ws[:small])           # too small for scratch: auto falls back
    assert d[2] == "twopass"
    with pytest.raises(F.FlashDPError) as ei:
        run_layer(X, dY, 1.0, 1.0, 7, 1, "scratch", workspace=ws[: need - 256])
    assert ei.value.status == F.WORKSPACE_TOO_SMALL
    need_x = F.flashdp_workspace_bytes(L, B, T, F.BF16, "explicit")
    assert need_x >= B * D * P * 4
    with pytest.raises(F.FlashDPError) as ei:
        run_layer(X, dY, 1.0, 1.0, 7, 1, "explicit", workspace=ws)          # sized for the 16-bit scratch only
    assert ei.value.status == F.WORKSPACE_TOO_SMALL
    e = run_layer(X, dY, 1.0, 1.0, 7, 1, "explicit", workspace=torch.empty(need_x, dtype=torch.uint8, device=DEV))
    assert e[2] == "explicit" and rel_fro(e[0], a[0].astype(np.float64)) <= 1e-2


def test_eleven_argument_entry_point_uses_context():
    base = W.WORKLOADS["gpt2_small_mlp_up"]
    w = W.scaled_down(base, B=2, T=64, dims=[(136, 264)])
    X, dY = W.make_layer(w, 0)
    B, T, P = X.shape
    D = dY.shape[2]
    dX, ddY = to_device(X), to_device(dY)
    out = torch.empty((D, P), device=DEV)
    norms = torch.empty((B,), device=DEV)
    F.flashdp_set_stream(None)
    F.flashdp_set_dtype(F.BF16)
    F.flashdp_set_layer(5)
    F.flashdp_set_schedule("auto")
    F.flashdp_set_workspace(None)
    F.flashdp_linear_dp_grad(dX, ddY, B, T, P, D, 1.0, 0.7, 123, out, norms)
    torch.cuda.synchronize()
    want, wn = O.linear_dp_grad(X, dY, 1.0, 0.7, 123, layer=5)
    assert rel_fro(out.cpu().numpy(), want) <= 1e-2
    z = O.noise_field(123, 5, D * P).reshape(D, P)
    sig, _ = O.linear_dp_grad(X, dY, 1.0, 0.0, 123, 5)
    assert rel_fro(out.cpu().numpy() - 0.7 * z, sig) <= 4e-3                     # the signal under the noise
    assert np.max(np.abs(norms.cpu().numpy() - wn) / wn) <= 1e-4
    F.flashdp_set_layer(0)


def test_block_variant_matches_layerwise_oracle():
    base = W.WORKLOADS["llama13b_block"]
    dims = [(128, 128), (128, 128), (128, 128), (128, 128), (128, 344), (128, 344), (344, 128)]
    w = W.scaled_down(base, B=3, T=96, dims=dims)
    layers, keep = [], []
    for l in range(len(dims)):
        X, dY = W.make_layer(w, l)
        P, D = dims[l]
        out = torch.full((D, P), float("nan"), device=DEV)
        norms = torch.full((w.B,), float("nan"), device=DEV)
        layers.append(dict(X=to_device(X), dY=to_device(dY), d_in=P, d_out=D, C=w.C, sigma=w.sigma,
                           seed=w.layer_seed(l), layer=l, out_grad=out, out_norms=norms))
        keep.append((X, dY))
    for schedule in ("scratch", "twopass"):
        F.flashdp_block_dp_grad(layers, w.B, w.T, F.BF16, schedule)
        torch.cuda.synchronize()
        for l, (X, dY) in enumerate(keep):
            sig, wn = O.linear_dp_grad(X, dY, w.C, 0.0, w.layer_seed(l), l)
            P, D = dims[l]
            z = O.noise_field(w.layer_seed(l), l, D * P).reshape(D, P)
            got = layers[l]["out_grad"].cpu().numpy()
            assert rel_fro(got - w.sigma * w.C * z, sig) <= tight_tol("bf16", schedule) + 1e-4   # fp32 cancellation of the noise
            assert np.max(np.abs(layers[l]["out_norms"].cpu().numpy() - wn) / wn) <= 1e-4


@pytest.mark.parametrize("schedule", ["scratch", "twopass"])
@pytest.mark.parametrize("shape", [(6, 96, 264, 392), (5, 40, 77, 131)])
def test_gradient_accumulation_over_micro_batches(schedule, shape):
    B, T, P, D = shape
    base = W.WORKLOADS["gpt2_small_mlp_up"]
    w = W.scaled_down(base, B=B, T=T, dims=[(P, D)])
    X, dY = W.make_layer(w, 0)
    split = [2, 1, B - 3]
    idx = np.cumsum([0] + split)
    mbs = [(X[a:b], dY[a:b]) for a, b in zip(idx[:-1], idx[1:])]
    sigma, seed, layer = 0.9, 21, 4
    want0, wn = O.accumulated_dp_grad(mbs, 1.0, 0.0, seed, layer)
    z = O.noise_field(seed, layer, D * P).reshape(D, P)
    out = torch.full((D, P), float("nan"), device=DEV)
    res = {}
    for sg in (0.0, sigma):
        got_norms = []
        for k, (xm, ym) in enumerate(mbs):
            b = xm.shape[0]
            norms = torch.full((b,), float("nan"), device=DEV)
            L = [dict(X=to_device(xm), dY=to_device(ym), d_in=P, d_out=D, C=1.0, sigma=sg, seed=seed, layer=layer,
                      out_grad=out, out_norms=norms)]
            F.flashdp_block_dp_grad_micro(L, b, T, F.BF16, schedule, accumulate=(k > 0), add_noise=(k == len(mbs) - 1))
            torch.cuda.synchronize()
            got_norms.append(norms.cpu().numpy())
        res[sg] = out.cpu().numpy().copy()
        for g, wv in zip(got_norms, wn):
            assert np.max(np.abs(g - wv) / wv) <= 1e-4
    assert rel_fro(res[0.0], want0) <= tight_tol("bf16", schedule)
    d = res[sigma].astype(np.float64) - res[0.0].astype(np.float64)
    assert np.max(np.abs(d - sigma * z)) <= 4e-6 * sigma * max(1.0, float(np.max(np.abs(res[0.0]))) / sigma)
    assert rel_fro(res[sigma], want0 + sigma * z) <= 1e-2
    # and it equals the one-call result on the whole batch up to fp32 summation order
    whole, _, _ = run_layer(X, dY, 1.0, 0.0, seed, layer, schedule)
    assert rel_fro(res[0.0], whole.astype(np.float64)) <= 1e-6


@pytest.mark.parametrize("tile", [6, 7, 8, 9])
@pytest.mark.parametrize("schedule", ["twopass", "scratch", "ghost"])
def test_direct_to_lds_kernel_f16_inputs_and_accumulation(schedule, tile):
    # the large-shape kernels (forced here on a small ragged shape; 6: 256 x 256 tiles, 7: 384 x 192, 8: 192 x 384):
    # fp16 operands, and the accumulate flag of the batch-summing mode across two micro-batches
    rng = np.random.default_rng(77)
    B, T, P, D = 4, 100, 264, 520
    X16 = rng.standard_normal((B, T, P)).astype(np.float16)
    dY16 = (rng.standard_normal((B, T, D)) * 0.05 * (10.0 ** rng.uniform(-1, 1, size=(B, 1, 1)))).astype(np.float16)
    want = O.linear_dp_grad(X16.astype(np.float32), dY16.astype(np.float32), 1.0, 0.0, 9, 2)
    check_case(X16, dY16, 1.0, 1.0, 9, 2, "f16", schedule, tile=tile, oracle=want)
    out = torch.full((D, P), float("nan"), device=DEV)
    with env(FLASHDP_TILE=tile):
        for k, (a0, a1) in enumerate([(0, 3), (3, 4)]):
            L = [dict(X=to_device(X16[a0:a1]), dY=to_device(dY16[a0:a1]), d_in=P, d_out=D, C=1.0, sigma=0.0, seed=9, layer=2,
                      out_grad=out, out_norms=None)]
            F.flashdp_block_dp_grad_micro(L, a1 - a0, T, F.F16, schedule, accumulate=(k > 0), add_noise=(k == 1))
    torch.cuda.synchronize()
    assert rel_fro(out.cpu().numpy(), want[0]) <= tight_tol("f16", schedule)


def test_fp32_matrix_core_and_generic_kernels_agree():
    # the same fp32 problem through the fp32 matrix-core kernel and (FLASHDP_TILE=-1) the generic kernel
    rng = np.random.default_rng(12)
    B, T, P, D = 3, 90, 260, 388
    X = rng.standard_normal((B, T, P)).astype(np.float32)
    dY = (rng.standard_normal((B, T, D)) * 0.02 * np.array([0.1, 1, 10], np.float32)[:, None, None]).astype(np.float32)
    want, wn = O.linear_dp_grad(X, dY, 1.0, 0.0, 2, 0)
    for schedule in ("scratch", "twopass"):
        a = run_layer(X, dY, 1.0, 0.0, 2, 0, schedule)
        b = run_layer(X, dY, 1.0, 0.0, 2, 0, schedule, tile=-1)
        for got in (a, b):
            assert rel_fro(got[0], want) <= 5e-5 and np.max(np.abs(got[1] - wn) / wn) <= 1e-4
        assert rel_fro(a[0], b[0].astype(np.float64)) <= 1e-5
    dX, ddY = to_device(X), to_device(dY)
    plain = torch.full((D, P), float("nan"), device=DEV)
    F.flashdp_plain_grad(dX, ddY, B, T, P, D, F.F32, plain)
    torch.cuda.synchronize()
    ref = dY.reshape(B * T, D).astype(np.float64).T @ X.reshape(B * T, P).astype(np.float64)
    assert rel_fro(plain.cpu().numpy(), ref) <= 5e-6


def test_fp16_inputs_with_large_gradients_do_not_overflow_the_scratch():
    # |G| far beyond fp16's largest finite value: the scratch must not turn it into inf
    rng = np.random.default_rng(4)
    B, T, P, D = 2, 64, 128, 136
    X = (rng.standard_normal((B, T, P)) * 200).astype(np.float16)
    dY = (rng.standard_normal((B, T, D)) * 200).astype(np.float16)
    want, wn = O.linear_dp_grad(X.astype(np.float32), dY.astype(np.float32), 1.0, 0.0, 0)
    assert np.max(np.abs(O.per_sample_gradient(X[0].astype(np.float32), dY[0].astype(np.float32)))) > 65504
    for schedule in ("scratch", "twopass"):
        got, gn, _ = run_layer(X, dY, 1.0, 0.0, 0, 0, schedule)
        assert np.all(np.isfinite(got)) and rel_fro(got, want) <= 4e-3
        assert np.max(np.abs(gn - wn) / wn) <= 1e-4


@pytest.mark.parametrize("schedule", ["scratch", "twopass"])
def test_twenty_runs_are_bit_identical(schedule):
    # every reduction has a fixed order (no atomics), so run-to-run differences would mean a race
    base = W.WORKLOADS["gpt2_small_mlp_up"]
    w = W.scaled_down(base, B=5, T=200, dims=[(520, 776)])
    X, dY = W.make_layer(w, 0)
    first = run_layer(X, dY, 1.0, 1.0, 3, 2, schedule)
    for _ in range(19):
        again = run_layer(X, dY, 1.0, 1.0, 3, 2, schedule)
        assert np.array_equal(first[0], again[0]) and np.array_equal(first[1], again[1])


@pytest.mark.parametrize("schedule", ["scratch", "twopass"])
def test_large_shape_kernel_is_bit_repeatable_and_matches_the_register_staged_one(schedule):
    # a shape big enough for the default path to pick the direct-to-LDS kernel (1024 work items of 256 x 256):
    # ten runs bit-identical (its loads and LDS reads are waited for by hand: a missed wait would show as run-to-run
    # noise), and the same numbers as the register-staged kernel up to the order of the additions
    rng = np.random.default_rng(5)
    B, T, P, D = 4, 96, 4096, 4096
    X = W.float32_to_bf16_bits(rng.standard_normal((B, T, P)).astype(np.float32))
    dY = W.float32_to_bf16_bits((rng.standard_normal((B, T, D)) * 0.01).astype(np.float32))
    first = run_layer(X, dY, 1.0, 0.0, 3, 2, schedule)
    for _ in range(9):
        again = run_layer(X, dY, 1.0, 0.0, 3, 2, schedule)
        assert np.array_equal(first[0], again[0]) and np.array_equal(first[1], again[1])
    assert F.flashdp_last_kernel() == "gemm_mfma_dma16_kernel"
    # the 32x32x16 form of the direct-to-LDS kernel has the accumulator layout of the register-staged kernel: the same
    # bits.  The default kernel's products and sums over the reduction index come out bit-identical too (the plain
    # gradient of the two forms is), but a lane holds other elements of the tile, so the tile's square sum is added up
    # in another order: a norm, and with it a clip factor, can differ in the last place
    wide = run_layer(X, dY, 1.0, 0.0, 3, 2, schedule, tile=6)
    staged = run_layer(X, dY, 1.0, 0.0, 3, 2, schedule, tile=4)
    assert np.array_equal(wide[1], staged[1])
    assert np.array_equal(wide[0], staged[0]) or rel_fro(wide[0], staged[0].astype(np.float64)) <= 1e-6
    assert np.allclose(first[1], staged[1], rtol=1e-6, atol=0) and rel_fro(first[0], staged[0].astype(np.float64)) <= 2e-6
    want, wn = O.linear_dp_grad(X, dY, 1.0, 0.0, 3, 2)
    assert np.max(np.abs(first[1] - wn) / wn) <= 1e-4
    assert rel_fro(first[0], want) <= tight_tol("bf16", schedule)


def _medium_shapes(n, seed):
    rng = np.random.default_rng(seed)
    shapes = [(1, 1, 8, 8), (2, 31, 264, 520), (1, 129, 776, 8), (3, 640, 1032, 1544)]
    shapes += [(int(rng.integers(1, 6)), int(rng.integers(1, 700)), 8 * int(rng.integers(1, 260)), 8 * int(rng.integers(1, 260)))
               for _ in range(n)]
    return shapes


@pytest.mark.parametrize("shape", _medium_shapes(10, 77))
def test_both_matrix_core_forms_of_the_large_tile_kernel_agree(shape):
    # the 16x16x32 kernel (hand-written main loop, its own LDS layout) against the 32x32x16 one on shapes of up to
    # 2000 features and 700 tokens, ragged in every dimension, through parking + aggregation and through the plain
    # batch gradient (the batch-accumulating mode, a k-range that runs across samples): no oracle, so no size limit
    B, T, P, D = shape
    rng = np.random.default_rng(hash(shape) % (1 << 31))
    X = W.float32_to_bf16_bits(rng.standard_normal((B, T, P)).astype(np.float32))
    dY = W.float32_to_bf16_bits((rng.standard_normal((B, T, D)) * 0.02 * (10.0 ** rng.uniform(-1, 1, size=(B, 1, 1)))).astype(np.float32))
    a = run_layer(X, dY, 1.0, 0.0, 5, 1, "scratch", tile=9)
    b = run_layer(X, dY, 1.0, 0.0, 5, 1, "scratch", tile=6)
    assert np.allclose(a[1], b[1], rtol=2e-6, atol=0)
    scale = float(np.sqrt(np.mean(b[0].astype(np.float64) ** 2))) + 1e-30
    assert np.max(np.abs(a[0].astype(np.float64) - b[0])) <= 2.0 ** -7 * float(np.max(np.abs(b[0]))) + 1e-6 * scale   # at most a last place of the parked bf16
    assert rel_fro(a[0], b[0].astype(np.float64)) <= 1e-4
    two = [run_layer(X, dY, 1.0, 0.0, 5, 1, "twopass", tile=t) for t in (9, 6)]
    assert np.allclose(two[0][1], two[1][1], rtol=2e-6, atol=0) and rel_fro(two[0][0], two[1][0].astype(np.float64)) <= 2e-6
    outs = []
    for t in (9, 6):
        out = torch.full((D, P), float("nan"), device=DEV)
        with env(FLASHDP_TILE=t):
            F.flashdp_plain_grad(to_device(X), to_device(dY), B, T, P, D, F.BF16, out)
        torch.cuda.synchronize()
        outs.append(out.cpu().numpy())
    assert np.all(np.isfinite(outs[0])) and np.array_equal(outs[0], outs[1])     # the contraction itself: bit for bit


def _random_shapes(n, seed):
    rng = np.random.default_rng(seed)
    return [(int(rng.integers(1, 6)), int(rng.integers(1, 300)), 8 * int(rng.integers(1, 76)), 8 * int(rng.integers(1, 76)))
            for _ in range(n)]


@pytest.mark.parametrize("shape", _random_shapes(12, 2024))
@pytest.mark.parametrize("tile", [4, 6, 7, 8, 9])
def test_random_shapes_both_kernel_families(shape, tile):
    # seeded random (B, T, d_in, d_out) with ragged tiles in every dimension, through the register-staged and the
    # direct-to-LDS kernels (6: 256 x 256 tiles, 7: 384 x 192, 8: 192 x 384, 9: 256 x 256 on the 16x16x32 instruction);
    # scratch schedule (norm + spill +
    # aggregation) and the plain batch gradient
    B, T, P, D = shape
    base = W.WORKLOADS["gpt2_small_mlp_up"]
    w = W.scaled_down(base, B=B, T=T, dims=[(P, D)])
    X, dY = W.make_layer(w, 0)
    check_case(X, dY, 1.0, 0.7, 17, 5, "bf16", "scratch", tile=tile)
    out = torch.full((D, P), float("nan"), device=DEV)
    with env(FLASHDP_TILE=tile):
        F.flashdp_plain_grad(to_device(X), to_device(dY), B, T, P, D, F.BF16, out)
    torch.cuda.synchronize()
    want, _ = O.linear_dp_grad(X, dY, 1e30, 0.0, 0, 0)      # nothing clips: the plain batch gradient
    assert rel_fro(out.cpu().numpy(), want) <= 5e-5


@pytest.mark.parametrize("shape,kernel", [((8, 70, 768, 3072), "gemm_mfma_dma_shaped_kernel"),      # 288 items of 256 x 256, 256 of 384 x 192
                                          ((8, 70, 3072, 768), "gemm_mfma_dma_shaped_kernel"),      # the same, 192 x 384
                                          ((8, 70, 760, 3064), "gemm_mfma_dma_shaped_kernel"),      # ragged edges in both
                                          ((8, 70, 1024, 3072), "gemm_mfma_dma16_kernel")])            # 384 items either way
@pytest.mark.parametrize("schedule", ["scratch", "twopass", "explicit"])
def test_tile_shape_follows_the_number_of_rounds(shape, kernel, schedule):
    # work items of a per-sample pass are equally long: where 384 x 192 (or 192 x 384) tiles need fewer rounds of the
    # 256 compute units than 256 x 256 tiles, the library takes them
    B, T, P, D = shape
    base = W.WORKLOADS["gpt2_small_mlp_up"]
    w = W.scaled_down(base, B=B, T=T, dims=[(P, D)])
    X, dY = W.make_layer(w, 0)
    check_case(X, dY, 1.0, 0.5, 29, 3, "bf16", schedule)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert F.flashdp_last_kernel() == kernel


@pytest.mark.parametrize("shape", [(64, 40, 512, 512), (3, 2100, 1024, 776), (9, 130, 1032, 1288), (2, 4000, 776, 1024)])
@pytest.mark.parametrize("schedule", ["auto", "twopass", "ghost"])
def test_medium_shapes_default_kernel_choice(shape, schedule):
    # shapes with enough 256 x 256 work items for the default choice to be the direct-to-LDS kernel: many
    # samples, a long ragged T, ragged feature sizes
    B, T, P, D = shape
    base = W.WORKLOADS["gpt2_small_mlp_up"]
    w = W.scaled_down(base, B=B, T=T, dims=[(P, D)])
    X, dY = W.make_layer(w, 0)
    e = check_case(X, dY, 1.0, 1.0, 23, 1, "bf16", schedule)
    print(shape, schedule, e)


@pytest.mark.timeout(200)
def test_fp16_inputs_on_a_llama_sized_layer():
    # fp16 operands at Llama-7B q_proj width (the default kernel choice is the direct-to-LDS kernel), T shortened so
    # that the fp64 oracle takes seconds; values as in the workloads (X ~ N(0,1), dY ~ 1e-2 N(0,1) x per-sample scale)
    rng = np.random.default_rng(99)
    B, T, P, D = 4, 256, 4096, 4096
    X = rng.standard_normal((B, T, P)).astype(np.float16)
    dY = (rng.standard_normal((B, T, D)) * 1e-2 * (10.0 ** rng.uniform(-1, 1, size=(B, 1, 1)))).astype(np.float16)
    want = O.linear_dp_grad(X.astype(np.float32), dY.astype(np.float32), 1.0, 0.0, 31, 2)
    for schedule in ("auto", "twopass"):
        e = check_case(X, dY, 1.0, 1.0, 31, 2, "f16", schedule, oracle=want)
        print("f16 4096x4096", schedule, e)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("B,T,dims", [(70, 2, [(1032, 264), (8, 2048)]), (180, 33, [(136, 1000)]), (40, 31, [(1304, 648), (384, 384), (648, 1304)]),
                                      (300, 5, [(136, 520)] * 9), (24, 100, [(776, 1544)])])
def test_short_sequences_take_two_passes_on_small_tiles(B, T, dims, dtype):
    # ragged tiles, k-tiles of few rows, more samples than a wave has lanes, more layers than one launch takes; workspaces
    # that hold partial sums, none, and only one layer at a time; added to an earlier micro-batch; noise.  Everything is fp32:
    # about sqrt(T + B) roundings of 2^-24 a term, 1e-6 with room for the largest case; norms 1e-6.
    g = torch.Generator(device=DEV)
    g.manual_seed(B * T)
    layers, want = [], []
    for l, (P, D) in enumerate(dims):
        X = torch.randn((B, T, P), generator=g, device=DEV).to(dtype)
        dY = (torch.randn((B, T, D), generator=g, device=DEV) * 0.05 * 10 ** (2 * torch.rand((B, 1, 1), generator=g, device=DEV) - 1)).to(dtype)
        G = torch.matmul(dY.double().transpose(1, 2).contiguous(), X.double())
        n = G.flatten(1).norm(dim=1)
        want.append(((G / torch.clamp(n / (1.0 + l), min=1.0)[:, None, None]).sum(0), n))
        layers.append(dict(X=X, dY=dY, d_in=P, d_out=D, C=1.0 + l, sigma=0.0, seed=9 + l, layer=l,
                           out_grad=torch.full((D, P), float("nan"), device=DEV), out_norms=torch.full((B,), float("nan"), device=DEV)))
    code = F.dtype_code(layers[0]["X"])
    small = max(F.flashdp_workspace_bytes([L], B, T, code, "twopass") for L in layers) * 64
    for ws in (None, torch.empty((small,), dtype=torch.uint8, device=DEV), torch.empty((F.flashdp_workspace_bytes(layers, B, T, code, "scratch"),), dtype=torch.uint8, device=DEV)):
        F.flashdp_block_dp_grad(layers, B, T, code, "auto", ws)
        assert F.flashdp_last_schedule() == "twopass" and F.flashdp_last_kernel() == "gemm_tile128_kernel"
        for L, (o, n) in zip(layers, want):
            assert float((L["out_grad"] - o).norm() / o.norm()) <= 1e-6
            assert float(((L["out_norms"] - n).abs() / n).max()) <= 1e-6
    first = [L["out_grad"].clone() for L in layers]
    noisy = [dict(L, sigma=0.5) for L in layers]
    F.flashdp_block_dp_grad_micro(noisy, B, T, code, "auto", ws, accumulate=True, add_noise=True)
    for L, f, (o, n) in zip(layers, first, want):
        z = torch.empty((L["d_in"] * L["d_out"],), device=DEV)
        F.flashdp_noise_field(L["seed"], L["layer"], z.numel(), z)
        got = L["out_grad"].double() - 0.5 * L["C"] * z.view(L["d_out"], L["d_in"]).double()
        # three fp32 additions of values of up to 6 sigma C beside the sum
        assert float((got - 2 * o).abs().max()) <= 1e-6 * 2 * float(o.abs().max()) + 3 * 2.0 ** -24 * (3 * L["C"] + 2 * float(o.abs().max()))


@pytest.mark.parametrize("B,T,P,D,how", [(20, 5, 1152, 640, "scratch"), (27, 11, 2304, 256, "scratch"), (47, 16, 144, 2944, "scratch"), (16, 5, 896, 1088, "scratch"),
                                         (25, 65, 576, 2048, "twopass"), (48, 16, 768, 896, "twopass")])
def test_short_sequences_of_few_tiles_that_one_workgroup_each_would_walk_over_are_parked(B, T, P, D, how):
    # the rule, and either way's result against fp64: parked tiles are rounded to bfloat16 (2^-9 each), the rest is fp32
    g = torch.Generator(device=DEV)
    g.manual_seed(B * P)
    X, dY = torch.randn((B, T, P), generator=g, device=DEV).bfloat16(), torch.randn((B, T, D), generator=g, device=DEV).bfloat16()
    G = torch.matmul(dY.double().transpose(1, 2).contiguous(), X.double())
    want = (G / torch.clamp(G.flatten(1).norm(dim=1), min=1.0)[:, None, None]).sum(0)
    out = torch.empty((D, P), device=DEV)
    L = [dict(X=X, dY=dY, d_in=P, d_out=D, C=1.0, sigma=0.0, seed=1, layer=0, out_grad=out)]
    F.flashdp_block_dp_grad(L, B, T, F.BF16, "auto", torch.empty((F.flashdp_workspace_bytes(L, B, T, F.BF16, "auto"),), dtype=torch.uint8, device=DEV))
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert F.flashdp_last_schedule() == how
    assert float((out - want).norm() / want.norm()) <= 4e-3


@pytest.mark.parametrize("B,T,P,D", [(1600, 5, 256, 128), (2000, 65, 128, 248), (300, 40, 256, 256)])
def test_short_sequences_of_many_samples_on_few_tiles(B, T, P, D):
    # more partial sums than layers that fill the chip have (up to 64), and the sample ends with a wait (T > 64) and without; with
    # the workspace that holds all of them, fewer and none.  fp32 sums of T and B terms: 1e-6, as above
    g = torch.Generator(device=DEV)
    g.manual_seed(B)
    X = torch.randn((B, T, P), generator=g, device=DEV).bfloat16()
    dY = (torch.randn((B, T, D), generator=g, device=DEV) * 0.05 * 10 ** (2 * torch.rand((B, 1, 1), generator=g, device=DEV) - 1)).bfloat16()
    G = torch.matmul(dY.float().transpose(1, 2).contiguous(), X.float())
    n = G.flatten(1).double().norm(dim=1)
    want = torch.zeros((D, P), dtype=torch.float64, device=DEV)
    for k in range(0, B, 64):
        y = dY[k:k + 64].double() * torch.clamp(1.0 / n[k:k + 64], max=1.0)[:, None, None]
        want += y.flatten(0, 1).T.contiguous() @ X[k:k + 64].double().flatten(0, 1)
    out, norms = torch.empty((D, P), device=DEV), torch.empty((B,), device=DEV)
    L = [dict(X=X, dY=dY, d_in=P, d_out=D, C=1.0, sigma=0.0, seed=1, layer=0, out_grad=out, out_norms=norms)]
    full = F.flashdp_workspace_bytes(L, B, T, F.BF16, "auto")
    for size in (None, full, (1 << 20) + 5 * 4 * P * D, 1 << 18):
        out.fill_(float("nan"))
        F.flashdp_block_dp_grad(L, B, T, F.BF16, "auto", None if size is None else torch.empty((size,), dtype=torch.uint8, device=DEV))
        assert F.flashdp_last_schedule() == "twopass" and F.flashdp_last_kernel() == "gemm_tile128_kernel"
        assert float((out - want).norm() / want.norm()) <= 1e-6 and float(((norms - n).abs() / n).max()) <= 1e-6


FRESH_PROCESS = """
import torch, paper_2507_01154_amd as F
g = torch.Generator(device="cuda:0"); g.manual_seed(1)
def call(B, T, dims):
    g.manual_seed(B)
    Ls = [dict(X=torch.randn((B, T, P), generator=g, device="cuda:0").bfloat16(), dY=torch.randn((B, T, D), generator=g, device="cuda:0").bfloat16(),
               d_in=P, d_out=D, C=1.0, sigma=0.0, seed=1, layer=l, out_grad=torch.empty((D, P), device="cuda:0")) for l, (P, D) in enumerate(dims)]
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    F.flashdp_block_dp_grad(Ls, B, T, F.BF16, "auto")
    torch.cuda.synchronize()
    return [L["out_grad"] for L in Ls], F.flashdp_last_schedule(), free - torch.cuda.mem_get_info()[0]
small = (16, 200, [(1024, 1024)] * 4)
a, s, _ = call(*small)
assert s == "twopass", s
_, s, taken = call(64, 16, [(5120, 13824)])
assert s == "twopass" and taken < 1 << 30, (s, taken)
_, s, _ = call(4, 1024, [(4096, 4096)])
assert s == "scratch", s
b, s, _ = call(*small)
assert s == "twopass" and all(torch.equal(x, y) for x, y in zip(a, b))
"""


def test_short_sequences_give_the_same_bits_whatever_the_library_workspace_holds():
    # in a process of its own, where the library's workspace is still empty: the number of partial sums is that of the call, not
    # of what an earlier, larger call has left; and no room for parked samples is taken where none are parked (9 GB there)
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", FRESH_PROCESS], cwd=root, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("B,T,P,D", [(16, 97, 768, 760), (5, 333, 1032, 1928), (3, 40, 1480, 2056), (3, 2100, 1032, 2056), (12, 130, 1288, 1288)])
def test_parking_on_small_tiles_where_their_rounds_are_shorter(B, T, P, D, dtype):
    # layers of enough 256 x 256 tiles for the large-tile kernel that park on 128 x 128 ones; a workspace with room for no
    # more norm partials than the large tiles have is still accepted, and takes those.  Tolerances of parked tiles.
    g = torch.Generator(device=DEV)
    g.manual_seed(B * T)
    X = torch.randn((B, T, P), generator=g, device=DEV).to(dtype)
    dY = (torch.randn((B, T, D), generator=g, device=DEV) * 0.05 * 10 ** (2 * torch.rand((B, 1, 1), generator=g, device=DEV) - 1)).to(dtype)
    G = torch.matmul(dY.double().transpose(1, 2).contiguous(), X.double())
    n = G.flatten(1).norm(dim=1)
    c = 1.0 / torch.clamp(n, min=1.0)
    want, bound = (G * c[:, None, None]).sum(0), (G.abs() * c[:, None, None]).sum(0)
    out, norms = torch.empty((D, P), device=DEV), torch.empty((B,), device=DEV)
    L = [dict(X=X, dY=dY, d_in=P, d_out=D, C=1.0, sigma=0.0, seed=1, layer=0, out_grad=out, out_norms=norms)]
    code = F.dtype_code(X)
    up = lambda k: (k + 255) // 256 * 256
    least = up(4 * B) + up(4 * B * (-(-P // 256)) * (-(-D // 256))) + up(2 * B * P * D)
    full = F.flashdp_workspace_bytes(L, B, T, code, "scratch")
    for size, kernel in ((full, "gemm_tile128_kernel"), (least, "gemm_mfma_dma16_kernel")):
        out.fill_(float("nan"))
        norms.fill_(float("nan"))
        F.flashdp_block_dp_grad(L, B, T, code, "scratch", torch.empty((size,), dtype=torch.uint8, device=DEV))
        assert F.flashdp_last_schedule() == "scratch" and F.flashdp_last_kernel() == kernel
        assert float((out - want).norm() / want.norm()) <= 4e-3 and float(((norms - n).abs() / n).max()) <= 1e-4
        assert bool(torch.all((out - want).abs() <= 1e-4 * float(bound.pow(2).mean().sqrt()) + 2.0 ** -8 * bound))
    with pytest.raises(F.FlashDPError):
        F.flashdp_block_dp_grad(L, B, T, code, "scratch", torch.empty((least - 256,), dtype=torch.uint8, device=DEV))


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("B,T,P,D,schedule,tile", [(3, 70, 1536, 1920, "scratch", 9), (5, 512, 1152, 1920, "scratch", 9), (2, 45, 2176, 2304, "scratch", 9), (12, 130, 768, 2432, "scratch", 9),
                                                   (64, 16, 896, 1152, "auto", 7), (64, 16, 1024, 1152, "auto", 9), (64, 5, 1152, 1024, "auto", 9), (32, 16, 768, 3200, "auto", 9),
                                                   (16, 333, 576, 1344, "scratch", 7), (13, 40, 960, 1152, "scratch", 7), (13, 200, 1408, 1728, "scratch", 8),
                                                   (25, 16, 960, 1408, "auto", 7), (25, 16, 1472, 960, "auto", 8), (25, 65, 576, 2048, "auto", 7)])
@pytest.mark.parametrize("operand,column,value", [("X", 0, "inf"), ("X", -1, "inf"), ("dY", 300, "inf"), ("dY", -1, "-inf"), ("X", 200, "nan"), ("dY", 7, "large")])
def test_operands_that_are_not_finite_poison_on_small_tiles_what_they_poison_on_large_ones(B, T, P, D, schedule, tile, dtype, operand, column, value):
    # a sample with an infinity beside the edge of a large tile has a norm of NaN, and all of the output with it; away from one an
    # infinite norm and a factor of 0, as finite values whose squares overflow have.  Small tiles have fewer edges (sizes
    # that are odd multiples of 128) or more (odd multiples of 192, on 384 x 192 tiles).  A sample that is finite keeps its norm.
    g = torch.Generator(device=DEV)
    g.manual_seed(P + D)
    t = {"X": torch.randn((B, T, P), generator=g, device=DEV).to(dtype), "dY": torch.randn((B, T, D), generator=g, device=DEV).to(dtype)}
    if value == "large":
        t["dY"][B - 1] = 1e20 if dtype == torch.bfloat16 else 6e4
        t["X"][B - 1] = 3e18 if dtype == torch.bfloat16 else 6e4
    else:
        t[operand][B - 1, T // 2, column] = float(value)
    code = F.dtype_code(t["X"])
    res = []
    for how, forced in ((schedule, None), ("scratch", tile)):
        out, norms = torch.full((D, P), 7.0, device=DEV), torch.full((B,), 7.0, device=DEV)
        with env(FLASHDP_TILE=forced):
            F.flashdp_block_dp_grad([dict(X=t["X"], dY=t["dY"], d_in=P, d_out=D, C=1.0, sigma=0.0, seed=1, layer=0, out_grad=out, out_norms=norms)], B, T, code, how)
        torch.cuda.synchronize()
        if forced is None:
            assert F.flashdp_last_kernel() == "gemm_tile128_kernel" and F.flashdp_last_schedule() == ("twopass" if how == "auto" else "scratch")
        res.append((out, norms))
    (o, n), (ro, rn) = res
    assert torch.equal(torch.isnan(n), torch.isnan(rn)) and torch.equal(torch.isinf(n), torch.isinf(rn))
    assert torch.equal(torch.isfinite(o), torch.isfinite(ro))
    assert bool(torch.all(torch.isfinite(n[:B - 1]))) and torch.allclose(n[:B - 1], rn[:B - 1], rtol=1e-4)


@pytest.mark.parametrize("B,T,P,D", [(3, 40, 64, 128), (2, 33, 192, 64), (5, 32, 64, 240), (2, 100, 252, 64), (2, 50, 8, 1024), (3, 64, 128, 124)])
@pytest.mark.parametrize("operand,column", [("X", 0), ("X", -1), ("dY", 0), ("dY", -1)])
def test_infinities_in_thin_fp32_layers_poison_what_they_poison_on_64_by_64_tiles(B, T, P, D, operand, column):
    # layers planned on the generic kernel's tiles that park on 128 x 128 ones, split into bfloat16 parts: a dimension of an odd multiple
    # of 64 has no edge there that an infinity could meet zeros beyond
    g = torch.Generator(device=DEV)
    g.manual_seed(P + D)
    t = {"X": torch.randn((B, T, P), generator=g, device=DEV), "dY": torch.randn((B, T, D), generator=g, device=DEV)}
    t[operand][B - 1, T // 2, column] = float("inf")
    res = []
    for tile in (None, -1):
        out, norms = torch.full((D, P), 7.0, device=DEV), torch.full((B,), 7.0, device=DEV)
        with env(FLASHDP_TILE=tile):
            F.flashdp_block_dp_grad([dict(X=t["X"], dY=t["dY"], d_in=P, d_out=D, C=1.0, sigma=0.0, seed=1, layer=0, out_grad=out, out_norms=norms)], B, T, F.F32, "scratch")
        torch.cuda.synchronize()
        assert F.flashdp_last_kernel() == ("gemm_simple_kernel" if tile else "gemm_f32x3_kernel")
        res.append((out, norms))
    (o, n), (ro, rn) = res
    assert torch.equal(torch.isnan(n), torch.isnan(rn)) and torch.equal(torch.isinf(n), torch.isinf(rn))
    assert torch.equal(torch.isfinite(o), torch.isfinite(ro))
    assert torch.allclose(n[:B - 1], rn[:B - 1], rtol=1e-6)


@pytest.mark.parametrize("B,T,P,D", [(8, 64, 768, 16), (64, 100, 120, 120), (4, 100, 8, 2044), (16, 70, 96, 160)])
def test_thin_fp32_layers_run_in_the_workspace_they_are_told_to_allocate(B, T, P, D):
    # the whole batch in the size that flashdp_workspace_bytes gives, k samples at a time in the chunked one; against fp64
    g = torch.Generator(device=DEV)
    g.manual_seed(P)
    X = torch.randn((B, T, P), generator=g, device=DEV)
    dY = torch.randn((B, T, D), generator=g, device=DEV)
    G = torch.matmul(dY.double().transpose(1, 2).contiguous(), X.double())
    n = G.flatten(1).norm(dim=1)
    want = (G / torch.clamp(n, min=1.0)[:, None, None]).sum(0)
    out, norms = torch.empty((D, P), device=DEV), torch.empty((B,), device=DEV)
    L = [dict(X=X, dY=dY, d_in=P, d_out=D, C=1.0, sigma=0.0, seed=1, layer=0, out_grad=out, out_norms=norms)]
    full = F.flashdp_workspace_bytes(L, B, T, F.F32, "scratch")
    k = B // 2 + 1
    for schedule, size, chunk in (("scratch", full, B), ("auto", full, B), ("auto", F.flashdp_workspace_bytes_chunked(L, B, T, F.F32, k, 1), k)):
        out.fill_(float("nan"))
        norms.fill_(float("nan"))
        F.flashdp_block_dp_grad(L, B, T, F.F32, schedule, torch.empty((size,), dtype=torch.uint8, device=DEV))
        assert F.flashdp_last_schedule() == "scratch" and F.flashdp_last_chunk() == chunk
        assert float((out - want).norm() / want.norm()) <= 1e-6 and float(((norms - n).abs() / n).max()) <= 1e-6


@pytest.mark.parametrize("B,T,P,D", [(1, 1, 1, 1), (4, 16, 32, 32), (16, 17, 32, 32), (4, 64, 64, 64), (3, 5, 33, 31), (16, 64, 30, 34), (2, 33, 7, 64), (1, 63, 64, 3)])
def test_tiny_fp32_layers_in_one_launch(B, T, P, D):
    # edges of the 32 x 32 blocks, one sample and the most, one element; added to an earlier micro-batch, with noise; a sample
    # that is not finite.  Tolerances of fp32 sums of T and B terms.
    g = torch.Generator(device=DEV)
    g.manual_seed(B * T + P)
    X = torch.randn((B, T, P), generator=g, device=DEV)
    dY = torch.randn((B, T, D), generator=g, device=DEV) * 10 ** (2 * torch.rand((B, 1, 1), generator=g, device=DEV) - 1)
    G = torch.matmul(dY.double().transpose(1, 2).contiguous(), X.double())
    n = G.flatten(1).norm(dim=1)
    want = (G / torch.clamp(n, min=1.0)[:, None, None]).sum(0)
    out, norms = torch.full((D, P), float("nan"), device=DEV), torch.full((B,), float("nan"), device=DEV)
    L = dict(X=X, dY=dY, d_in=P, d_out=D, C=1.0, sigma=0.5, seed=3, layer=2, out_grad=out, out_norms=norms)
    z = torch.empty((D * P,), device=DEV)
    F.flashdp_noise_field(3, 2, D * P, z)
    F.flashdp_block_dp_grad_micro([L], B, T, F.F32, "scratch", accumulate=False, add_noise=False)
    assert F.flashdp_last_kernel() == "tiny_dp_kernel"
    assert float((out - want).abs().max()) <= 2e-6 * float(want.abs().max()) and torch.allclose(norms.double(), n, rtol=1e-6, atol=0)
    F.flashdp_block_dp_grad_micro([L], B, T, F.F32, "scratch", accumulate=True, add_noise=True)
    assert float((out - 2 * want - 0.5 * z.view(D, P)).abs().max()) <= 4e-6 * (float(want.abs().max()) + 1.0)
    F.flashdp_linear_dp_grad_static(X, dY, B, T, P, D, F.F32, 1.0, 0.0, 3, 2, out, norms)
    assert F.flashdp_last_kernel() == "tiny_dp_kernel" and float((out - want).abs().max()) <= 2e-6 * float(want.abs().max())
    X[B - 1, T - 1, P - 1] = float("inf")
    res = []
    for tile in (None, -1):
        with env(FLASHDP_TILE=tile):
            F.flashdp_block_dp_grad([dict(L, sigma=0.0)], B, T, F.F32, "scratch")
        torch.cuda.synchronize()
        res.append((torch.isfinite(out).clone(), torch.isnan(norms).clone()))
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])


@pytest.mark.parametrize("B,T,P,D", [(3, 4, 128, 132), (2, 33, 136, 1028), (4, 64, 36, 68), (2, 1030, 300, 260), (9, 31, 516, 128)])
@pytest.mark.parametrize("values", ["plain", "tiny", "mixed", "overflow", "infinite", "subnormal"])
def test_fp32_split_into_bfloat16_parts(B, T, P, D, values):
    # against fp64, and where values leave what the split covers (operands below 2^-109, sums or squares that overflow,
    # infinities), against the generic kernel resp. the two-pass schedule's: there both are plain fp32 sums.  Tolerances of
    # fp32 sums of T terms.
    g = torch.Generator(device=DEV)
    g.manual_seed(T * P)
    X = torch.randn((B, T, P), generator=g, device=DEV)
    dY = torch.randn((B, T, D), generator=g, device=DEV) * 10 ** (2 * torch.rand((B, 1, 1), generator=g, device=DEV) - 1)
    if values == "tiny":
        X, dY = X * 1e-36, dY * 1e30
    elif values == "mixed":
        X[:, ::3, ::5] *= 1e-35
        dY[:, 1::4] *= 1e-20
    elif values == "overflow":
        X, dY = X * 1e18, dY * 1e4
    elif values == "infinite":
        X[1, T // 2, 7] = float("inf")
    elif values == "subnormal":
        X = X * 1e-42
    L = dict(X=X, dY=dY, d_in=P, d_out=D, C=1e-3 if values != "tiny" else 1e-9, sigma=0.0, seed=1, layer=0)
    res = []
    for tile in (None, -1):
        out, norms = torch.full((D, P), 7.0, device=DEV), torch.full((B,), 7.0, device=DEV)
        two = values == "infinite" and tile is not None   # (the tiles that a ragged edge is counted in)
        with env(FLASHDP_TILE=None if two else tile):
            F.flashdp_block_dp_grad([dict(L, out_grad=out, out_norms=norms)], B, T, F.F32, "twopass" if two else "scratch")
        torch.cuda.synchronize()
        split = "gemm_f32x3_kernel" if T >= 16 else "gemm_mfma_f32_kernel"   # (fewer tokens: the fp32 instructions, which err less there)
        assert two or F.flashdp_last_kernel() == ("gemm_simple_kernel" if tile else split)
        res.append((out, norms))
    (o, n), (ro, rn) = res
    assert torch.equal(torch.isfinite(o), torch.isfinite(ro)) and torch.equal(torch.isinf(n), torch.isinf(rn)) and torch.equal(torch.isnan(n), torch.isnan(rn))
    ok = torch.isfinite(ro)
    # (subnormal: the generic kernel rounds every one of T additions to a multiple of 2^-149, half of that each; the split only
    # its result, checked against fp64 below: 2^-149 a sample and its place in the sum)
    steps = 2.0 ** -150 * (T + B) * o.numel() ** 0.5 if values == "subnormal" else 0.0
    assert float((o[ok] - ro[ok]).double().norm()) <= 2e-6 * float(ro[ok].double().norm()) + steps
    if values == "subnormal" and T >= 16:
        exact = torch.matmul(dY.double().transpose(1, 2).contiguous(), X.double()).sum(0)
        assert bool(torch.all((o - exact).abs() <= B * 2.0 ** -149 + 1e-6 * exact.abs()))
    fin = torch.isfinite(rn)
    assert torch.allclose(n[fin], rn[fin], rtol=1e-6, atol=0)
    if values in ("plain", "tiny", "mixed"):
        G = torch.matmul(dY.double().transpose(1, 2).contiguous(), X.double())
        nn = G.flatten(1).norm(dim=1)
        want = (G * torch.clamp(L["C"] / nn, max=1.0)[:, None, None]).sum(0)
        assert float((o - want).norm() / want.norm()) <= 1e-6 and float(((n - nn) / nn).abs().max()) <= 1e-6


@pytest.mark.parametrize("T", [15, 16, 31, 33, 100])
@pytest.mark.parametrize("values", ["normal", "largest parts"])
def test_fp32_products_that_stand_alone_are_rounded_once(T, values):
    # one token of the sample is not zero: every element of the gradient is one product, and as near to it as fp32 has it:
    # 2^-24, and 2^-32 for the parts' sums on the way.  "largest parts": significands that leave the largest second and third
    # parts (1 + 2^-8 - 2^-17 and neighbours), whose products must not be missing.
    g = torch.Generator(device=DEV)
    g.manual_seed(T)
    P, D = 388, 260
    X, dY = (torch.randn((1, T, n), generator=g, device=DEV) for n in (P, D))
    if values != "normal":
        X, dY = ((1.0 + 2.0 ** -8 - 2.0 ** -17 + 2.0 ** -23 * torch.randint(-40, 41, v.shape, generator=g, device=DEV)).float() for v in (X, dY))
    dY[:, torch.arange(T, device=DEV) != T // 2] = 0.0
    want = dY[0, T // 2].double()[:, None] * X[0, T // 2].double()[None, :]
    out, norms = torch.empty((D, P), device=DEV), torch.empty((1,), device=DEV)
    F.flashdp_block_dp_grad([dict(X=X, dY=dY, d_in=P, d_out=D, C=1e30, sigma=0.0, seed=1, layer=0, out_grad=out, out_norms=norms)], 1, T, F.F32, "scratch")
    assert F.flashdp_last_kernel() == ("gemm_f32x3_kernel" if T >= 16 else "gemm_mfma_f32_kernel")
    assert float(((out - want).abs() / want.abs()).max()) <= 2.0 ** -24 * (1 + 2.0 ** -7)


@pytest.mark.parametrize("small", [1e-34, 1e-38, 1e-42, 1e-45])
def test_fp32_values_next_to_nothing_leave_their_tile_as_it_is(small):
    # tails of softmax and GELU: such values take the way of all others (redone in another order of additions, the rows
    # beside them would differ in their last bits) and lose nothing themselves.  Their own row: sums of 100 products with the
    # bits that a subnormal result has (half of 2^-149 each) beside some roundings of 2^-24.
    g = torch.Generator(device=DEV)
    g.manual_seed(4)
    B, T, P, D = 1, 100, 300, 260
    X, dY = (torch.randn((B, T, n), generator=g, device=DEV) for n in (P, D))
    tiny = torch.randn((B, T), generator=g, device=DEV).sign() * small
    res = []
    for row in (torch.zeros_like(tiny), tiny):
        y = dY.clone()
        y[:, :, 7] = row
        out, norms = torch.empty((D, P), device=DEV), torch.empty((B,), device=DEV)
        F.flashdp_block_dp_grad([dict(X=X, dY=y, d_in=P, d_out=D, C=1e30, sigma=0.0, seed=1, layer=0, out_grad=out, out_norms=norms)], B, T, F.F32, "scratch")
        assert F.flashdp_last_kernel() == "gemm_f32x3_kernel"
        res.append(out)
    others = torch.arange(D, device=DEV) != 7
    assert torch.equal(res[0][others], res[1][others]) and float(res[0][7].abs().max()) == 0.0
    want, mag = tiny[0].double() @ X[0].double(), tiny[0].double().abs() @ X[0].double().abs()
    assert bool(torch.all((res[1][7] - want).abs() <= 8 * 2.0 ** -24 * mag + 2.0 ** -149))


@pytest.mark.parametrize("P,D", [(300, 260), (128, 132), (516, 256)])
def test_fp32_largest_values_beside_a_ragged_edge_stay_finite(P, D):
    # neighbouring operands whose sum overflows, in gradients that do not: against the generic kernel
    g = torch.Generator(device=DEV)
    g.manual_seed(P)
    B, T = 2, 40
    X, dY = torch.randn((B, T, P), generator=g, device=DEV), torch.randn((B, T, D), generator=g, device=DEV) * 1e-35
    X[0, 3, :] = 2e38
    X[1, 5, ::3] = -2e38
    res = []
    for tile in (None, -1):
        out, norms = torch.empty((D, P), device=DEV), torch.empty((B,), device=DEV)
        with env(FLASHDP_TILE=tile):
            F.flashdp_block_dp_grad([dict(X=X, dY=dY, d_in=P, d_out=D, C=1.0, sigma=0.0, seed=1, layer=0, out_grad=out, out_norms=norms)], B, T, F.F32, "scratch")
        assert F.flashdp_last_kernel() == ("gemm_simple_kernel" if tile else "gemm_f32x3_kernel")
        res.append((out, norms))
    (o, n), (ro, rn) = res
    assert bool(torch.all(torch.isfinite(o))) and torch.allclose(n, rn, rtol=1e-6, atol=0)
    assert float((o - ro).double().norm()) <= 2e-6 * float(ro.double().norm())


@pytest.mark.parametrize("schedule", ["scratch", "twopass", "explicit", "ghost"])
def test_nan_in_one_sample_poisons_the_output_instead_of_passing_unclipped(schedule):
    base = W.WORKLOADS["gpt2_small_mlp_up"]
    w = W.scaled_down(base, B=3, T=40, dims=[(264, 136)])
    X, dY = W.make_layer(w, 0)
    X = X.copy()
    X[1, 7, 19] = 0x7FC0                      # bfloat16 quiet NaN in sample 1
    # the paper's formula says nothing about a NaN norm (and max(1, NaN) is whatever the language makes of it); the
    # library's documented choice is the safe one for privacy: the factor is NaN and the whole output with it.
    # The other samples' norms are still the oracle's.
    _, wn = O.linear_dp_grad(X, dY, 1.0, 0.0, 1, 0)
    assert np.isnan(wn[1])
    got, gn, _ = run_layer(X, dY, 1.0, 0.0, 1, 0, schedule)
    assert np.isnan(gn[1]) and np.all(np.isfinite(gn[[0, 2]]))
    assert np.allclose(gn[[0, 2]], wn[[0, 2]], rtol=1e-4)
    assert np.all(np.isnan(got))


# ---------------------------------------------------------------------------------------------------
# bounded-memory scratch: a workspace that holds fewer samples than the batch
# ---------------------------------------------------------------------------------------------------

@pytest.mark.parametrize("chunk,slots,want_schedule", [(2, 1, "scratch"), (1, 1, "scratch"), (2, 2, "overlap"), (1, 2, "overlap")])
@pytest.mark.parametrize("tile", [None, 6])
def test_auto_goes_through_the_batch_in_chunks_when_the_workspace_is_small(chunk, slots, want_schedule, tile):
    B, T, P, D = 5, 96, 520, 776          # chunks of 2, 2, 1 (or five of 1); ragged 256-tiles
    w = W.scaled_down(W.WORKLOADS["gpt2_small_mlp_up"], B=B, T=T, dims=[(P, D)])
    X, dY = W.make_layer(w, 0)
    L = [dict(X=None, dY=None, d_in=P, d_out=D, C=1.0, sigma=1.0, seed=3, layer=2, out_grad=None)]
    need = F.flashdp_workspace_bytes_chunked(L, B, T, F.BF16, chunk, slots)
    assert slots * chunk * D * P * 2 <= need < slots * (chunk * D * P * 2 + (1 << 16))
    assert need < F.flashdp_workspace_bytes(L, B, T, F.BF16, "scratch")
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    want0, wn = O.linear_dp_grad(X, dY, 1.0, 0.0, 3, 2)
    _, _, bound = oracle_signal_and_bound(X, dY, 1.0)
    z = O.noise_field(3, 2, D * P).reshape(D, P)
    if slots == 2 and (tile is None or chunk == 1):
        want_schedule = "scratch"            # the small-shape kernel has no overlapped form, and single-sample chunks are
                                             # not worth overlapping: the two slots are used as one
    outs = {}
    for sigma in (0.0, 1.0):
        got, gn, used = run_layer(X, dY, 1.0, sigma, 3, 2, "auto", workspace=ws, tile=tile)
        assert used == want_schedule
        # two slots that end up as one (no overlapped form) hold a chunk twice as large
        assert F.flashdp_last_chunk() == (chunk if (slots == 1 or used == "overlap") else min(2 * chunk, B - 1))
        outs[sigma] = got
        assert np.max(np.abs(gn - wn) / wn) <= 1e-4
    assert rel_fro(outs[0.0], want0) <= 4e-3
    worst, k = elementwise_excess(outs[0.0], want0, bound, True)
    assert worst <= 1.0, (divmod(k, P), worst)
    d = outs[1.0].astype(np.float64) - outs[0.0].astype(np.float64)
    assert np.max(np.abs(d - z)) <= 4e-6 * max(1.0, float(np.max(np.abs(outs[0.0]))))     # noise added once, with the last chunk
    # the unchunked schedule on the same data: same norms bit for bit, same sum up to fp32 summation order
    full, fn, _ = run_layer(X, dY, 1.0, 0.0, 3, 2, "scratch", tile=tile)
    assert np.array_equal(fn, gn) and rel_fro(outs[0.0], full.astype(np.float64)) <= 1e-6


# ---------------------------------------------------------------------------------------------------
# the balanced plain gradient (comparator of the DP ratio)
# ---------------------------------------------------------------------------------------------------

@pytest.mark.parametrize("shape", [
    (3, 160, 264, 392),      # one ragged block of 4 tiles, 15 k-tiles: cut along the reduction index into 4 pieces
    (2, 100, 1544, 2056),    # 63 tiles: a full block and a ragged one, each cut
    (2, 64, 4096, 4096),     # 256 tiles = 8 blocks, one whole block per XCD: nothing is cut
    (2, 192, 5120, 5120),    # 400 tiles = 12.5 blocks, 12 k-tiles each: whole blocks and cut blocks side by side
    (1, 33, 264, 24),        # a single sample, T not a multiple of the k-tile, thin output
])
def test_balanced_plain_grad_is_the_batched_gradient(shape):
    B, T, P, D = shape
    w = W.scaled_down(W.WORKLOADS["gpt2_small_mlp_up"], B=B, T=T, dims=[(P, D)])
    X, dY = W.make_layer(w, 0)
    dX, ddY = to_device(X), to_device(dY)
    want = O.widen(dY).reshape(B * T, D).T @ O.widen(X).reshape(B * T, P)        # Eq. batched-grad
    ws = torch.empty(F.flashdp_plain_grad_balanced_workspace_bytes(), dtype=torch.uint8, device=DEV)
    outs = []
    for rep in range(2):
        out = torch.full((D, P), float("nan"), device=DEV)
        F.flashdp_plain_grad_balanced(dX, ddY, B, T, P, D, F.BF16, out, ws)
        torch.cuda.synchronize()
        outs.append(out.cpu().numpy())
    assert np.all(np.isfinite(outs[0])) and rel_fro(outs[0], want) <= 5e-6
    err = np.abs(outs[0] - want)
    assert np.max(err) <= 1e-4 * np.sqrt(np.mean(want ** 2)) + 1e-5 * np.max(np.abs(want))
    assert np.array_equal(outs[0], outs[1])                                       # fixed-order sum of the pieces
    ref = torch.full((D, P), float("nan"), device=DEV)
    F.flashdp_plain_grad(dX, ddY, B, T, P, D, F.BF16, ref)
    torch.cuda.synchronize()
    assert rel_fro(outs[0], ref.cpu().numpy().astype(np.float64)) <= 2e-6
    with pytest.raises(F.FlashDPError) as ei:
        F.flashdp_plain_grad_balanced(dX, ddY, B, T, P, D, F.BF16, out, ws[: ws.numel() // 2])
    assert ei.value.status == F.WORKSPACE_TOO_SMALL


# ---------------------------------------------------------------------------------------------------
# the single-launch, grid-synchronised schedule
# ---------------------------------------------------------------------------------------------------

@pytest.mark.parametrize("shape", SMALL + [
    (4, 100, 1160, 1320),    # 30 tiles, ragged in every dimension, T not a multiple of the k-tile: zero-padded k-tiles per sample
    (1, 96, 520, 264),       # a single sample: nothing is parked, the accumulators go straight to the output
    (9, 40, 264, 520),       # more samples than fingers on one hand
])
def test_fused_single_launch_schedule_bf16(shape):
    B, T, P, D = shape
    w = W.scaled_down(W.WORKLOADS["gpt2_small_mlp_up"], B=B, T=T, dims=[(P, D)])
    X, dY = W.make_layer(w, 0)
    e = check_case(X, dY, 1.0, 1.0, 11, 3, "bf16", "fused")
    assert e[3] == "fused" and F.flashdp_last_kernel() == "fused_dp_kernel"
    print(shape, "fused", e)


def test_fused_schedule_branches_f16_accumulation_and_repeatability():
    w = W.scaled_down(W.WORKLOADS["gpt2_small_mlp_up"], B=4, T=96, dims=[(264, 392)])
    X, dY = W.make_layer(w, 0)
    _, norms = O.linear_dp_grad(X, dY, 1.0, 0.0, 0)
    C = float(np.sort(norms)[1] * 1.5)          # two samples below the threshold, two above
    check_case(X, dY, C, 0.7, 5, 1, "bf16", "fused")
    # fp16 inputs
    rng = np.random.default_rng(17)
    X16 = rng.standard_normal((3, 70, 136)).astype(np.float16)
    dY16 = (rng.standard_normal((3, 70, 264)) * 0.05).astype(np.float16)
    want = O.linear_dp_grad(X16.astype(np.float32), dY16.astype(np.float32), 1.0, 0.0, 9, 2)
    check_case(X16, dY16, 1.0, 1.0, 9, 2, "f16", "fused", oracle=want)
    # bit-repeatable (fixed-order reductions, barrier or not)
    a = run_layer(X, dY, 1.0, 1.0, 7, 1, "fused")
    b = run_layer(X, dY, 1.0, 1.0, 7, 1, "fused")
    assert a[2] == "fused" and np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    # same norms as the scratch schedule up to the order of the partial sums (the last sample's comes from the fp32
    # accumulators instead of the parked tile)
    c = run_layer(X, dY, 1.0, 1.0, 7, 1, "scratch")
    assert np.allclose(a[1][:-1], c[1][:-1], rtol=1e-6, atol=0) and abs(a[1][-1] - c[1][-1]) <= 1e-4 * c[1][-1]
    # gradient accumulation over micro-batches through the fused schedule
    B, T, P = X.shape
    D = dY.shape[2]
    out = torch.full((D, P), float("nan"), device=DEV)
    mbs = [(X[:1], dY[:1]), (X[1:3], dY[1:3]), (X[3:], dY[3:])]
    for k, (xm, ym) in enumerate(mbs):
        nm = torch.empty((xm.shape[0],), device=DEV)
        L = [dict(X=to_device(xm), dY=to_device(ym), d_in=P, d_out=D, C=1.0, sigma=0.9, seed=21, layer=4, out_grad=out, out_norms=nm)]
        F.flashdp_block_dp_grad_micro(L, xm.shape[0], T, F.BF16, "fused", None, None, accumulate=k > 0, add_noise=k == len(mbs) - 1)
        assert F.flashdp_last_schedule() == "fused"
    torch.cuda.synchronize()
    want, _ = O.accumulated_dp_grad(mbs, 1.0, 0.9, 21, 4)
    sig, _ = O.accumulated_dp_grad(mbs, 1.0, 0.0, 21, 4)
    z = O.noise_field(21, 4, D * P).reshape(D, P)
    got = out.cpu().numpy()
    assert rel_fro(got - 0.9 * z, sig) <= 4e-3 + 1e-4 and rel_fro(got, want) <= 1e-2


def test_fused_schedule_falls_back_where_it_does_not_apply():
    # fp32 inputs and layers with more 256 x 256 tiles than the chip has compute units take the scratch schedule
    rng = np.random.default_rng(2)
    X32 = rng.standard_normal((2, 33, 50)).astype(np.float32)
    dY32 = (rng.standard_normal((2, 33, 70)) * 0.05).astype(np.float32)
    got, gn, used = run_layer(X32, dY32, 1.0, 0.0, 1, 0, "fused")
    assert used == "fused" and F.flashdp_last_kernel() != "fused_dp_kernel"
    want, wn = O.linear_dp_grad(X32, dY32, 1.0, 0.0, 1, 0)
    assert rel_fro(got, want) <= 5e-5
    L = [dict(X=None, dY=None, d_in=5120, d_out=5120, C=1.0, sigma=1.0, seed=0, layer=0, out_grad=None)]
    assert F.flashdp_workspace_bytes(L, 8, 2048, F.BF16, "fused") == F.flashdp_workspace_bytes(L, 8, 2048, F.BF16, "scratch")
    L = [dict(X=None, dY=None, d_in=4096, d_out=4096, C=1.0, sigma=1.0, seed=0, layer=0, out_grad=None)]
    assert F.flashdp_workspace_bytes(L, 4, 2048, F.BF16, "fused") < 0.8 * F.flashdp_workspace_bytes(L, 4, 2048, F.BF16, "scratch")   # one sample is never parked


def test_contraction_timeline_measurement_aid():
    B, T, P, D = 3, 256, 1160, 1320          # 30 tiles of 256 x 256 per sample, ragged
    w = W.scaled_down(W.WORKLOADS["gpt2_small_mlp_up"], B=B, T=T, dims=[(P, D)])
    X, dY = W.make_layer(w, 0)
    dX, ddY = to_device(X), to_device(dY)
    L = [dict(X=None, dY=None, d_in=P, d_out=D, C=1.0, sigma=0.0, seed=0, layer=0, out_grad=None)]
    ws = torch.empty(F.flashdp_workspace_bytes(L, B, T, F.BF16, "scratch"), dtype=torch.uint8, device=DEV)
    for park in (False, True):
        trace = torch.zeros(8 * 256, dtype=torch.int64, device=DEV)
        n = F.flashdp_contraction_timeline(dX, ddY, B, T, P, D, park, ws, trace)
        torch.cuda.synchronize()
        t = trace.cpu().numpy().reshape(-1, 8)
        assert n == 256 and int(t[:, 7].sum()) == B * 30            # one entry per (sample, tile), none for the empty grid slots
        t = t[t[:, 7] == 1]
        assert np.all(t[:, 0] <= t[:, 1]) and np.all(t[:, 1] < t[:, 2]) and np.all(t[:, 2] <= t[:, 3]) and np.all(t[:, 3] <= t[:, 4])
        assert np.all(t[:, 6] >= 1024 * (T // 32)) and np.all(t[:, 6] < 100 * 1024 * (T // 32))   # the matrix cores cannot be busier than always
        assert np.all((t[:, 5] >> 32) < 8)
    with pytest.raises(F.FlashDPError) as ei:
        F.flashdp_contraction_timeline(dX, ddY, B, T, P, D, True, ws, torch.zeros(8 * 64, dtype=torch.int64, device=DEV))
    assert ei.value.status == F.WORKSPACE_TOO_SMALL
