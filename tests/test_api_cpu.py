"""CPU-side checks of the boundary: the shared library loads, exports every symbol the header
declares, and rejects bad arguments before touching a device.  No kernel is launched here."""
import ctypes
import os
import re

import pytest
import torch

import paper_2507_01154_amd as F

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    src = open(os.path.join(ROOT, "include", "flashdp.h")).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(flashdp_[a-z0-9_]+)\s*\(", src)))


def test_library_exports_every_declared_symbol():
    names = declared_functions()
    assert "flashdp_linear_dp_grad" in names and "flashdp_block_dp_grad" in names and len(names) >= 14
    L = F.lib()
    for n in names:
        assert hasattr(L, n), n
    assert F.flashdp_version() >= 100
    assert F.status_string(0) == "ok" and "workspace" in F.status_string(F.WORKSPACE_TOO_SMALL)


def test_binding_wraps_every_entry_point_by_name():
    for n in declared_functions():
        if n in ("flashdp_status_string",):
            continue
        assert hasattr(F, n), n


A, B_, O_ = 0x10000, 0x20000, 0x30000      # fake, aligned, never dereferenced: every call below fails validation first


@pytest.mark.parametrize("args,want", [
    ((None, B_, 1, 1, 8, 8, 1.0, 0.0, 0, O_, None), F.INVALID_ARGUMENT),
    ((A, None, 1, 1, 8, 8, 1.0, 0.0, 0, O_, None), F.INVALID_ARGUMENT),
    ((A, B_, 1, 1, 8, 8, 1.0, 0.0, 0, None, None), F.INVALID_ARGUMENT),
    ((A, B_, 0, 1, 8, 8, 1.0, 0.0, 0, O_, None), F.INVALID_ARGUMENT),
    ((A, B_, 1, -3, 8, 8, 1.0, 0.0, 0, O_, None), F.INVALID_ARGUMENT),
    ((A, B_, 1, 1, 0, 8, 1.0, 0.0, 0, O_, None), F.INVALID_ARGUMENT),
    ((A, B_, 1, 1, 8, 0, 1.0, 0.0, 0, O_, None), F.INVALID_ARGUMENT),
    ((A, B_, 1, 1, 8, 8, 0.0, 0.0, 0, O_, None), F.INVALID_ARGUMENT),
    ((A, B_, 1, 1, 8, 8, -1.0, 0.0, 0, O_, None), F.INVALID_ARGUMENT),
    ((A, B_, 1, 1, 8, 8, float("nan"), 0.0, 0, O_, None), F.INVALID_ARGUMENT),
    ((A, B_, 1, 1, 8, 8, float("inf"), 0.0, 0, O_, None), F.INVALID_ARGUMENT),
    ((A, B_, 1, 1, 8, 8, 1.0, -0.5, 0, O_, None), F.INVALID_ARGUMENT),
    ((A, B_, 1, 1, 8, 8, 1.0, float("nan"), 0, O_, None), F.INVALID_ARGUMENT),
    ((A + 8, B_, 1, 1, 8, 8, 1.0, 0.0, 0, O_, None), F.MISALIGNED),
    ((A, B_ + 2, 1, 1, 8, 8, 1.0, 0.0, 0, O_, None), F.MISALIGNED),
    ((A, B_, 1, 1, 8, 8, 1.0, 0.0, 0, O_ + 4, None), F.MISALIGNED),
    ((A, B_, 1, 1 << 20, 1 << 12, 8, 1.0, 0.0, 0, O_, None), F.UNSUPPORTED_SHAPE),
    ((A, B_, 1, 4, 8, 1 << 31, 1.0, 0.0, 0, O_, None), F.UNSUPPORTED_SHAPE),
])
def test_argument_validation(args, want):
    assert F.lib().flashdp_linear_dp_grad(*args) == want


def test_context_setters_validate():
    L = F.lib()
    assert L.flashdp_set_dtype(7) == F.INVALID_ARGUMENT and L.flashdp_set_dtype(F.BF16) == F.OK
    assert L.flashdp_set_schedule(9) == F.INVALID_ARGUMENT and L.flashdp_set_schedule(0) == F.OK
    assert L.flashdp_set_workspace(None, 16) == F.INVALID_ARGUMENT
    assert L.flashdp_set_workspace(0x1008, 64) == F.MISALIGNED
    assert L.flashdp_set_workspace(None, 0) == F.OK
    assert L.flashdp_block_dp_grad(None, 1, 1, 1, 0, 0, None, 0, None) == F.INVALID_ARGUMENT
    assert L.flashdp_plain_grad(A, B_, 1, 1, 8, 8, 5, O_, None) == F.INVALID_ARGUMENT
    assert L.flashdp_noise_field(1, 0, 0, O_, None) == F.INVALID_ARGUMENT
    assert L.flashdp_box_muller(None, 4, O_, None) == F.INVALID_ARGUMENT


def test_workspace_bytes_formula():
    mk = lambda p, d: dict(X=None, dY=None, d_in=p, d_out=d, C=1.0, sigma=1.0, seed=0, layer=0, out_grad=None)
    B, T = 8, 2048
    big = F.flashdp_workspace_bytes([mk(5120, 13824), mk(5120, 5120)], B, T, F.BF16, "scratch")
    assert big >= B * 5120 * 13824 * 2 and big < B * 5120 * 13824 * 2 + (1 << 20)      # 16-bit scratch of the largest layer
    assert F.flashdp_workspace_bytes([mk(5120, 13824)], B, T, F.F32, "scratch") >= B * 5120 * 13824 * 4
    assert 0 < F.flashdp_workspace_bytes([mk(5120, 13824)], B, T, F.BF16, "twopass") < (1 << 20)
    assert F.flashdp_workspace_bytes([mk(0, 8)], B, T, F.BF16, "scratch") == 0
    # ghost-norm schedule: one partial per 128-row block pair on or above the diagonal (T = 2048: 136 per sample)
    ghost = F.flashdp_workspace_bytes([mk(5120, 5120)], B, T, F.BF16, "ghost")
    nb = (T + 127) // 128
    assert B * max(nb * (nb + 1) // 2, 400) * 4 <= ghost < (1 << 20)
    L = F.lib()
    assert L.flashdp_set_schedule(6) == F.OK and L.flashdp_set_schedule(7) == F.INVALID_ARGUMENT
    assert L.flashdp_set_schedule(0) == F.OK


@pytest.mark.parametrize("dtype", ["bf16", "f16", "fp32"])
def test_workspace_sizes_suffice_for_the_tiles_a_call_asks_room_for(dtype):
    # a call is refused, or goes through the batch in chunks, below the clip factors, the norm partials of the plan's own
    # tiles (both together are the two-pass workspace) and the parked samples; the sizing calls may give more, never less.
    # fp32 layers of fewer than 128 x 128 elements are planned on 64 x 64 tiles and park on 128 x 128 ones from T = 32 on.
    import random
    rng = random.Random(5)
    up = lambda n: (n + 255) // 256 * 256
    code, e = {"bf16": (F.BF16, 2), "f16": (F.F16, 2), "fp32": (F.F32, 4)}[dtype]
    shapes = [(8, 64, 768, 16), (64, 1024, 120, 120), (4, 1024, 8, 2044), (16, 512, 96, 160), (8, 1024, 768, 3072), (5, 333, 1096, 2312)]
    for _ in range(400):
        a = rng.choice([1, 4, 8, 64])
        shapes.append((rng.randint(1, 300), rng.choice([rng.randint(1, 64), rng.randint(32, 2048)]),
                       *(max(a, int(2 ** rng.uniform(2, 12)) // a * a) for _ in range(2))))
    for B, T, P, D in shapes:
        L = [dict(X=None, dY=None, d_in=P, d_out=D, C=1.0, sigma=1.0, seed=0, layer=0, out_grad=None)]
        least = lambda b: F.flashdp_workspace_bytes(L, b, T, code, "twopass") + up(e * b * P * D)
        for schedule in ("scratch", "auto"):
            assert F.flashdp_workspace_bytes(L, B, T, code, schedule) >= least(B), (B, T, P, D)
        assert F.flashdp_workspace_bytes(L, B, T, code, "overlap") >= 2 * least(B), (B, T, P, D)
        k = rng.randint(1, B)
        for slots in (1, 2):
            assert F.flashdp_workspace_bytes_chunked(L, B, T, code, k, slots) >= slots * least(k), (B, T, P, D, k)


@pytest.mark.parametrize("B,T,P,D,small", [
    (10, 1566, 384, 4352, False), (25, 1279, 1408, 384, False), (58, 512, 3072, 768, False),
    (11, 1891, 3768, 184, False), (13, 716, 4224, 512, False), (64, 330, 768, 3072, False),
    (4, 395, 3128, 1400, True), (4, 1024, 768, 3072, True), (5, 333, 1032, 1928, True)])
def test_operands_that_come_from_memory_count_in_the_choice_of_small_tiles(B, T, P, D, small):
    # host logic only: small tiles would be the faster ones for all of these with operands in the caches, and are the slower ones
    # for the first six with operands that come from memory.  Read off the room for norm partials.
    up = lambda n: (n + 255) // 256 * 256
    size = lambda bm, bn: up(4 * B) + up(4 * B * -(-D // bm) * -(-P // bn)) + up(2 * B * P * D)
    L = [dict(X=None, dY=None, d_in=P, d_out=D, C=1.0, sigma=1.0, seed=0, layer=0, out_grad=None)]
    got = F.flashdp_workspace_bytes(L, B, T, F.BF16, "scratch")
    assert got == size(128, 128) if small else got < size(128, 128)


def test_tile_shape_follows_the_rounds_of_equally_long_work_items(monkeypatch):
    # host logic only, read off the number of norm partials (B x tiles floats, rounded up to 256 bytes) in the two-pass
    # workspace.  Without a device 256 compute units are assumed.
    mk = lambda p, d: [dict(X=None, dY=None, d_in=p, d_out=d, C=1.0, sigma=1.0, seed=0, layer=0, out_grad=None)]

    def partial_bytes(p, d, B, T, tile=None):
        if tile is None:
            monkeypatch.delenv("FLASHDP_TILE", raising=False)
        else:
            monkeypatch.setenv("FLASHDP_TILE", str(tile))
        n = F.flashdp_workspace_bytes(mk(p, d), B, T, F.BF16, "twopass")
        monkeypatch.delenv("FLASHDP_TILE", raising=False)
        return n - 256          # the clip factors take the first 256 bytes (B <= 64)

    up = lambda n: (n + 255) // 256 * 256
    # 768 -> 3072 at B = 8: 36 tiles of 256 x 256 (288 items, two rounds) against 32 of 384 x 192 (256 items, one round)
    assert partial_bytes(768, 3072, 8, 1024, tile=6) == up(8 * 36 * 4)
    assert partial_bytes(768, 3072, 8, 1024) == up(8 * 32 * 4)
    assert partial_bytes(3072, 768, 8, 1024) == up(8 * 32 * 4)              # transposed: 192 x 384
    assert partial_bytes(768, 3072, 8, 1024, tile=7) == up(8 * 32 * 4)
    # the Llama shapes keep 256 x 256: 400 / 1080 / 256 tiles
    assert partial_bytes(5120, 5120, 8, 2048) == up(8 * 400 * 4)
    assert partial_bytes(5120, 13824, 8, 2048) == up(8 * 1080 * 4)
    assert partial_bytes(4096, 4096, 4, 2048) == up(4 * 256 * 4)
    # equal tile-rounds (1024 x 3072 at B = 8: 384 items either way): the square tile stays
    assert partial_bytes(1024, 3072, 8, 1024) == up(8 * 48 * 4)


def test_fp32_sizes_no_multiple_of_4_take_the_kernel_that_is_faster_there():
    # read off the norm partials as above (64 x 64 tiles: generic kernel, 256 x 256: matrix cores); 256 compute units
    def tiles(p, d, B, T):
        L = [dict(X=None, dY=None, d_in=p, d_out=d, C=1.0, sigma=1.0, seed=0, layer=0, out_grad=None)]
        up = lambda n: (n + 255) // 256 * 256
        n = F.flashdp_workspace_bytes(L, B, T, F.F32, "twopass") - up(4 * B)
        t = lambda b: -(-p // b) * -(-d // b)
        assert n in (up(4 * B * t(64)), up(4 * B * t(256)))
        return 64 if n == up(4 * B * t(64)) else 256

    for shape, side in (((1001, 1001, 4, 512), 64), ((257, 3001, 2, 1024), 64), ((255, 255, 64, 512), 64), ((200, 90, 64, 256), 64),
                        ((1001, 1001, 64, 16), 256), ((3001, 3001, 1, 2048), 256), ((255, 255, 128, 64), 256), ((769, 1025, 8, 333), 256),
                        ((512, 512, 8, 64), 256), ((2222, 2222, 1, 2048), 64), ((509, 255, 44, 37), 64), ((509, 255, 52, 37), 256), ((106, 2964, 50, 85), 64), ((3, 40000, 8, 64), 64)):
        assert tiles(*shape) == side, shape


def test_16_bit_sizes_no_multiple_of_8_take_the_tile_with_the_shorter_rounds():
    # read off the norm partials as above; 256 compute units
    def tiles(p, d, B, T):
        L = [dict(X=None, dY=None, d_in=p, d_out=d, C=1.0, sigma=1.0, seed=0, layer=0, out_grad=None)]
        up = lambda n: (n + 255) // 256 * 256
        n = F.flashdp_workspace_bytes(L, B, T, F.BF16, "twopass") - up(4 * B)
        t = {b: up(4 * B * -(-p // b) * -(-d // b)) for b in (64, 128, 256)}
        assert len(set(t.values())) == 3                  # the shape tells the three apart
        return next(b for b in t if t[b] == n)

    for shape, side in (((768, 10, 64, 1024), 128), ((300, 30, 64, 256), 128), ((265, 129, 130, 512), 128), ((4096, 33, 16, 1024), 128),
                        ((3001, 3001, 1, 2048), 256), ((250, 250, 200, 512), 256), ((513, 513, 64, 17), 256), ((2049, 129, 16, 100), 256),
                        ((768, 50257, 2, 1024), 256), ((1001, 1001, 4, 512), 128),
                        ((1000, 10, 256, 16), 64), ((1000, 10, 256, 17), 256), ((1000, 10, 31, 16), 128), ((1000, 65, 256, 16), 256), ((1000, 65, 256, 64), 128),
                        ((1000, 7, 256, 64), 64)):
        assert tiles(*shape) == side, shape


@pytest.mark.skipif(torch.cuda.is_available(), reason="only meaningful on a host without a GPU")
def test_no_device_is_an_error_not_a_crash():
    assert F.lib().flashdp_linear_dp_grad(A, B_, 1, 1, 8, 8, 1.0, 0.0, 0, O_, None) == F.NO_DEVICE
    assert F.lib().flashdp_noise_field(1, 0, 16, O_, None) == F.NO_DEVICE


def test_bench_refuses_more_than_one_gpu():
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert r.returncode != 0 and "one GPU" in r.stderr


def test_header_is_plain_c_and_links(tmp_path):
    import subprocess
    exe = str(tmp_path / "abi_check")
    lib_dir = os.path.join(ROOT, "paper_2507_01154_amd")
    subprocess.check_call(["gcc", "-std=c99", "-Wall", "-Werror", "-pedantic", "-o", exe, os.path.join(ROOT, "tests", "abi_check.c"),
                           "-L" + lib_dir, "-lflashdp", "-Wl,-rpath," + lib_dir])
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.split()[0] == str(F.flashdp_version())


def test_register_budget_of_the_overlapped_schedule():
    """The overlapped schedule runs two 4-wave aggregation workgroups per CU beside one resident 8-wave
    contraction workgroup.  That only fits while, per SIMD, 2 contraction waves + 2 aggregation waves stay within
    the 512 vector registers (allocated in blocks of 8); a contraction kernel grown to 218 registers measured
    4 % slower end to end for this reason alone.  Checked from the compiler's own resource report."""
    import re
    import subprocess
    import tempfile
    from paper_2507_01154_amd import build as B
    with tempfile.TemporaryDirectory() as tmp:
        cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "-O3", "-std=c++17",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "--cuda-device-only", "-c",
               "-Rpass-analysis=kernel-resource-usage", B.sources()[0], "-o", os.path.join(tmp, "api.o")]
        res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    usage, cur = {}, None
    for line in res.stderr.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            cur = m.group(1)
            usage[cur] = {}
        m = re.search(r"remark:\s+(VGPRs|AGPRs|VGPRs Spill|SGPRs Spill|ScratchSize \[bytes/lane\]): (\d+)", line)
        if m and cur:
            usage[cur][m.group(1)] = int(m.group(2))
    up8 = lambda n: (n + 7) // 8 * 8
    # MODE_SPILL, bf16 and f16, untraced, of the two 256 x 256 direct-to-LDS kernels (16x16x32: the default; 32x32x16)
    spill = [k for k in usage if ("gemm_mfma_dma_kernel" in k or "gemm_mfma_dma16_kernel" in k) and "ELi1ELi" in k and k.endswith("Lb0EEEvNS_8GemmArgsE")]
    # the streaming kernels that run beside it: the bounded-grid forms (clip factors folded in, one load in flight; and
    # the plain one used when the factors come from a launch of their own)
    agg = [k for k in usage if "aggregate16_persistent_kernel" in k or ("clip_aggregate16_kernel" in k and "Lb0EEE" in k)]
    assert len(spill) == 4 and len(agg) == 2
    # one aggregation workgroup per CU = one of its waves per SIMD beside two contraction waves
    for k in spill:
        for g in agg:
            assert 2 * up8(usage[k]["VGPRs"] + usage[k]["AGPRs"]) + up8(usage[g]["VGPRs"]) <= 512, (k, usage[k], g, usage[g])
    # and no kernel of the library spills registers to memory - except the single-launch comparison kernel, which keeps
    # a dozen values of its sample-boundary code in memory across the main loop (none is touched inside the loop)
    for k, u in usage.items():
        if "fused_dp_kernel" in k:
            assert u.get("ScratchSize [bytes/lane]", 0) <= 64, (k, u)
            continue
        assert u.get("VGPRs Spill", 0) == 0 and u.get("ScratchSize [bytes/lane]", 0) == 0, (k, u)


@pytest.mark.parametrize("dt", ["DT_BF16", "DT_F16"])
def test_the_accumulating_pass_of_short_sequences_does_not_drain_its_loads_at_every_sample(dt, tmp_path):
    """The compiler does not see the direct loads to LDS (inline assembly), but its waits for loads that it does see count
    them: a wait for all of them belongs where the clip factors of the next 64 samples are fetched, not where one
    is used.  Read off the basic blocks between the first and the last matrix instruction."""
    import re
    import subprocess
    from paper_2507_01154_amd import build as B
    src = tmp_path / "accum.hip"
    src.write_text('#include "gemm_tile128.hip.h"\n'
                   f"template __global__ void flashdp::gemm_tile128_kernel<flashdp::MODE_ACCUM, flashdp::{dt}>(const flashdp::Tile128Args);\n")
    out = tmp_path / "accum.s"
    res = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature",
                          "-Xclang", "-packed-fp32-ops", "--cuda-device-only", "-S", "-I" + B.CSRC, str(src), "-o", str(out)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    text = out.read_text()
    start = re.search(r"\n(_ZN7flashdp19gemm_tile128_kernel\w+):", text)
    blocks = re.split(r"\n(?=\.LBB\w+:|; %bb)", text[start.end():text.index(".Lfunc_end", start.end())])
    with_products = [i for i, b in enumerate(blocks) if "v_mfma" in b]
    loop = blocks[with_products[0]:with_products[-1] + 1]
    assert len(with_products) == 8 and sum("v_readlane_b32" in b for b in loop) >= 3      # (four k-tiles, each with a sample's first products)
    full = [b for b in loop if re.search(r"s_waitcnt[^\n]*vmcnt\(0\)", b)]
    # where the factors are fetched, and in a branch of its own for longer sequences
    fetch, own = [b for b in full if "global_load" in b], [b for b in full if "global_load" not in b]
    assert len(fetch) >= 3 and all("v_readlane" not in b and "v_mfma" not in b for b in own)
