"""Maps read as given by the bf16 kernels: the packed images that an unflagged
call leaves behind serve a later flagged call, and token segments (head counts
that do not divide over the XCDs) leave no token out."""

import numpy as np
import pytest
import torch

from paper_2608_03893_amd import synth
from _parity import TOL, assert_parity, np32, oracle_rows, run_gpu, sample_tokens

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
Q = synth.CONFIGS["qwen3_14b_32b"]
I1 = synth.rope_dict(1e6, style=1)

CASES = {
    "ks2_k4": (Q.replace(L_s=9, L_t=22, T=300), "map_ks2_kernel"),
    "ks2_k2_interleaved_odd_layers": (Q.replace(L_s=9, L_t=17, k=2, T=40, rope_src=I1, rope_tgt=I1),
                                      "map_ks2_kernel"),
    "ks_k3": (Q.replace(L_s=9, L_t=19, k=3, T=513), "map_ks_kernel"),
    "ks_k1_interleaved": (Q.replace(L_s=9, L_t=16, k=1, T=5, rope_src=I1, rope_tgt=I1), "map_ks_kernel"),
    "w_k4": (Q.replace(L_s=9, L_t=3, H=3, T=600), "map_w_kernel"),
    "w_k1": (Q.replace(L_s=9, L_t=2, H=1, k=1, T=17), "map_w_kernel"),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_packed_images_of_an_unflagged_call(gpu_kvx, name, monkeypatch):
    cfg, kernel = CASES[name]
    kvx = gpu_kvx
    if kernel == "map_ks_kernel":   # by default short calls at k = 1 and 3 take map_w_kernel
        monkeypatch.setenv("KVX_KERNEL", "ks")
    inp = synth.make_inputs(cfg, DEV)
    dims = kvx.Dims(L_s=cfg.L_s, L_t=cfg.L_t, H=cfg.H, T=cfg.T, d=cfg.d, k=cfg.k)
    assert kvx.map_kernel_name(dims) == kernel
    ws = torch.full((kvx.workspace_bytes(dims),), 0x7f, dtype=torch.uint8, device=DEV)
    first = run_gpu(kvx, inp, workspace=ws)
    assert_parity(np32(first), oracle_rows(inp), TOL["bf16"], name)
    inp["W_K"], inp["W_V"] = torch.zeros_like(inp["W_K"]), torch.zeros_like(inp["W_V"])
    again = run_gpu(kvx, inp, workspace=ws, flags=kvx.FLAG_WEIGHTS_PACKED)
    assert torch.equal(first.view(torch.int16), again.view(torch.int16))


@pytest.mark.parametrize("H,T,k,L_t", [(1, 5120, 4, 32), (1, 5157, 3, 32), (6, 2561, 2, 32),
                                       (12, 1330, 4, 32), (1, 8200, 2, 40)])
def test_token_segments(gpu_kvx, H, T, k, L_t):
    # about the shortest segments that take the segmented plan; 40 layers: two groups
    cfg = Q.replace(L_s=6, L_t=L_t, H=H, T=T, k=k)
    kvx = gpu_kvx
    dims = kvx.Dims(L_s=cfg.L_s, L_t=cfg.L_t, H=H, T=T, d=cfg.d, k=k)
    assert kvx.map_kernel_name(dims) == ("map_ks_kernel" if k == 3 else "map_ks2_kernel")
    inp = synth.make_inputs(cfg, DEV)
    out = torch.full((cfg.L_t, 2, H, T, cfg.d), float("nan"), dtype=torch.bfloat16, device=DEV)
    run_gpu(kvx, inp, out=out)
    assert bool(torch.isfinite(out).all())
    edges = [e for s in range(1, 8) for e in (s * (T // 8), s * (T // 8) + 15, s * (T // 8) + 16)]
    tokens = sample_tokens(T, 96, 3, extra=edges)
    got = np32(out[:, :, :, torch.as_tensor(tokens, device=DEV)])
    assert_parity(got, oracle_rows(inp, tokens=tokens), TOL["bf16"], f"H{H} T{T} k{k}")


@pytest.mark.parametrize("H,T,k,L_t", [(1, 5157, 4, 32), (3, 5131, 3, 32), (6, 2561, 2, 32), (1, 8200, 1, 40)])
def test_token_segments_images_slots_second_rope(gpu_kvx, H, T, k, L_t):
    """Segmented calls with a target RoPE of their own: the images that an unflagged
    call leaves serve a flagged one, dense and slot-addressed outputs agree with
    the oracle, and rows that no slot names stay."""
    cfg = Q.replace(L_s=6, L_t=L_t, H=H, T=T, k=k, rope_src=synth.rope_dict(1e4))
    kvx = gpu_kvx
    dims = kvx.Dims(L_s=cfg.L_s, L_t=L_t, H=H, T=T, d=cfg.d, k=k)
    assert kvx.map_kernel_name(dims) == ("map_ks_kernel" if k in (1, 3) else "map_ks2_kernel")
    inp = synth.make_inputs(cfg, DEV)
    ws = torch.full((kvx.workspace_bytes(dims),), 0x7f, dtype=torch.uint8, device=DEV)
    first = run_gpu(kvx, inp, workspace=ws)
    tokens = sample_tokens(T, 96, 3, extra=[e for s in range(1, 8) for e in (s * (T // 8), s * (T // 8) + 16)])
    at = torch.as_tensor(tokens, device=DEV)
    want = oracle_rows(inp, tokens=tokens)
    assert_parity(np32(first[:, :, :, at]), want, TOL["bf16"], f"H{H} T{T} k{k} dense")

    slots = torch.arange(T - 1, -1, -1, dtype=torch.int32, device=DEV) + 3
    slots[5::9] = -1
    pool = torch.full((L_t, 2, H, T + 8, cfg.d), 7.0, dtype=torch.bfloat16, device=DEV)
    kvx.map_cache_slots(inp["src"], inp["idx"], inp["W_K"], inp["W_V"], inp["b_K"], inp["b_V"],
                        inp["rope_src"], inp["rope_tgt"], inp["positions"], slots, pool)
    kept = at[slots[at] >= 0]
    assert_parity(np32(pool[:, :, :, slots[kept].long()]), want[:, :, :, np32(slots[at]) >= 0],
                  TOL["bf16"], f"H{H} T{T} k{k} slots")
    free = torch.ones(T + 8, dtype=torch.bool, device=DEV)
    free[slots[slots >= 0].long()] = False
    assert bool((pool[:, :, :, free] == 7.0).all())

    inp["W_K"], inp["W_V"] = torch.zeros_like(inp["W_K"]), torch.zeros_like(inp["W_V"])
    again = run_gpu(kvx, inp, workspace=ws, flags=kvx.FLAG_WEIGHTS_PACKED)
    assert torch.equal(first.view(torch.int16), again.view(torch.int16))


@pytest.mark.parametrize("k,L_t,T", [(4, 82, 300), (2, 65, 40), (3, 83, 130), (1, 129, 70)])
def test_packed_images_of_several_layer_groups(gpu_kvx, k, L_t, T, monkeypatch):
    # 64 layers and a remainder in one or more groups
    cfg = Q.replace(L_s=9, L_t=L_t, T=T, k=k)
    kvx = gpu_kvx
    if k in (1, 3):
        monkeypatch.setenv("KVX_KERNEL", "ks")
    dims = kvx.Dims(L_s=cfg.L_s, L_t=L_t, H=cfg.H, T=T, d=cfg.d, k=k)
    assert kvx.map_kernel_name(dims) == ("map_ks_kernel" if k in (1, 3) else "map_ks2_kernel")
    inp = synth.make_inputs(cfg, DEV)
    ws = torch.full((kvx.workspace_bytes(dims),), 0x7f, dtype=torch.uint8, device=DEV)
    first = run_gpu(kvx, inp, workspace=ws)
    layers = [0, 1, 62, 63, 64, L_t - 2, L_t - 1]
    assert_parity(np32(first[layers]), oracle_rows(inp, layers=layers), TOL["bf16"], f"k{k} L_t{L_t}")
    inp["W_K"], inp["W_V"] = torch.zeros_like(inp["W_K"]), torch.zeros_like(inp["W_V"])
    again = run_gpu(kvx, inp, workspace=ws, flags=kvx.FLAG_WEIGHTS_PACKED)
    assert torch.equal(first.view(torch.int16), again.view(torch.int16))
