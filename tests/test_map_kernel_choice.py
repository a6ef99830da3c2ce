"""Host-only: which kernel a bf16 call at head dimension 128 takes, at the edges
of the rules on heads, layers and tokens."""

import pytest


@pytest.mark.parametrize("L_t,H,T,k,kernel", [
    (64, 8, 1, 4, "map_ks2_kernel"),
    (64, 8, 1, 2, "map_ks2_kernel"),
    (15, 8, 4096, 4, "map_w_kernel"),        # too few layers
    # few or odd heads: token segments of at least 20 tiles per CU and unit
    (80, 1, 16384, 4, "map_ks2_kernel"),
    (32, 1, 5120, 4, "map_ks2_kernel"),
    (32, 1, 5112, 4, "map_w_kernel"),
    (32, 12, 1280, 2, "map_ks2_kernel"),     # 12 heads: two segments
    (32, 12, 1278, 2, "map_w_kernel"),
    (36, 3, 4096, 3, "map_w_kernel"),
    # segments over two layer groups, three (k = 2, 4), more
    (40, 1, 16384, 3, "map_ks_kernel"),
    (56, 1, 16384, 4, "map_ks2_kernel"),
    (56, 1, 16384, 3, "map_w_kernel"),
    (60, 1, 16384, 4, "map_w_kernel"),
    (63, 1, 65536, 2, "map_w_kernel"),
    (63, 8, 16384, 2, "map_ks2_kernel"),     # whole heads per XCD
    # short calls at k = 1 and 3
    (36, 8, 1024, 3, "map_w_kernel"),
    (36, 8, 1025, 3, "map_ks_kernel"),
    (64, 8, 511, 3, "map_ks_kernel"),
    (64, 8, 512, 3, "map_w_kernel"),
    (16, 8, 64, 3, "map_ks_kernel"),
    (36, 8, 512, 1, "map_w_kernel"),
    (36, 8, 513, 1, "map_ks_kernel"),
    (64, 8, 512, 1, "map_ks_kernel"),
    (64, 8, 8192, 5, "map_kernel"),
    # planes of 4 GiB and more, whose offsets the k-split kernels cannot hold
    (16, 8, 20_000_000, 4, "map_sweep_kernel"),
    (16, 1, 16_000_000, 4, "map_ks2_kernel"),
    (16, 1, 20_000_000, 4, "map_w_kernel"),
    (40, 3, 17_000_000, 3, "map_w_kernel"),
])
def test_choice(L_t, H, T, k, kernel, monkeypatch):
    from paper_2608_03893_amd import kvx
    monkeypatch.delenv("KVX_KERNEL", raising=False)
    assert kvx.map_kernel_name(kvx.Dims(L_s=40, L_t=L_t, H=H, T=T, d=128, k=k)) == kernel
