"""Kernels at the edges of their launch plans (tile remainders, register passes, segment counts), against the oracle or
plain torch.  Integer results are compared exactly; tolerances of the others are derived where they are stated."""
import numpy as np
import pytest
import torch

pytestmark = [pytest.mark.gpu]


@pytest.mark.parametrize("tiles,gh,gw,w", [
    (1, 1, 1, 1), (1, 7, 9, 2), (1, 8, 8, 3), (1, 5, 13, 0),       # 1, 63, 64, 65 tokens: around one 64-token run
    (1, 31, 33, 4), (1, 32, 32, 5), (1, 25, 41, 2),                # 1023, 1024, 1025: around one pass of the workgroup
    (1, 63, 65, 7), (1, 64, 64, 3), (1, 17, 241, 2),               # 4095, 4096, 4097: the last pass kept in registers
    (2, 64, 64, 2), (1, 90, 91, 8),                                # beyond it, windows recomputed when placing
    (3, 16, 16, 9), (1, 20, 20, 17),                               # 243 and 289 windows: across the 64-window steps
])
def test_window_partition_around_its_passes(tiles, gh, gw, w):
    import paper_2605_00789_amd as L
    from oracle import lightkv_oracle as O
    n = tiles * gh * gw
    batch = 2
    h_cu = np.array([0, n, 2 * n], dtype=np.int32)
    pos = np.tile(np.arange(n, dtype=np.int32), batch)
    wps = 1 if w == 0 else tiles * w * w
    wo = torch.full((batch * wps + 1,), -7, dtype=torch.int32, device="cuda")
    wt = torch.full((batch * n,), -7, dtype=torch.int32, device="cuda")
    L.lightkv_build_windows(batch, h_cu, torch.from_numpy(h_cu).cuda(), torch.from_numpy(pos).cuda(), tiles, gh, gw, w, wo, wt)
    ro, rt = O.build_windows(pos, h_cu, tiles, gh, gw, w)
    np.testing.assert_array_equal(wo.cpu().numpy(), ro)
    np.testing.assert_array_equal(wt.cpu().numpy(), rt)


@pytest.mark.parametrize("dtype,d", [("bf16", 96), ("bf16", 1088), ("f32", 128)])
@pytest.mark.parametrize("gh,gw", [(1, 2), (5, 13), (6, 11), (8, 16), (3, 43), (10, 13), (12, 16), (1, 193), (4, 65), (15, 26)])
def test_one_window_around_the_column_tiles_of_the_epilogue(gh, gw, dtype, d):
    """One window of 2, 65, 66, 128, 129, 130, 192, 193, 260 and 390 tokens: one to seven column tiles of 32 B nodes,
    whole and partial, on the small-tile path; every stage against the oracle at the protocol's tolerances."""
    from workloads import make_custom
    from parity import check_workload
    n = gh * gw
    wl = make_custom(name="window_%d" % n, seed=n, dtype=dtype, batch=2, grid_h=gh, grid_w=gw, text_lens=(5, 33), d=d,
                     heads=d // 32, head_dim=32, n_c=12, structure="iid", windows_per_axis=(0,), targets=(n - max(1, n // 5),))
    check_workload(wl)
