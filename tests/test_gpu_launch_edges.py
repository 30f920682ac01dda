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


@pytest.mark.parametrize("dtype,d,n,tail", [
    ("bf16", 32, 70, 0), ("bf16", 512, 70, 3), ("bf16", 544, 71, 2), ("bf16", 2048, 33, 5), ("bf16", 2560, 33, 1),
    ("bf16", 4096, 65, 9), ("bf16", 4160, 30, 2), ("bf16", 5120, 37, 6), ("bf16", 8192, 20, 1), ("bf16", 8704, 20, 3),
    ("f32", 128, 40, 2), ("f32", 1280, 40, 2), ("f32", 5120, 21, 4),
    ("bf16", 4096, 31, 1), ("bf16", 6144, 25, 3), ("f32", 2048, 30, 1), ("f32", 3072, 30, 2), ("f32", 4608, 29, 3),   # 2 to 4 segments, squared norms across them
    ("bf16", 4096, 6000, 40),          # beyond 128 MB: whole rows per wave, nontemporal stores
    ("bf16", 2816, 6140, 4), ("bf16", 2816, 6141, 4),   # the last launch of short segments with squared norms, the first without
])
def test_merge_over_the_row_segments(dtype, d, n, tail):
    """One to five segments per row, whole and partial, with and without rows behind the vision span and squared norms;
    groups of one, two, three and more than 64 sources.  Reference: the merge in float64.  The kernel rounds once on
    store (bf16 keeps 8 significant bits: half a unit in the last place is at most 2^-8 of a value) after fp32 arithmetic with at most 80 terms (80 x 2^-24 = 5e-6 of the
    largest row); squared norms are those of the rows as stored, summed in fp32 over d terms."""
    import paper_2605_00789_amd as L
    g = torch.Generator(device="cuda").manual_seed(d + n)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    X, K, V = (torch.randn(n + tail, d, generator=g, device="cuda").to(tdt) for _ in range(3))
    rng = np.random.default_rng(d)
    dst = np.full(n, -1)
    leave = rng.permutation(n)[:n // 3]
    dst[leave] = -2
    stay = np.flatnonzero(dst == -1)
    for k, a in enumerate(leave):
        dst[a] = stay[0] if k < 70 and n > 300 else stay[k // 3 % len(stay)]
    gone = dst >= 0
    order = np.argsort(dst[gone], kind="stable")
    src = np.flatnonzero(gone)[order].astype(np.int32)
    new_index = np.where(gone, -1, np.cumsum(~gone) - 1).astype(np.int32)
    offsets = np.concatenate([[0], np.cumsum(np.bincount(dst[gone], minlength=n))]).astype(np.int32)
    xi = (rng.gamma(2.0, 1.0, n) + 1e-3).astype(np.float32)
    out = int((~gone).sum())
    h_cu = np.array([0, n], dtype=np.int32)
    cu = torch.from_numpy(h_cu).cuda()
    prob = L.Problem(batch=1, d=d, heads=d // 32, head_dim=32, dtype=dtype, h_cu_vis=h_cu, cu_vis=cu)
    outs = [torch.full((out + tail, d), 7.0, dtype=tdt, device="cuda") for _ in range(3)]
    sq = torch.empty(out, device="cuda")
    pos = torch.arange(n + tail, dtype=torch.int32, device="cuda")
    pos_out = torch.empty(out + tail, dtype=torch.int32, device="cuda")
    L.lightkv_aggregate_compact(prob, torch.from_numpy(new_index).cuda(), torch.from_numpy(offsets).cuda(),
                                torch.from_numpy(src).cuda(), torch.from_numpy(xi).cuda(), X, K, V, pos, *outs, pos_out,
                                x_sqnorm_out=sq, tail_rows=tail, cu_vis_out=torch.tensor([0, out], dtype=torch.int32, device="cuda"))
    w = torch.from_numpy(xi).cuda().double()
    a, b = torch.from_numpy(np.flatnonzero(gone)).cuda(), torch.from_numpy(dst[gone]).cuda()
    keep = torch.from_numpy(~gone).cuda()
    for y, o in zip((X, K, V), outs):
        y64 = y.double()
        num, den = w[:, None] * y64[:n], w.clone()
        num.index_add_(0, b, w[a][:, None] * y64[a])
        den.index_add_(0, b, w[a])
        want = torch.cat([(num / den[:, None])[keep], y64[n:]])
        err = (o.double() - want).abs()
        bound = (2.0 ** -8 if dtype == "bf16" else 0.0) * want.abs() + 6e-6 * want.abs().max()
        assert bool((err <= bound).all()), float((err - bound).max())
    want_sq = outs[0][:out].double().square().sum(1)
    assert bool(((sq.double() - want_sq).abs() <= 1e-6 * want_sq).all())
    assert torch.equal(pos_out, torch.cat([pos[:n][keep], pos[n:]]))


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 2048), ("bf16", 4096), ("bf16", 5120), ("f32", 1024), ("f32", 2560)])
def test_groups_of_any_number_of_sources(dtype, d):
    """Groups of 1 to 9 sources (the later ones come in pairs), and of 63 to 66 around the sources whose weights a wave keeps,
    in place and with the compaction.  Reference and bound as in test_merge_over_the_row_segments."""
    import paper_2605_00789_amd as L
    sizes = [1, 2, 3, 4, 5, 6, 7, 8, 9, 63, 64, 65, 66]
    n = sum(sizes) + len(sizes)
    rng = np.random.default_rng(d)
    perm = rng.permutation(n)
    dst, at = np.full(n, -1), len(sizes)
    for k, m in enumerate(sizes):
        dst[perm[at:at + m]] = perm[k]
        at += m
    gone = dst >= 0
    src = np.flatnonzero(gone)[np.argsort(dst[gone], kind="stable")].astype(np.int32)
    new_index = np.where(gone, -1, np.cumsum(~gone) - 1).astype(np.int32)
    offsets = np.concatenate([[0], np.cumsum(np.bincount(dst[gone], minlength=n))]).astype(np.int32)
    xi = (rng.gamma(2.0, 1.0, n) + 1e-3).astype(np.float32)
    g = torch.Generator(device="cuda").manual_seed(d)
    X, K, V = (torch.randn(n, d, generator=g, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32) for _ in range(3))
    h_cu = np.array([0, n], dtype=np.int32)
    prob = L.Problem(batch=1, d=d, heads=d // 32, head_dim=32, dtype=dtype, h_cu_vis=h_cu, cu_vis=torch.from_numpy(h_cu).cuda())
    off_d, src_d, xi_d = torch.from_numpy(offsets).cuda(), torch.from_numpy(src).cuda(), torch.from_numpy(xi).cuda()
    keep = torch.from_numpy(~gone).cuda()
    outs = [torch.full((len(sizes), d), 7.0, dtype=X.dtype, device="cuda") for _ in range(3)]
    pos = torch.arange(n, dtype=torch.int32, device="cuda")
    L.lightkv_aggregate_compact(prob, torch.from_numpy(new_index).cuda(), off_d, src_d, xi_d, X, K, V, pos, *outs, pos[:len(sizes)].clone())
    in_place = [t.clone() for t in (X, K, V)]
    L.lightkv_aggregate(prob, off_d, src_d, xi_d, *in_place)
    a, b = torch.from_numpy(np.flatnonzero(gone)).cuda(), torch.from_numpy(dst[gone]).cuda()
    w = xi_d.double()
    for y, o, p in zip((X, K, V), outs, in_place):
        y64 = y.double()
        num, den = w[:, None] * y64, w.clone()
        num.index_add_(0, b, w[a][:, None] * y64[a])
        den.index_add_(0, b, w[a])
        want = (num / den[:, None])[keep]
        bound = (2.0 ** -8 if dtype == "bf16" else 0.0) * want.abs() + 6e-6 * want.abs().max()
        assert bool(((o.double() - want).abs() <= bound).all())
        assert torch.equal(p[keep], o)
        assert torch.equal(p[~keep], y[~keep])


@pytest.mark.parametrize("dtype,d,n,tail", [("bf16", 64, 30, 3), ("bf16", 4096, 30, 0), ("bf16", 4160, 31, 2), ("bf16", 8704, 30, 3),
                                            ("bf16", 4224, 2100, 5), ("f32", 4352, 33, 1)])
def test_rows_in_one_wave_or_several(dtype, d, n, tail):
    """lightkv_compact takes a row in one wave's passes and must move its bytes unchanged, rows behind the vision span
    included; lightkv_aggregate followed by it gives the bits of lightkv_aggregate_compact, whatever segments each launch cuts."""
    import paper_2605_00789_amd as L
    g = torch.Generator(device="cuda").manual_seed(d + n)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    X, K, V = (torch.randn(n + tail, d, generator=g, device="cuda").to(tdt) for _ in range(3))
    rng = np.random.default_rng(n)
    dst = np.full(n, -1)
    leave = np.sort(rng.permutation(n)[:n // 4])
    dst[leave] = -2
    stay = np.flatnonzero(dst == -1)
    dst[leave] = rng.choice(stay, len(leave))
    gone = dst >= 0
    src = np.flatnonzero(gone)[np.argsort(dst[gone], kind="stable")].astype(np.int32)
    new_index = np.where(gone, -1, np.cumsum(~gone) - 1).astype(np.int32)
    off = np.concatenate([[0], np.cumsum(np.bincount(dst[gone], minlength=n))]).astype(np.int32)
    out, h = int((~gone).sum()), np.array([0, n], dtype=np.int32)
    p = L.Problem(batch=1, d=d, heads=d // 32, head_dim=32, dtype=dtype, h_cu_vis=h, cu_vis=torch.from_numpy(h).cuda())
    new_index, off, src = (torch.from_numpy(a).cuda() for a in (new_index, off, src))
    xi, pos = torch.rand(n, generator=g, device="cuda") + 0.1, torch.arange(n + tail, dtype=torch.int32, device="cuda")
    cu_out = torch.tensor([0, out], dtype=torch.int32, device="cuda")
    kw = dict(tail_rows=tail, cu_vis_out=cu_out)
    rows = torch.cat([torch.from_numpy(np.flatnonzero(~gone)).cuda(), torch.arange(n, n + tail, device="cuda")])

    def fresh():
        return [torch.full((out + tail, d), 7.0, dtype=tdt, device="cuda") for _ in range(3)] + [torch.empty(out + tail, dtype=torch.int32, device="cuda")]
    a = fresh()
    L.lightkv_compact(p, new_index, X, K, V, pos, *a, **kw)
    for got, y in zip(a, (X, K, V, pos)):
        assert torch.equal(got, y[rows])
    b, c = fresh(), fresh()
    L.lightkv_aggregate_compact(p, new_index, off, src, xi, X, K, V, pos, *b, **kw)
    m = [t.clone() for t in (X, K, V)]
    L.lightkv_aggregate(p, off, src, xi, *m)
    L.lightkv_compact(p, new_index, *m, pos, *c, **kw)
    for x, y in zip(b, c):
        assert torch.equal(x, y)


@pytest.mark.parametrize("batch,gh,gw,w,d", [
    (1, 4, 4, 2, 128), (2, 8, 8, 2, 64), (1, 16, 16, 4, 1088),     # windows of 4, 16 (packed tiles) and 16 tokens
    (1, 8, 8, 0, 128), (1, 5, 13, 0, 128), (1, 12, 16, 0, 192),    # 64, 65 and 192 tokens: two, three and six tiles a side
    (3, 16, 16, 1, 128), (1, 16, 17, 0, 128), (1, 27, 27, 0, 64),  # 256, 272 and 729 tokens: both selection sizes
    (1, 32, 32, 0, 64), (16, 16, 16, 2, 64),                       # 1024 tiles of 32: beyond the small tiles
])
def test_full_pairwise_around_the_small_tiles(batch, gh, gw, w, d):
    """Every token's nearest neighbour against float64 (ties and near-ties within 1e-5 of the best, the protocol's bound
    for bf16), and the selection exactly against the visit applied to the scores the library reported."""
    import paper_2605_00789_amd as L
    from paper_2605_00789_amd import binding as B
    from oracle import lightkv_oracle as O
    n = gh * gw
    g = torch.Generator(device="cuda").manual_seed(n + d)
    X = torch.randn(16, d, generator=g, device="cuda")[torch.randint(0, 16, (batch * n,), generator=g, device="cuda")]
    X = (X + torch.rand(batch * n, 1, generator=g, device="cuda") * torch.randn(batch * n, d, generator=g, device="cuda")).bfloat16()
    X[3] = X[1]                                       # an exact copy: divergence zero
    per = 1 if w == 0 else w * w
    h = (np.arange(batch + 1) * n).astype(np.int32)
    cu = torch.from_numpy(h).cuda()
    pos = torch.arange(n, dtype=torch.int32).repeat(batch).cuda()
    i32 = dict(dtype=torch.int32, device="cuda")
    wo, wt, rem = torch.empty(batch * per + 1, **i32), torch.empty(batch * n, **i32), torch.empty(batch * per, **i32)
    L.lightkv_build_windows(batch, h, cu, pos, 1, gh, gw, w, wo, wt)
    L.lightkv_window_counts(batch, batch * per, wo, B.COUNT_RATIO, rem, rho=0.3)
    p = L.Problem(batch=batch, d=d, heads=d // 32, head_dim=32, dtype="bf16", h_cu_vis=h, cu_vis=cu, n_windows=batch * per,
                  max_window_tokens=min(n, L.lightkv_max_window_cells(1, gh, gw, w)), win_offsets=wo, win_tokens=wt,
                  win_remove=rem, match=B.MATCH_FULL_PAIRWISE)
    ws = torch.empty(L.lightkv_workspace_size(p), dtype=torch.uint8, device="cuda")
    N = batch * n
    xi, fd, dst, best = torch.ones(N, device="cuda"), torch.empty(N, device="cuda"), torch.empty(N, **i32), torch.empty(N, **i32)
    new, off, src, cu_out = torch.empty(N, **i32), torch.empty(N + 1, **i32), torch.empty(N, **i32), torch.empty(batch + 1, **i32)
    L.lightkv_score_select(p, X, None, None, xi, fd, best, dst, new, off, src, cu_out, ws, xi_mode=B.XI_GIVEN)
    fd2, best2 = torch.empty(N, device="cuda"), torch.empty(N, **i32)
    L.lightkv_score(p, X, None, None, xi, fd2, best2, ws, xi_mode=B.XI_GIVEN)
    assert torch.equal(fd, fd2) and torch.equal(best, best2)
    h_wo, h_wt, h_fd, h_best, h_dst = (t.cpu().numpy() for t in (wo, wt, fd, best, dst))
    x64 = X.double()
    x64 = x64 / x64.norm(dim=1, keepdim=True)
    for k in range(batch * per):
        toks = h_wt[h_wo[k]:h_wo[k + 1]]
        t = torch.from_numpy(toks.astype(np.int64)).cuda()
        m = (1.0 - x64[t] @ x64[t].T.contiguous()).clamp_min(0).cpu().numpy()
        np.fill_diagonal(m, np.inf)
        local = {int(a): i for i, a in enumerate(toks)}
        nb = np.array([local[int(b)] for b in h_best[toks]])
        assert np.all(np.abs(h_fd[toks] - m[np.arange(len(toks)), nb]) <= 1e-5)
        assert np.all(h_fd[toks] <= m.min(1) + 1e-5)
        r, gone, kept, want = int(0.3 * len(toks) + 1e-9), set(), set(), np.full(len(toks), -1)
        for i in np.argsort(h_fd[toks], kind="stable"):
            if len(gone) < min(r, (len(toks) + 1) // 2) and i not in kept and nb[i] not in gone:
                gone.add(i)
                kept.add(nb[i])
                want[i] = toks[nb[i]]
        np.testing.assert_array_equal(h_dst[toks], want)
    np.testing.assert_array_equal(new.cpu().numpy(), O.kept_index(h_dst))


@pytest.mark.parametrize("dtype,batch,gh,gw,w,d,ties", [
    ("bf16", 1, 4, 4, 2, 64, False), ("bf16", 2, 12, 12, 3, 256, False), ("f32", 1, 14, 14, 2, 128, False),   # 4, 16, 49 tokens
    ("bf16", 1, 14, 14, 1, 96, False), ("bf16", 1, 16, 16, 1, 256, True),                    # 196 and 256: the largest in LDS
    ("bf16", 1, 17, 16, 1, 128, False), ("bf16", 2, 17, 31, 1, 64, True),                    # 272 and 527: the key matrix
    ("bf16", 9, 16, 16, 4, 64, False), ("f32", 3, 28, 28, 2, 32, True),                      # an index scan per sequence
])
@pytest.mark.parametrize("with_xi", [False, True])
def test_edge_selection_in_any_window_order(dtype, batch, gh, gw, w, d, ties, with_xi):
    """The k lowest edges of every window against the rule applied in float64 to the scores the library reports for its
    own order (exact), with windows listed in order and shuffled over the batch: the same edges either way.  `ties`:
    tokens are copies of a few rows, so that nearly every divergence is shared by many pairs."""
    import paper_2605_00789_amd as L
    from paper_2605_00789_amd import binding as B
    n, N = gh * gw, batch * gh * gw
    g = torch.Generator(device="cuda").manual_seed(n + d)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    rows = torch.randn(5 if ties else 24, d, generator=g, device="cuda")
    X = rows[torch.randint(0, rows.shape[0], (N,), generator=g, device="cuda")]
    if not ties:
        X = X + (0.2 + torch.rand(N, 1, generator=g, device="cuda")) * torch.randn(N, d, generator=g, device="cuda")
    X = X.to(tdt)
    K, Q = torch.randn(N, d, generator=g, device="cuda").to(tdt), torch.randn(7 * batch, d, generator=g, device="cuda").to(tdt)
    per = w * w
    h, ht = (np.arange(batch + 1) * n).astype(np.int32), (np.arange(batch + 1) * 7).astype(np.int32)
    cu, cut = torch.from_numpy(h).cuda(), torch.from_numpy(ht).cuda()
    i32 = dict(dtype=torch.int32, device="cuda")
    wo, wt = torch.empty(batch * per + 1, **i32), torch.empty(N, **i32)
    L.lightkv_build_windows(batch, h, cu, torch.arange(n, dtype=torch.int32).repeat(batch).cuda(), 1, gh, gw, w, wo, wt)
    wo, wt = wo.cpu().numpy(), wt.cpu().numpy()
    lists = [wt[wo[i]:wo[i + 1]] for i in range(batch * per)]
    got = []
    for order in (np.arange(batch * per), np.random.default_rng(3).permutation(batch * per)):
        ls = [lists[i] for i in order]
        owo = torch.from_numpy(np.concatenate([[0], np.cumsum([len(l) for l in ls])]).astype(np.int32)).cuda()
        owt = torch.from_numpy(np.concatenate(ls)).cuda()
        rem = torch.from_numpy(np.array([min(int(0.18 * len(l)), (len(l) + 1) // 2 * (len(l) // 2)) for l in ls], dtype=np.int32)).cuda()
        p = L.Problem(batch=batch, d=d, heads=d // 32, head_dim=32, dtype=dtype, h_cu_vis=h, cu_vis=cu, h_cu_txt=ht, cu_txt=cut,
                      n_windows=batch * per, max_window_tokens=max(len(l) for l in ls), win_offsets=owo, win_tokens=owt,
                      win_remove=rem, match=B.MATCH_EDGE_TOPK)
        ws = torch.full((L.lightkv_workspace_size(p),), 0x5a, dtype=torch.uint8, device="cuda")
        xi, fd = torch.ones(N, device="cuda"), torch.empty(N, device="cuda")
        best, dst, new, src = (torch.full((N,), -9, **i32) for _ in range(4))
        off, cu_out = torch.empty(N + 1, **i32), torch.empty(batch + 1, **i32)
        L.lightkv_score_select(p, X, Q if with_xi else None, K if with_xi else None, xi, fd, best, dst, new, off, src, cu_out, ws,
                               xi_mode=B.XI_TEXT_QUERY if with_xi else B.XI_GIVEN)
        total = int(off[-1])
        got.append([t.cpu().numpy() for t in (fd, best, dst, new, off, cu_out)] + [src[:total].cpu().numpy()])
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)
    fd, best, dst, new, off, cu_out, src = got[0]
    x64 = X.double()
    x64 = x64 / x64.norm(dim=1, keepdim=True)
    for l in lists:
        a, b = l[0::2], l[1::2]
        k = min(int(0.18 * len(l)), len(a) * len(b))
        edges = [(s, int(t)) for t in b for s in src[off[t]:off[t + 1]]]
        assert len(edges) == k and len(set(edges)) == k
        if not len(b):
            continue
        ta, tb = (torch.from_numpy(v.astype(np.int64)).cuda() for v in (a, b))
        m = (1.0 - x64[ta] @ x64[tb].T.contiguous()).clamp_min(0).cpu().numpy()
        ia, ib = {int(v): i for i, v in enumerate(a)}, {int(v): i for i, v in enumerate(b)}
        mine = np.zeros(m.shape, dtype=bool)
        for s, t in edges:
            mine[ia[int(s)], ib[t]] = True
        # nothing left out is lower than anything taken by more than fp32 scores resolve (1e-5 bf16 protocol, 1e-6 fp32)
        tol = 1e-5 if dtype == "bf16" else 1e-6
        if 0 < k < m.size:
            assert m[mine].max() <= m[~mine].min() + tol
        for t in b:
            assert list(src[off[t]:off[t + 1]]) == sorted(src[off[t]:off[t + 1]])
        assert set(np.flatnonzero(mine.any(1))) == {i for i, v in enumerate(a) if dst[v] >= 0}
        if ties and k:   # copies: exact zeros, taken in (A position, B position) order
            zero = m <= tol
            if zero.sum() >= k:
                want = np.zeros(m.size, dtype=bool)
                want[np.flatnonzero(zero.reshape(-1))[:k]] = True
                np.testing.assert_array_equal(mine.reshape(-1), want)


@pytest.mark.parametrize("dtype,heads,hd,batch,gh,gw,w,match,direction", [
    ("bf16", 2, 64, 3, 9, 7, 2, "best", 0), ("f32", 3, 128, 2, 12, 11, 1, "best", 0), ("bf16", 3, 32, 2, 13, 16, 1, "best", 1),
    ("f32", 2, 32, 1, 3, 3, 3, "best", 0), ("bf16", 2, 64, 2, 11, 12, 2, "pair", 0), ("bf16", 2, 128, 1, 20, 20, 1, "pair", 0),
    ("bf16", 4, 128, 2, 24, 24, 1, "best", 0),      # the tiled path: two streams
])
@pytest.mark.parametrize("mode", ["text", "text_lse", "vision"])
def test_scores_of_both_halves_are_those_of_each_half(dtype, heads, hd, batch, gh, gw, w, match, direction, mode):
    """lightkv_score with both halves in shared launches against one call per half: the same bits, also when a sequence has
    no prompt and into buffers that held something else."""
    import paper_2605_00789_amd as L
    from paper_2605_00789_amd import binding as B
    n, d = gh * gw, heads * hd
    N, texts = batch * n, [0 if b and mode != "text_lse" else 5 + 90 * b for b in range(batch)]
    T = sum(texts)
    g = torch.Generator(device="cuda").manual_seed(n + d)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    X, V = (torch.randn(N, d, generator=g, device="cuda").to(tdt) for _ in range(2))
    P = torch.randn(T, d, generator=g, device="cuda").to(tdt)
    Q, K = (V, P) if mode == "vision" else (P, V)
    lse = None if mode == "text" else 3.0 + torch.randn(heads, N if mode == "vision" else T, generator=g, device="cuda")
    h, ht = (np.arange(batch + 1) * n).astype(np.int32), np.concatenate([[0], np.cumsum(texts)]).astype(np.int32)
    i32 = dict(dtype=torch.int32, device="cuda")
    wo, wt = torch.empty(batch * w * w + 1, **i32), torch.empty(N, **i32)
    cu = torch.from_numpy(h).cuda()
    L.lightkv_build_windows(batch, h, cu, torch.arange(n, **i32).repeat(batch), 1, gh, gw, w, wo, wt)
    p = L.Problem(batch=batch, d=d, heads=heads, head_dim=hd, dtype=dtype, h_cu_vis=h, cu_vis=cu, h_cu_txt=ht,
                  cu_txt=torch.from_numpy(ht).cuda(), n_windows=batch * w * w, max_window_tokens=-(-gh // w) * -(-gw // w),
                  win_offsets=wo, win_tokens=wt, win_remove=torch.zeros(batch * w * w, **i32), direction=direction,
                  match=B.MATCH_BEST_PER_A if match == "best" else B.MATCH_FULL_PAIRWISE)
    ws = torch.empty(L.lightkv_workspace_size(p), dtype=torch.uint8, device="cuda")
    kw = dict(xi_mode=B.XI_VISION_QUERY if mode == "vision" else B.XI_TEXT_QUERY, lse=lse)

    def fresh():
        return torch.full((N,), -3.0, device="cuda"), torch.full((N,), -3.0, device="cuda"), torch.full((N,), -3, **i32)
    one, two = fresh(), fresh()
    for rep in range(2):
        ws.fill_(0x5a + rep)
        L.lightkv_score(p, X, Q, K, *one, ws, **kw)
    ws.fill_(0x33)
    L.lightkv_score(p, None, Q, K, two[0], None, None, ws, **kw)
    L.lightkv_score(p, X, None, None, two[0], two[1], two[2], ws, xi_mode=B.XI_GIVEN)
    for a, b in zip(one, two):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))
    assert (one[0] != -3.0).all()


@pytest.mark.parametrize("gh,gw,w", [(24, 24, 1), (24, 24, 4), (5, 13, 0)])
def test_full_pairwise_without_room_for_the_small_tiles(gh, gw, w):
    """A workspace that holds the squared norms, one to four key planes, xi and the selection scratch alone is enough: the
    large tiles need no partial sums.  Scores agree with those of the full workspace to the 1e-5 that two fp32 summation
    orders of bf16 products may differ by; the call alone, both halves in one call, and a ratio-driven schedule."""
    import paper_2605_00789_amd as L
    from paper_2605_00789_amd import binding as B
    n, d, heads, t = gh * gw, 256, 4, 33
    g = torch.Generator(device="cuda").manual_seed(n)
    X, K = (torch.randn(n, d, generator=g, device="cuda").bfloat16() for _ in range(2))
    Q = torch.randn(t, d, generator=g, device="cuda").bfloat16()
    per, i32 = max(w * w, 1), dict(dtype=torch.int32, device="cuda")
    h, ht = np.array([0, n], dtype=np.int32), np.array([0, t], dtype=np.int32)
    cu, cut, pos = torch.from_numpy(h).cuda(), torch.from_numpy(ht).cuda(), torch.arange(n, **i32)
    wo, wt, rem = torch.empty(per + 1, **i32), torch.empty(n, **i32), torch.empty(per, **i32)
    L.lightkv_build_windows(1, h, cu, pos, 1, gh, gw, w, wo, wt)
    L.lightkv_window_counts(1, per, wo, B.COUNT_RATIO, rem, rho=0.3)
    bound = min(n, L.lightkv_max_window_cells(1, gh, gw, w))
    p = L.Problem(batch=1, d=d, heads=heads, head_dim=d // heads, dtype="bf16", h_cu_vis=h, cu_vis=cu, h_cu_txt=ht, cu_txt=cut,
                  n_windows=per, max_window_tokens=bound, win_offsets=wo, win_tokens=wt, win_remove=rem, match=B.MATCH_FULL_PAIRWISE)

    def least(planes):
        parts = [4 * n, 8 * n * planes, 4 * heads * t * -(-n // 128) * 2, 4 * heads * n, 4 * n, 4 * n]
        return sum(-(-b // 256) * 256 for b in parts) + 256
    planes = max(1, -(-(bound // 2) // 96))
    planes = planes if planes <= 4 else 1
    small, full = least(planes), L.lightkv_workspace_size(p)
    assert small < full
    got = {}
    for name, size in (("small", small), ("full", full)):
        ws = torch.full((size + 4096,), 0x5a, dtype=torch.uint8, device="cuda")
        xi, fd, best = torch.empty(n, device="cuda"), torch.empty(n, device="cuda"), torch.empty(n, **i32)
        L.lightkv_score(p, X, Q, K, xi, fd, best, ws[:size])
        dst, new, src, fd2, best2 = (torch.empty(n, **i32) for _ in range(5))
        fd2, off, cu_out = torch.empty(n, device="cuda"), torch.empty(n + 1, **i32), torch.empty(2, **i32)
        L.lightkv_score_select(p, X, Q, K, xi, fd2, best2, dst, new, off, src, cu_out, ws[:size])
        assert torch.equal(fd, fd2) and torch.equal(best, best2)
        assert bool((ws[size:] == 0x5a).all())
        got[name] = (xi, fd, int(cu_out[1]))
    assert torch.equal(got["small"][0], got["full"][0])
    assert float((got["small"][1] - got["full"][1]).abs().max()) <= 1e-5
    assert got["small"][2] < n and got["full"][2] < n
    with pytest.raises(L.LightKVError, match="workspace"):
        L.lightkv_score(p, X, Q, K, xi, fd, best, torch.empty(small - 512, dtype=torch.uint8, device="cuda"))
    s = L.EdgeTopKSchedule(dtype="bf16", batch=1, d=d, heads=heads, head_dim=d // heads, tiles=1, grid_h=gh, grid_w=gw, cu_txt=ht,
                           windows_per_axis=[w, w], rho=[0.3, 0.3], match="full_pairwise")
    s._ws = torch.empty(small, dtype=torch.uint8, device="cuda")
    out = s.run(h, X, K, K, Q, pos)
    assert len(out) == 2 and 0 < int(out[-1].h_cu_vis_out[1]) < int(out[0].h_cu_vis_out[1]) < n


@pytest.mark.parametrize("batch,n,v,k,T", [(1, 576, 36, 17, 3), (8, 576, 36, 16, 3), (8, 576, 36, 17, 3), (29, 565, 37, 4, 3),
                                           (29, 566, 37, 4, 3), (29, 565, 16, 3, 3), (29, 565, 16, 3, 1000)])
@pytest.mark.parametrize("with_xi", [False, True])
def test_edge_lists_placed_by_the_scan_and_by_a_launch_of_their_own(batch, n, v, k, T, with_xi):
    """Counts known to the host (the list gets a launch of its own beyond 2048 edges) and to the device alone (beyond 16384
    tokens): lists of 272, 2048, 2176 edges and of 16385 and 16414 tokens; 1044 windows with short prompts and (T) with ones of 1000, where xi
    has a stream of its own.  The same bits either way, and the sources of
    every token are the edges that the tokens' own columns say."""
    import paper_2605_00789_amd as L
    from paper_2605_00789_amd import binding as B
    N, d = batch * n, 64
    g = torch.Generator(device="cuda").manual_seed(N)
    X, K = (torch.randn(N, d, generator=g, device="cuda").bfloat16() for _ in range(2))
    Q = torch.randn(T * batch, d, generator=g, device="cuda").bfloat16()
    h, ht = (np.arange(batch + 1) * n).astype(np.int32), (np.arange(batch + 1) * T).astype(np.int32)
    wo = np.unique(np.concatenate([np.append(np.arange(b * n, (b + 1) * n, v), (b + 1) * n) for b in range(batch)])).astype(np.int32)
    sizes = np.diff(wo)
    rem = np.minimum(k, (sizes + 1) // 2 * (sizes // 2)).astype(np.int32)
    i32 = dict(dtype=torch.int32, device="cuda")
    cu, cut, d_wo, d_rem = (torch.from_numpy(a).cuda() for a in (h, ht, wo, rem))
    wt = torch.arange(N, **i32)
    got = []
    for host in (True, False):
        p = L.Problem(batch=batch, d=d, heads=2, head_dim=32, dtype="bf16", h_cu_vis=h, cu_vis=cu, h_cu_txt=ht, cu_txt=cut,
                      n_windows=len(sizes), max_window_tokens=v, win_offsets=d_wo, win_tokens=wt, win_remove=d_rem,
                      match=B.MATCH_EDGE_TOPK, h_win_offsets=wo if host else None, h_win_remove=rem if host else None)
        ws = torch.full((L.lightkv_workspace_size(p),), 0x21, dtype=torch.uint8, device="cuda")   # a stale list of valid tokens
        xi, fd = torch.ones(N, device="cuda"), torch.empty(N, device="cuda")
        best, dst, new, src = (torch.full((N,), -9, **i32) for _ in range(4))
        off, cu_out = torch.empty(N + 1, **i32), torch.empty(batch + 1, **i32)
        L.lightkv_score_select(p, X, Q if with_xi else None, K if with_xi else None, xi, fd, best, dst, new, off, src, cu_out, ws,
                               xi_mode=B.XI_TEXT_QUERY if with_xi else B.XI_GIVEN)
        got.append([t.cpu().numpy() for t in (fd, best, dst, new, off, cu_out, src, xi)])
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)
    fd, best, dst, new, off, cu_out, src, xi = got[0]
    assert off[-1] == rem.sum()
    assert (src[off[-1]:] == -9).all()
    win = np.repeat(np.arange(len(sizes)), sizes)
    owner = np.repeat(np.arange(N), np.diff(off))
    assert (win[src[:off[-1]]] == win[owner]).all() and ((owner - wo[win[owner]]) % 2 == 1).all()
    assert set(src[:off[-1]]) == set(np.flatnonzero(dst >= 0))
    np.testing.assert_array_equal(np.bincount(win[owner], minlength=len(sizes)), rem)


@pytest.mark.parametrize("n,d,share", [(36, 256, 0.5), (64, 512, 0.4), (65, 512, 0.4), (144, 1024, 0.02), (144, 1024, 0.3), (144, 1024, 0.5), (144, 1024, 0.9),
                                       (255, 512, 0.5), (256, 512, 1.0)])
def test_edge_selection_of_many_pairs(n, d, share):
    """Unrelated tokens: the divergences crowd around one, and the threshold lies where hundreds of them share its first
    bin.  The pairs taken against their divergence in float64 (bf16 protocol: nothing left out is lower by more than 1e-5), four
    windows with another order each."""
    import paper_2605_00789_amd as L
    from paper_2605_00789_amd import binding as B
    W, N = 4, 4 * n
    g = torch.Generator(device="cuda").manual_seed(n + int(100 * share))
    X = torch.randn(N, d, generator=g, device="cuda").bfloat16()
    lists = [np.sort(p) for p in np.split(np.random.default_rng(n).permutation(N).astype(np.int32), W)]
    wo, h = (np.arange(W + 1) * n).astype(np.int32), np.array([0, N], dtype=np.int32)
    na, nb = (n + 1) // 2, n // 2
    k = int(share * na * nb)
    rem = np.full(W, k, dtype=np.int32)
    i32 = dict(dtype=torch.int32, device="cuda")
    p = L.Problem(batch=1, d=d, heads=d // 32, head_dim=32, dtype="bf16", h_cu_vis=h, cu_vis=torch.from_numpy(h).cuda(), n_windows=W,
                  max_window_tokens=n, win_offsets=torch.from_numpy(wo).cuda(), win_tokens=torch.from_numpy(np.concatenate(lists)).cuda(),
                  win_remove=torch.from_numpy(rem).cuda(), match=B.MATCH_EDGE_TOPK, h_win_offsets=wo, h_win_remove=rem)
    ws = torch.full((L.lightkv_workspace_size(p),), 0x5a, dtype=torch.uint8, device="cuda")
    xi, fd = torch.ones(N, device="cuda"), torch.empty(N, device="cuda")
    best, dst, new = (torch.empty(N, **i32) for _ in range(3))
    off, cu_out, src = torch.empty(N + 1, **i32), torch.empty(2, **i32), torch.full((W * k,), -9, **i32)
    L.lightkv_score_select(p, X, None, None, xi, fd, best, dst, new, off, src, cu_out, ws, xi_mode=B.XI_GIVEN)
    off, src, dst = off.cpu().numpy(), src.cpu().numpy(), dst.cpu().numpy()
    x64 = X.double()
    x64 = x64 / x64.norm(dim=1, keepdim=True)
    for l in lists:
        a, b = l[0::2], l[1::2]
        ta, tb = (torch.from_numpy(v.astype(np.int64)).cuda() for v in (a, b))
        m = (1.0 - x64[ta] @ x64[tb].T.contiguous()).clamp_min(0).cpu().numpy()
        ia, mine = {int(v): i for i, v in enumerate(a)}, np.zeros(m.shape, dtype=bool)
        for j, t in enumerate(b):
            s = src[off[t]:off[t + 1]]
            assert list(s) == sorted(s)
            mine[[ia[int(v)] for v in s], j] = True
        assert mine.sum() == k
        if k < m.size:
            assert m[mine].max() <= m[~mine].min() + 1e-5
        np.testing.assert_array_equal(dst[a] >= 0, mine.any(1))
        low = np.where(mine, m, np.inf)
        hit = np.flatnonzero(mine.any(1))
        to = np.array([int(np.flatnonzero(b == dst[a[i]])[0]) for i in hit], dtype=int)
        assert mine[hit, to].all() and (low[hit, to] <= low[hit].min(1) + 1e-5).all()


@pytest.mark.parametrize("W", [1, 63, 64, 65, 191, 192, 193, 700, 4097, 9000])
@pytest.mark.parametrize("kind", ["equal", "ragged"])
def test_token_budgets_over_many_windows(W, kind):
    """One wave up to 192 windows of a sequence, the workgroup beyond; window sizes in LDS and (beyond 8192) in memory.
    Budgets of nothing, a third, all but one and all of what the windows can give, and two that cannot be met."""
    import paper_2605_00789_amd as L
    from paper_2605_00789_amd import binding as B
    from oracle import lightkv_oracle as O
    rng = np.random.default_rng(W)
    sizes = np.full(W, 5) if kind == "equal" else rng.integers(0, 40, W)
    caps = np.where(sizes >= 2, (sizes + 1) // 2, 0)
    n, most = int(sizes.sum()), int(caps.sum())
    batch = 6
    leave = [0, most // 3, max(most - 1, 0), most, min(most + 1, n), -3]
    wo = np.concatenate([[0], np.cumsum(np.tile(sizes, batch))]).astype(np.int32)
    cu = (np.arange(batch + 1) * n).astype(np.int32)
    target = np.concatenate([[0], np.cumsum([n - l for l in leave])]).astype(np.int32)
    out = torch.full((batch * W,), -7, dtype=torch.int32, device="cuda")
    status = torch.full((batch,), -7, dtype=torch.int32, device="cuda")
    L.lightkv_window_counts(batch, batch * W, torch.from_numpy(wo).cuda(), B.COUNT_TARGET, out, cu_vis=torch.from_numpy(cu).cuda(),
                            cu_vis_target=torch.from_numpy(target).cuda(), status=status)
    got = out.cpu().numpy().reshape(batch, W)
    for b, l in enumerate(leave):
        bad = l < 0 or l > most
        assert int(status[b]) == int(bad)
        if bad:
            np.testing.assert_array_equal(got[b], caps if l > most else 0)
            continue
        q = max(v for v in range(int(caps.max()) + 2) if np.minimum(caps, v).sum() <= l)   # the rule as the header states it
        want = np.minimum(caps, q)
        want[np.flatnonzero(caps > q)[:l - int(want.sum())]] += 1
        np.testing.assert_array_equal(got[b], want)


@pytest.mark.parametrize("tiles,gh,gw,w", [(1, 8, 8, 90), (1, 3, 5, 9), (2, 7, 11, 8), (1, 1, 129, 5), (1, 97, 89, 8), (1, 128, 128, 4), (1, 128, 128, 16)])
def test_window_partition_with_scattered_cells(tiles, gh, gw, w):
    """Tokens in any order, cells missing and repeated, more windows than tokens; grids whose sides are no powers of two."""
    import paper_2605_00789_amd as L
    from oracle import lightkv_oracle as O
    n = min(tiles * gh * gw, 9000)
    rng = np.random.default_rng(n + w)
    pos = rng.integers(0, tiles * gh * gw, 2 * n).astype(np.int32)
    h_cu = np.array([0, n, 2 * n], dtype=np.int32)
    wps = tiles * w * w
    ro, rt = O.build_windows(pos, h_cu, tiles, gh, gw, w)
    wo = torch.full((2 * wps + 1,), -7, dtype=torch.int32, device="cuda")
    wt = torch.full((2 * n,), -7, dtype=torch.int32, device="cuda")
    L.lightkv_build_windows(2, h_cu, torch.from_numpy(h_cu).cuda(), torch.from_numpy(pos).cuda(), tiles, gh, gw, w, wo, wt)
    np.testing.assert_array_equal(wo.cpu().numpy(), ro)
    np.testing.assert_array_equal(wt.cpu().numpy(), rt)


SCHEDULES = [
    # tokens beyond those whose window and rank the riding partition keeps in registers; a batch with windows of unequal sizes
    (1, 56, 58, (8, 4, 2), (2700, 2200, 1800), 2, 64), (2, 61, 67, (5, 3, 2), (3500, 3000, 2500), 1, 64),
    (1, 80, 80, (8, 16, 8), (5500, 4700, 4000), 2, 32),      # 256 windows: the counts do not fit beside the rows
    (1, 80, 80, (8, 30, 28), (5500, 4700, 4000), 2, 32),     # 900 windows: nor the partition's own LDS (sorted)
    (1, 64, 64, (4, 2, 1), (3300, 2700, 2200), 8, 32),       # the tiled divergence, where xi forks as well
]


def _schedule(batch, gh, gw, windows, targets, heads, hd):
    import paper_2605_00789_amd as L
    n, d, t = gh * gw, heads * hd, 9
    g = torch.Generator(device="cuda").manual_seed(n)
    X, K, V = (torch.randn(batch * n, d, generator=g, device="cuda").bfloat16() for _ in range(3))
    Q = torch.randn(batch * t, d, generator=g, device="cuda").bfloat16()
    pos = torch.arange(n, dtype=torch.int32, device="cuda").repeat(batch)
    kw = dict(dtype="bf16", batch=batch, d=d, heads=heads, head_dim=hd, tiles=1, grid_h=gh, grid_w=gw,
              cu_txt=(np.arange(batch + 1) * t).astype(np.int32), windows_per_axis=windows)
    return L, kw, (X, K, V, Q, pos)


@pytest.mark.parametrize("shape", SCHEDULES, ids=lambda s: "%dx%dx%d_%s" % (s[0], s[1], s[2], "-".join(map(str, s[3]))))
def test_schedule_builds_windows_in_every_place(shape):
    """The next stage's windows ride in the merge's launch or are built beside it: the schedule in one call against the same
    stages call by call, bit for bit, eagerly and as a replayed graph."""
    L, kw, (X, K, V, Q, pos) = _schedule(*shape)
    names = ("win_offsets", "win_tokens", "win_remove", "status", "xi", "best_fd", "dst", "new_index", "grp_offsets", "cu_vis_out",
             "X_out", "K_out", "V_out", "pos_out")
    one, steps = (L.CompressionPipeline(targets=shape[4], **kw) for _ in range(2))
    a, sq = (X, K, V, pos), None
    for s in range(len(shape[3])):
        st = steps.run_stage(s, *a[:3], Q, a[3], x_sqnorm=sq)
        a, sq = (st.X_out, st.K_out, st.V_out, st.pos_out), st.x_sq_out

    def check(what):
        torch.cuda.synchronize()
        for s, (x, y) in enumerate(zip(one.stages, steps.stages)):
            assert int(x.status.sum()) == 0
            for n in names:
                assert torch.equal(getattr(x, n), getattr(y, n)), (what, s, n)

    def scribble():
        for st in one.stages:
            st.X_out.zero_(); st.win_tokens.fill_(-1); st.win_remove.fill_(-1); st.xi.fill_(float("nan")); st.dst.fill_(-3)
    for rep in range(2):
        scribble()
        one.run(X, K, V, Q, pos)
        check("eager %d" % rep)
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        one.run(X, K, V, Q, pos)
    for rep in range(3):
        scribble()
        torch.cuda.synchronize()
        graph.replay()
        check("replay %d" % rep)


@pytest.mark.parametrize("match", ["best_per_a", "edge_topk", "full_pairwise"])
@pytest.mark.parametrize("shape", SCHEDULES, ids=lambda s: "%dx%dx%d_%s" % (s[0], s[1], s[2], "-".join(map(str, s[3]))))
def test_ratio_schedule_builds_windows_in_every_place(shape, match):
    """The same for schedules whose counts depend on the data: one call against the stages call by call."""
    L, kw, (X, K, V, Q, pos) = _schedule(*shape)
    h = (np.arange(shape[0] + 1) * (shape[1] * shape[2])).astype(np.int32)
    res = []
    for form in ("run", "run_steps"):
        s = L.EdgeTopKSchedule(rho=[0.2] * len(shape[3]), match=match, **kw)
        last = [getattr(s, form)(h, X, K, V, Q, pos) for _ in range(2)][-1]
        torch.cuda.synchronize()
        res.append([r.h_cu_vis_out for r in last] + [t.cpu() for t in (last[-1].X, last[-1].K, last[-1].V, last[-1].pos)])
    for x, y in zip(*res):
        if isinstance(x, np.ndarray):
            np.testing.assert_array_equal(x, y)
        else:
            assert torch.equal(x, y)


def _ratio_job(seed, match, batch=1, gh=24, gw=24, windows=(4, 2, 1), d=256, heads=4):
    import paper_2605_00789_amd as L
    n, t = gh * gw, 7
    g = torch.Generator(device="cuda").manual_seed(seed)
    X, K, V = (torch.randn(batch * n, d, generator=g, device="cuda").bfloat16() for _ in range(3))
    Q = torch.randn(batch * t, d, generator=g, device="cuda").bfloat16()
    pos = torch.arange(n, dtype=torch.int32, device="cuda").repeat(batch)
    h = (np.arange(batch + 1) * n).astype(np.int32)

    def make():
        return L.EdgeTopKSchedule(dtype="bf16", batch=batch, d=d, heads=heads, head_dim=d // heads, tiles=1, grid_h=gh, grid_w=gw,
                                  cu_txt=(np.arange(batch + 1) * t).astype(np.int32), windows_per_axis=windows,
                                  rho=[0.25] * len(windows), match=match)
    return make, (h, X, K, V, Q, pos)


def _ratio_result(out):
    return [r.h_cu_vis_out.copy() for r in out] + [t.cpu().numpy() if t.dtype == torch.int32 else t.float().cpu().numpy()
                                                   for t in (out[-1].X, out[-1].K, out[-1].V, out[-1].pos)]


def test_ratio_schedules_of_several_threads_at_once():
    """Six host threads, more than there are mailboxes for the offsets of a stage, run data-dependent schedules of different
    matchings and sizes on streams and buffers of their own, again and again: the bits of a run alone, every time."""
    import threading
    jobs = []
    for i, match in enumerate(["edge_topk", "best_per_a", "full_pairwise", "edge_topk", "best_per_a", "full_pairwise"]):
        make, args = _ratio_job(i, match, batch=1 + i % 3, gh=12 + 4 * (i % 4), windows=(4, 2, 1) if i % 2 else (3, 1))
        s = make()
        want = _ratio_result(s.run(*args))
        jobs.append((s, args, want))
    torch.cuda.synchronize()
    errors, start = [], threading.Barrier(len(jobs))

    def work(k):
        try:
            s, args, want = jobs[k]
            stream = torch.cuda.Stream()
            start.wait(timeout=60)
            with torch.cuda.stream(stream):
                for it in range(25):
                    for j, (a, b) in enumerate(zip(_ratio_result(s.run(*args)), want)):
                        if not np.array_equal(a, b):
                            errors.append((k, it, j))
        except Exception as e:   # noqa: BLE001
            errors.append(repr(e))
    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join(timeout=100)
    assert not any(t.is_alive() for t in threads)
    assert not errors, errors[:5]


@pytest.mark.parametrize("batch", [1022, 1023, 1024, 1100])
@pytest.mark.parametrize("match", ["edge_topk", "best_per_a"])
def test_ratio_schedule_of_more_sequences_than_a_mailbox_holds(batch, match):
    """Up to 1023 sequences the offsets come through the mailbox, beyond that by a copy: against the stages call by call."""
    make, args = _ratio_job(batch, match, batch=batch, gh=2, gw=3, windows=(1, 1), d=64, heads=2)
    want = _ratio_result(make().run_steps(*args))
    s = make()
    for _ in range(3):
        for a, b in zip(_ratio_result(s.run(*args)), want):
            np.testing.assert_array_equal(a, b)


def test_ratio_schedule_beside_an_open_capture():
    """The first ratio-driven call of a process, which allocates its mailbox, on one thread while another has a capture open: the
    right result, and the capture ends and replays."""
    import os
    import subprocess
    import sys
    code = r"""
import sys, threading
sys.path.insert(0, '.'); sys.path.insert(0, 'tests')
import numpy as np, torch
from test_gpu_launch_edges import _ratio_job, _ratio_result
make, args = _ratio_job(3, 'edge_topk')
s, ref = make(), make()
a, b = torch.ones(1000, device='cuda'), torch.zeros(1000, device='cuda')
torch.cuda.synchronize()
got, errors = [], []
def other():
    try:
        with torch.cuda.stream(torch.cuda.Stream()):
            got.append(_ratio_result(s.run(*args)))
    except Exception as e:
        errors.append(repr(e))
graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
with torch.cuda.graph(graph, stream=stream, capture_error_mode='thread_local'):
    b.add_(a)
    t = threading.Thread(target=other); t.start(); t.join(timeout=60)
    b.add_(a)
assert not errors and len(got) == 1, errors
for _ in range(3): graph.replay()
torch.cuda.synchronize()
assert float(b.min()) == 6.0 == float(b.max())
for x, y in zip(got[0], _ratio_result(ref.run_steps(*args))): np.testing.assert_array_equal(x, y)
print('beside-capture ok', flush=True)
"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-u", "-c", code], cwd=root, capture_output=True, text=True, timeout=100)
    print(r.stdout[-2000:], r.stderr[-3000:], flush=True)
    assert r.returncode == 0 and "beside-capture ok" in r.stdout


@pytest.mark.parametrize("v", [2, 3, 7, 8, 9, 16, 17, 63, 190, 191, 193, 194, 400, 511, 512, 513, 514, 801])
def test_ranks_among_equal_scores(v):
    """lightkv_select on scores with many ties (three distinct values, +inf among them): an A node's rank counts the earlier
    nodes with its score, a source's rank the earlier sources of its target.  Windows around the groups of four of the counting
    loops, the segments of the window kernel and the line to the kernel of large windows; plain Python as reference."""
    import paper_2605_00789_amd as L
    rng = np.random.default_rng(v)
    n_w, nA, nB = 3, (v + 1) // 2, v // 2
    n = n_w * v
    fd, prop = np.full(n, np.inf, dtype=np.float32), np.full(n, -1, dtype=np.int32)
    for w in range(n_w):
        a, b = np.arange(w * v, (w + 1) * v, 2), np.arange(w * v + 1, (w + 1) * v, 2)
        fd[a] = rng.choice(np.array([0.0, 0.25, np.inf], dtype=np.float32), nA)
        prop[a] = rng.choice(b[:max(1, nB // 3)], nA)
    remove = np.array([nA, max(1, nA // 2), 1], dtype=np.int32)
    h_cu, wo = np.array([0, n], dtype=np.int32), (np.arange(n_w + 1) * v).astype(np.int32)
    i32 = lambda t: torch.from_numpy(np.ascontiguousarray(t, dtype=np.int32)).cuda()
    empty = lambda k: torch.full((k,), -7, dtype=torch.int32, device="cuda")
    prob = L.Problem(batch=1, d=64, heads=2, head_dim=32, dtype="bf16", h_cu_vis=h_cu, cu_vis=i32(h_cu), n_windows=n_w,
                     max_window_tokens=v, win_offsets=i32(wo), win_tokens=i32(np.arange(n)), win_remove=i32(remove))
    ws = torch.empty(L.lightkv_workspace_size(prob), dtype=torch.uint8, device="cuda")
    dst, new_index, offs, src, cu = empty(n), empty(n), empty(n + 1), empty(n), empty(2)
    L.lightkv_select(prob, torch.from_numpy(fd).cuda(), i32(prop), dst, new_index, offs, src, cu, ws)
    want = np.full(n, -1)
    for w in range(n_w):
        a = np.arange(w * v, (w + 1) * v, 2)
        gone = a[np.argsort(fd[a], kind="stable")[:remove[w]]]
        want[gone] = prop[gone]
    np.testing.assert_array_equal(dst.cpu().numpy(), want)
    keep = want < 0
    np.testing.assert_array_equal(new_index.cpu().numpy(), np.where(keep, np.cumsum(keep) - 1, -1))
    order = np.flatnonzero(~keep)[np.argsort(want[~keep], kind="stable")]
    np.testing.assert_array_equal(offs.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(want[~keep], minlength=n))]))
    np.testing.assert_array_equal(src.cpu().numpy()[:len(order)], order)


def _window_scores(X, n_w, v, d, dtype):
    """best_fd of n_w windows of v tokens each."""
    import paper_2605_00789_amd as L
    from paper_2605_00789_amd import binding as B
    n = n_w * v
    i32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    h_cu = np.array([0, n], dtype=np.int32)
    prob = L.Problem(batch=1, d=d, heads=d // 32, head_dim=32, dtype=dtype, h_cu_vis=h_cu, cu_vis=i32(h_cu), n_windows=n_w,
                     max_window_tokens=v, win_offsets=i32(np.arange(n_w + 1) * v), win_tokens=i32(np.arange(n)),
                     win_remove=i32(np.zeros(n_w)))
    ws = torch.empty(L.lightkv_workspace_size(prob), dtype=torch.uint8, device="cuda")
    fd, dst = torch.empty(n, device="cuda"), torch.empty(n, dtype=torch.int32, device="cuda")
    L.lightkv_score(prob, X, None, None, torch.ones(n, device="cuda"), fd, dst, ws, xi_mode=B.XI_GIVEN)
    return fd


@pytest.mark.parametrize("n_w,v,d,dtype", [
    (45, 70, 4096, "bf16"), (20, 96, 4096, "bf16"), (96, 36, 5120, "bf16"), (127, 40, 4096, "bf16"),   # long slices
    (200, 36, 2048, "bf16"), (255, 36, 2048, "bf16"), (140, 36, 1280, "bf16"), (300, 40, 1280, "bf16"),
    (100, 36, 4160, "bf16"), (70, 40, 4192, "bf16"), (80, 36, 4672, "bf16"), (130, 36, 2336, "bf16"),  # ... with pieces no wave or not every wave has a span of
    (256, 36, 2048, "bf16"), (400, 36, 2048, "bf16"),                                                  # short ones
    (16, 36, 4096, "bf16"), (180, 16, 4096, "bf16"), (144, 36, 3712, "bf16"), (90, 40, 4096, "f32"),
])
def test_error_of_the_divergence_of_near_equal_rows(n_w, v, d, dtype):
    """1 - cos of rows that differ by a few percent, against 64 bits: what is left of the error of the inner products and the
    squared norms.  A chain of m fp32 additions of equal shares rounds to u/sqrt(3) * sqrt(m/3) of its sum (rms, u = 2^-24);
    over C chains that is u/3 * sqrt(m / C) of the whole, and of 1 - cos = 1 - ab / sqrt(aa bb) sqrt(1 + 1/4 + 1/4) times as
    much.  No chain is longer than 128 elements of bf16 (64 of fp32): m = 16 (32), C = d / 128 (d / 64).  Half as much again is
    allowed, for the sums that are rounded on their way to memory."""
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    m, chains = (16, d / 128) if dtype == "bf16" else (32, d / 64)
    bound = 1.5 * 1.5 ** 0.5 * 2.0 ** -24 / 3 * (m / chains) ** 0.5
    err = []
    for seed in range(2):
        g = torch.Generator(device="cuda").manual_seed(seed)
        base = torch.randn(n_w, 1, d, generator=g, device="cuda")
        X = (base + 0.03 * torch.randn(n_w, v, d, generator=g, device="cuda")).reshape(n_w * v, d).to(dt)
        fd = _window_scores(X, n_w, v, d, dtype).double().view(n_w, v)[:, 0::2]
        x = X.double().view(n_w, v, d)
        a, b = x[:, 0::2], x[:, 1::2]
        dot = torch.stack([p @ q.T.contiguous() for p, q in zip(a, b)])
        want = (1.0 - dot / ((a * a).sum(2)[:, :, None] * (b * b).sum(2)[:, None, :]).sqrt()).min(2).values
        err.append((fd - want).flatten())
    rms = float(torch.cat(err).square().mean().sqrt())
    assert rms <= bound, (rms, bound)


def test_sums_beyond_the_largest_float():
    """Rows so large that the squared norm of half a row is beyond the largest fp32 value, but no short slice of it: the
    divergence is that of the same rows scaled down by a power of two.  Rows with an infinity or a NaN have none."""
    n_w, v, d = 200, 36, 2048
    g = torch.Generator(device="cuda").manual_seed(5)
    X = (1.2 * torch.randn(n_w, 1, d, generator=g, device="cuda").expand(n_w, v, d)
         + 0.2 * torch.randn(n_w, v, d, generator=g, device="cuda")).reshape(n_w * v, d).to(torch.bfloat16)
    half = X[:, :d // 2].double().square().sum(1).min()
    assert float(half) * 4.0 ** 59 > 3.4028234663852886e38
    small, large = _window_scores(X, n_w, v, d, "bf16"), _window_scores(X * 2.0 ** 59, n_w, v, d, "bf16")
    assert bool(((small - large).abs() <= 1e-7)[torch.isfinite(small)].all())
    assert torch.equal(torch.isfinite(small), torch.isfinite(large))
    X[0, 3], X[2 * v, 5] = float("inf"), float("nan")
    bad = _window_scores(X, n_w, v, d, "bf16")
    assert not torch.isfinite(bad[0]) and not torch.isfinite(bad[2 * v])
    good = torch.isfinite(small)
    good[0] = good[2 * v] = False
    assert torch.equal(bad[good], small[good])
