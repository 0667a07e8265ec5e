"""GPU kernels at the edges of the ranges their dispatch rules give them, against the CPU oracle."""
import numpy as np
import pytest
import torch

import gpu_helpers as H
from oracle_helpers import gmm_model, oracle_setup
from paper_2505_03983_amd import binding, runtime

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _denoise(cfg, n, seed=3, keep=None, tiled=False, split=None, change=None):
    """tiled: on the tiled kernels, whichever the call would take by itself; else it is expected not to take them.  split
    (not None): the switch of the split operands, and whether the call is expected to have taken them.  change: of the means."""
    T, p, model = oracle_setup(cfg)
    rng = np.random.default_rng(seed)
    if change is not None:
        p["means"] = change(p["means"])
    if cfg["kind"] == "gmm":     # unequal weights
        p["log_w"] = np.log(rng.dirichlet(np.ones(cfg["C"]))).astype(np.float32)
        from oracle_helpers import gmm_model
        model = gmm_model(T, p)
    ctx = runtime.open_ctx(cfg, p, seed=0, chains=-(-n // cfg["L"]))
    ctx.use_few_rows(not tiled)
    if split is not None:
        ctx.use_split_gemm(split)
        assert ctx.split_gemm_active() == split
    ctx.profile_enable(True)
    tau = rng.integers(1, cfg["K"] + 1, n).astype(np.int32)
    ab = T["abar"][tau]
    x0 = p["means"][rng.integers(0, cfg["C"], n)] + 0.5 * rng.standard_normal((n, cfg["d"]))
    x = (np.sqrt(ab)[:, None] * x0 + np.sqrt(1 - ab)[:, None] * rng.standard_normal((n, cfg["d"]))).astype(np.float32)
    if keep is not None:         # a call of the first rows only
        n, x, tau = keep, x[:keep], tau[:keep]
    out = torch.full((n, cfg["d"]), float("nan"), dtype=torch.float32, device=DEV)
    ctx.denoise(torch.from_numpy(x).to(DEV), torch.from_numpy(tau).to(DEV), out)
    torch.cuda.synchronize()
    assert ctx.profile_read(binding.PROF["GMM_LOGITS" if tiled else "GMM_ROWWISE"], 1)[0] == 1
    if split is not None:
        assert ctx.profile_read(binding.PROF["GMM_SOFTMAX"], 1)[0] == int(split)
    ctx.close()
    if keep is not None:
        return out.cpu().numpy(), None
    return out.cpu().numpy(), model(cfg["K"] - tau, x.astype(np.float64))


@pytest.mark.parametrize("d, C, n", [
    (1, 1, 1), (2, 64, 5), (3, 80, 1024), (15, 17, 1030), (64, 4, 16383), (3, 21, 32768),   # the row-wise kernel
    (4, 1, 1), (16, 16, 17), (4, 128, 77), (512, 20, 1024),     # the one with the mixture in LDS: a row per wavefront
    (16, 16, 16384), (256, 16, 8195), (1000, 7, 32771),         # four rows per wavefront, the last ones missing
    (8, 32, 16384), (516, 4, 512), (4, 129, 77), (4, 16, 131072), (3, 22, 16384),       # just past them
    (1, 257, 1), (257, 1, 3), (15, 18, 15), (17, 16, 16),       # one partial tile in every direction
    (100, 64, 33), (97, 65, 16), (256, 1024, 1), (260, 1028, 47), (301, 1003, 40),   # k shared by 1, 2, 4 wavefronts
    (5, 33, 8200), (64, 1024, 1025), (130, 1027, 993),    # 32 x 32 tiles: last row, column and k step partial
    (2000, 3000, 9), (1093, 3003, 9), (1093, 3003, 700),  # mixtures that no LDS holds, and the largest of odd sizes
])
def test_mixture_calls_of_few_rows(d, C, n):
    """fp32 products and sums: logits of up to ~2^9 in fp32 move a weight by at most 2^9 2^-24 = 3e-5 of itself, and
    the mean by no more."""
    got, want = _denoise(dict(kind="gmm", d=d, C=C, K=50, L=16, var=0.25), n)
    assert H.rel_err(got, want) <= 3e-5


def test_mixture_calls_larger_than_their_scratch():
    """66048 rows of logits fit the scratch of this mixture: two whole parts and 76 rows.  Same bound as above; a call of
    fewer rows on the same tiles gives the same bits."""
    cfg = dict(kind="gmm", d=3, C=999, K=50, L=16, var=0.25)
    n = 2 * 66048 + 76
    got, want = _denoise(cfg, n)
    assert H.rel_err(got, want) <= 3e-5
    part, _ = _denoise(cfg, n, keep=67000)
    assert np.array_equal(part, got[:67000])


@pytest.mark.parametrize("d, C", [(1, 256), (1, 300)])     # the row-wise kernel; the kernels for few rows
def test_mixture_scratch_is_bounded(d, C):
    """A context of a million rows takes some tens of bytes a row and at most 256 MiB of logits (a gigabyte if every row
    had its own)."""
    cfg = dict(kind="gmm", d=d, C=C, K=4, L=64, var=0.25)
    T, p, _ = oracle_setup(cfg)
    runtime.open_ctx(cfg, p, chains=1).close()     # (the first context of a process also loads the kernels)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    ctx = runtime.open_ctx(cfg, p, chains=16384)
    taken = free - torch.cuda.mem_get_info()[0]
    ctx.close()
    assert taken <= 64 * 16384 * 64 + (384 << 20), taken


@pytest.mark.parametrize("d, C, n", [(96, 1056, 15000), (80, 1040, 19000), (500, 1000, 8100),
                                     (96, 1056, 16400), (160, 640, 16400)])
def test_mixture_calls_on_the_tiled_kernels(d, C, n):
    """Two fp16 terms, three bf16 terms, fp32; then the least rows that go to 256-wide tiles, C ending inside one (same
    bound)."""
    got, want = _denoise(dict(kind="gmm", d=d, C=C, K=50, L=16, var=0.25), n, tiled=True)
    assert H.rel_err(got, want) <= 3e-5


@pytest.mark.parametrize("d, C, n, part", [
    (1000, 4000, 1001, 500),      # 256 tiles of the first product, 64 of the second (64 x 64 instead); 128 (64 x 128) and 32
    (500, 1000, 9000, 8127),      # both products on smaller tiles, none full at the edges; neither
    (512, 2052, 8100, 4100),      # neither; both
])
def test_fp32_tiles_do_not_depend_on_their_size(d, C, n, part):
    """Calls of the fp32 kernels on either side of the rule that picks smaller tiles, and parts of them, which go to others:
    the sums of an element are the same in every tile, so shared rows are equal bit for bit; against the oracle as above."""
    cfg = dict(kind="gmm", d=d, C=C, K=50, L=16, var=0.25)
    got, want = _denoise(cfg, n, tiled=True, split=False)
    assert H.rel_err(got, want) <= 3e-5
    first, _ = _denoise(cfg, n, keep=part, tiled=True, split=False)
    assert np.array_equal(first, got[:part])


@pytest.mark.parametrize("terms", [1, 2])
@pytest.mark.parametrize("d, E, width, blocks, rows", [
    (8, 0, 8, 1, (1, 2)),                            # one slab of K, most of it padding
    (40, 24, 72, 2, (31, 32, 33, 300)),              # ragged columns; rows around a tile of 32
    (104, 16, 1000, 1, (15, 65, 520, 1000, 3000)),   # every tile shape of a 1000-wide layer, none of them full
    (64, 64, 2056, 1, (127, 129, 300, 2000)),        # weights large enough for the taller ones
])
def test_mlp_rows_do_not_depend_on_the_tile_that_computes_them(d, E, width, blocks, rows, terms):
    """The network on row counts that go to different tile shapes: every shape adds an element's products in the same
    order, so the rows two calls share are equal bit for bit; the smallest and the largest call against the oracle
    (two terms: products of fp32 sums of 2056 terms of 2^-17 accuracy, 1e-4; one term: 2^-9, amplified, 5e-3)."""
    from oracle_helpers import mlp_model
    cfg = dict(kind="mlp", d=d, E=E, width=width, n_blocks=blocks, K=20, L=16, act_terms=terms)
    T, p, _ = oracle_setup(cfg)
    p["out_clip"] = 0.0
    ctx = runtime.open_ctx(cfg, p, seed=0, chains=-(-max(rows) // 16))
    rng = np.random.default_rng(5)
    x = rng.standard_normal((max(rows), d)).astype(np.float32)
    tau = rng.integers(1, cfg["K"] + 1, max(rows)).astype(np.int32)
    xd, td = torch.from_numpy(x).to(DEV), torch.from_numpy(tau).to(DEV)
    outs = []
    for n in rows:
        out = torch.full((n, d), float("nan"), dtype=torch.float32, device=DEV)
        ctx.denoise(xd[:n], td[:n], out)
        outs.append(out)
    torch.cuda.synchronize()
    ctx.close()
    for a, b in zip(outs, outs[1:]):
        assert torch.equal(a, b[:len(a)])
    n = min(len(x), 300)
    want = mlp_model(T, p)(cfg["K"] - tau[:n], x[:n].astype(np.float64))
    assert H.rel_err(outs[-1][:n].cpu().numpy(), want) <= (5e-3 if terms == 1 else 1e-4)


@pytest.mark.parametrize("d, L, batches", [
    (8, 37, (1, 3, 300, 600, 1100, 2100, 4100)),   # a wavefront a row: 16, 8, 4, 2, 1 of them share the slots
    (264, 37, (2, 600, 1100, 2100)),               # two wavefronts a row, the second nearly empty
    (1544, 9, (2, 300, 600)),                      # seven: two groups at most
    (4104, 5, (1, 20)),                            # more than a workgroup's threads
])
def test_round_kernels_do_not_depend_on_how_many_wavefronts_share_a_chain(d, L, batches):
    """Rounds through the stage calls in batches of sizes that share a chain's slots among more or fewer wavefronts: the
    chains two batches have in common are equal bit for bit (the network's rows do not depend on the batch)."""
    cfg = dict(kind="mlp", d=d, E=8, width=8, n_blocks=1, K=60, L=L, act_terms=2)
    T, p, _ = oracle_setup(cfg)
    runs = []
    for B in batches:
        ctx = runtime.open_ctx(cfg, p, seed=4, chains=B)
        g = torch.Generator(device=DEV).manual_seed(1)
        n = min(B, min(batches[1:]))
        y0 = torch.zeros(B, d, device=DEV)
        y0[:n] = torch.randn(n, d, generator=g, device=DEV)
        traj = torch.zeros(B, cfg["K"] + 1, d, device=DEV)
        traj[:, 0] = y0
        a = torch.zeros(B, dtype=torch.int32, device=DEV)
        x0hat = torch.zeros(B, L, d, device=DEV)
        acc = torch.zeros(4, B, dtype=torch.int32, device=DEV)
        for r in range(4):
            ctx.draft(traj, a)
            ctx.verify(traj, a, x0hat)
            ctx.accept(traj, a, x0hat, acc[r])
        torch.cuda.synchronize()
        ctx.close()
        runs.append((n, traj[:n].cpu(), a[:n].cpu(), acc[:, :n].cpu()))
    assert (runs[-1][3] >= 1).all() and len(set(runs[-1][3].flatten().tolist())) > 1
    for (n1, t1, a1, c1), (n2, t2, a2, c2) in zip(runs, runs[1:]):
        n = min(n1, n2)
        assert torch.equal(a1[:n], a2[:n]) and torch.equal(c1[:, :n], c2[:, :n])
        for i in range(n):
            assert torch.equal(t1[i, :int(a1[i]) + 1], t2[i, :int(a2[i]) + 1])


@pytest.mark.parametrize("chains", [3, 300, 700, 1200, 5000])      # 16, 8, 4, 2 and 1 groups of wavefronts a chain
def test_accept_statistics_end_with_the_group_of_the_first_rejection(chains):
    """asd_accept leaves the entries behind the group of eight slots that holds the first rejection as they were, however
    many slots it looks at together."""
    cfg = dict(kind="gmm", d=12, C=3, K=60, L=32, var=0.25)
    T, p, _ = oracle_setup(cfg)
    ctx = runtime.open_ctx(cfg, p, seed=6, chains=chains)
    K, L, d = cfg["K"], cfg["L"], cfg["d"]
    traj = torch.zeros(chains, K + 1, d, device=DEV)
    traj[:, 0] = torch.randn(chains, d, generator=torch.Generator(device=DEV).manual_seed(1), device=DEV)
    a = torch.zeros(chains, dtype=torch.int32, device=DEV)
    x0hat = torch.zeros(chains, L, d, device=DEV)
    acc = torch.zeros(chains, dtype=torch.int32, device=DEV)
    ends = set()
    for _ in range(5):
        before = a.cpu().numpy()
        stats = torch.full((chains, L, 4), -7.0, device=DEV)
        ctx.draft(traj, a)
        ctx.verify(traj, a, x0hat)
        ctx.accept(traj, a, x0hat, acc, stats)
        torch.cuda.synchronize()
        written = (stats.cpu().numpy() != -7.0).any(axis=2)
        for c in range(chains):
            w, n = min(L, K - before[c]), int(acc[c]) if before[c] < K else 0
            end = 0 if before[c] == K else w if n == w else min(w, n // 8 * 8 + 8)
            assert written[c, :end].all() and not written[c, end:].any(), (c, before[c], n)
            ends.add(end)
    ctx.close()
    assert 8 in ends and len(ends) > 2


@pytest.mark.parametrize("terms, width, chains", [(1, 2304, 5), (2, 2304, 5), (2, 2304, 33), (2, 2560, 24), (1, 2560, 64)])
def test_mlp_draft_call_of_few_rows_with_a_large_matrix(terms, width, chains):
    """The draft call of a few chains adds its sums over K in parts where the weights are large (parts of 18 and of 10
    slabs here: inside and across the stages of the kernel): the model values against those of asd_denoise, which adds
    in one part.  fp32 sums in another order, re-rounded to 2^-17 (2^-9 with one term) between layers: 1e-5, 2e-2."""
    cfg = dict(kind="mlp", d=64, E=16, width=width, n_blocks=2, K=20, L=2, act_terms=terms)
    T, p, _ = oracle_setup(cfg)
    p["out_clip"] = 0.0
    ctx = runtime.open_ctx(cfg, p, seed=0, chains=chains)
    g = torch.Generator(device=DEV).manual_seed(2)
    traj = torch.zeros(chains, cfg["K"] + 1, 64, device=DEV)
    traj[:, 0] = torch.randn(chains, 64, generator=g, device=DEV)
    a = torch.zeros(chains, dtype=torch.int32, device=DEV)
    x0hat = torch.zeros(chains, 2, 64, device=DEV)
    want = torch.zeros(chains, 64, device=DEV)
    ctx.denoise(traj[:, 0].contiguous(), torch.full((chains,), cfg["K"], dtype=torch.int32, device=DEV), want)
    ctx.draft(traj, a)
    ctx.verify(traj, a, x0hat)
    torch.cuda.synchronize()
    ctx.close()
    assert torch.isfinite(want).all()
    assert H.rel_err(x0hat[:, 0].cpu().numpy(), want.cpu().numpy()) <= (2e-2 if terms == 1 else 1e-5)


def test_mlp_weights_may_start_anywhere():
    """Weight matrices that are parts of a larger array, at an odd element: the same bits as from arrays of their own."""
    cfg = dict(kind="mlp", d=24, E=8, width=72, n_blocks=2, K=20, L=4, act_terms=2)
    T, p, _ = oracle_setup(cfg)
    x = torch.randn(37, 24, generator=torch.Generator(device=DEV).manual_seed(3), device=DEV)
    tau = torch.full((37,), 9, dtype=torch.int32, device=DEV)
    outs = []
    for shift in (0, 1):
        den = runtime.device_params(cfg, p)
        den["n_tau"] = cfg["K"] + 1
        for k in ("w_in", "w_blk", "w_out"):
            flat = torch.zeros(den[k].numel() + 8, dtype=den[k].dtype, device=DEV)
            flat[shift:shift + den[k].numel()] = den[k].flatten()
            den[k] = flat[shift:shift + den[k].numel()].view(den[k].shape)
        ctx = binding.Ctx(binding.asd_schedule_ddpm_linear(cfg["K"]), den, cfg["L"], 10)
        out = torch.zeros_like(x)
        ctx.denoise(x, tau, out)
        torch.cuda.synchronize()
        ctx.close()
        outs.append(out)
    assert bool(torch.isfinite(outs[0]).all()) and torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("d, C", [(64, 60), (128, 130), (96, 1056)])     # mixture in LDS; few rows; operands packed once
def test_mixture_means_may_start_anywhere(d, C):
    """Means that are part of a larger array, at an odd element: the same bits as from an array of their own."""
    cfg = dict(kind="gmm", d=d, C=C, K=20, L=64, var=0.25)
    T, p, _ = oracle_setup(cfg)
    n = 15000 if C == 1056 else 200
    x = torch.randn(n, d, generator=torch.Generator(device=DEV).manual_seed(3), device=DEV)
    tau = torch.full((n,), 9, dtype=torch.int32, device=DEV)
    sched = binding.asd_schedule_ddpm_linear(cfg["K"])
    outs = []
    for shift in (0, 1):
        den = runtime.device_params(cfg, p)
        flat = torch.zeros(C * d + 8, device=DEV)
        flat[shift:shift + C * d] = den["means"].flatten()
        den.update(n_tau=cfg["K"] + 1, abar=sched["abar"], means=flat[shift:shift + C * d].view(C, d))
        ctx = binding.Ctx(sched, den, cfg["L"], 240)
        out = torch.zeros_like(x)
        ctx.denoise(x, tau, out)
        torch.cuda.synchronize()
        ctx.close()
        outs.append(out)
    assert bool(torch.isfinite(outs[0]).all()) and torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("terms", [1, 2])
def test_split_sums_do_not_depend_on_the_kernel(terms):
    """Draft calls whose sums over K are added in parts: 24 rows take the kernel for few rows, which adds its parts in
    registers, 64 rows the 64 x 64 tiles and a second launch that adds them from memory, in the same four parts.  The rows
    they share are equal bit for bit."""
    cfg = dict(kind="mlp", d=64, E=16, width=4096, n_blocks=2, K=20, L=2, act_terms=terms)
    T, p, _ = oracle_setup(cfg)
    p["out_clip"] = 0.0
    y0 = torch.randn(64, 64, generator=torch.Generator(device=DEV).manual_seed(2), device=DEV)
    values = []
    for B in (24, 64):
        ctx = runtime.open_ctx(cfg, p, seed=0, chains=B)
        traj = torch.zeros(B, cfg["K"] + 1, 64, device=DEV)
        traj[:, 0] = y0[:B]
        a = torch.zeros(B, dtype=torch.int32, device=DEV)
        x0hat = torch.zeros(B, 2, 64, device=DEV)
        ctx.draft(traj, a)
        ctx.verify(traj, a, x0hat)
        torch.cuda.synchronize()
        ctx.close()
        values.append(x0hat[:24, 0].clone())
    assert bool(torch.isfinite(values[0]).all()) and torch.equal(values[0], values[1])


@pytest.mark.parametrize("d, E, width, blocks, K, L, chains, terms, eps", [
    (112, 16, 1024, 2, 60, 16, 256, 2, False),      # the draft kernel packs what it lists; accept chunks as long as a window
    (264, 24, 1024, 1, 90, 37, 200, 1, False),      # rows of two wavefronts, packed by a kernel of its own; chunks of eight slots
    (1032, 16, 2056, 1, 50, 24, 64, 2, False),      # a draft call that is split over K
    (16, 8, 2048, 2, 40, 7, 2200, 2, False),        # a wavefront a chain throughout
    (112, 16, 1024, 2, 60, 16, 256, 2, True),       # a network that estimates the noise: its values also take the rows evaluated
])
def test_windows_in_pieces_change_no_bit(d, E, width, blocks, K, L, chains, terms, eps):
    """Whole samples with windows taken in pieces and whole, as graphs and plain launches: the same trajectories, round
    counts and number of rounds, from fewer model rows."""
    cfg = dict(kind="mlp", d=d, E=E, width=width, n_blocks=blocks, K=K, L=L, act_terms=terms)
    _, p, _ = oracle_setup(cfg)
    p["predict_eps"] = eps
    ctx = runtime.open_ctx(cfg, p, seed=0, chains=chains)
    runs = []
    for pieces, graphs, profile in ((False, True, False), (True, True, False), (True, False, False), (False, True, True), (True, True, True)):
        ctx.use_window_pieces(pieces)
        ctx.use_graphs(graphs)
        ctx.profile_enable(profile)
        ctx.set_seed(6)
        traj = torch.full((chains, K + 1, d), float("nan"), device=DEV)
        rounds = torch.zeros(chains, dtype=torch.int32, device=DEV)
        n = ctx.sample(traj, rounds)
        torch.cuda.synchronize()
        runs.append((traj, rounds, n, ctx.profile_rows()))
    ctx.close()
    traj, rounds, n, _ = runs[0]
    assert bool(torch.isfinite(traj).all()) and n == int(rounds.max())
    for t, r, m, _ in runs[1:]:
        assert m == n and torch.equal(r, rounds) and torch.equal(t, traj)
    (starts, whole), (starts_p, pieces) = runs[3][3], runs[4][3]
    assert starts == starts_p == int(rounds.sum()) and pieces < 0.8 * whole


@pytest.mark.parametrize("graphs", [True, False])
def test_controlled_windows_do_not_depend_on_the_rows_a_round_is_launched_for(graphs):
    """Rounds are launched in forms for the rows the round but one before brought, 4, 8, 16, 32 a chain or the most there can
    be, each with its own tiles.  A batch goes through them in its own time: the chains two batches share are equal bit for
    bit, trajectory and rounds."""
    cfg = dict(kind="mlp", d=264, E=24, width=1032, n_blocks=2, K=120, L=48, act_terms=1, predict_eps=True)
    _, p, _ = oracle_setup(cfg)
    runs = []
    for chains in (150, 3):
        ctx = runtime.open_ctx(cfg, p, seed=3, chains=chains)
        ctx.use_adaptive_window(True)
        ctx.use_graphs(graphs)
        traj, rounds = torch.full((chains, 121, 264), float("nan"), device=DEV), torch.zeros(chains, dtype=torch.int32, device=DEV)
        assert ctx.sample(traj, rounds) == int(rounds.max())
        ctx.close()
        runs.append((traj[:3].clone(), rounds[:3].clone()))
    assert bool(torch.isfinite(runs[0][0]).all())
    assert torch.equal(runs[0][0], runs[1][0]) and torch.equal(runs[0][1], runs[1][1])


@pytest.mark.parametrize("K, taken", [(80, True), (300, False)])
def test_windows_are_whole_where_pieces_would_cost_more(K, taken):
    """A piece's products are on the kernel for whole windows' rows: it pays on a coarse schedule, whose windows end after two
    slots, and not on a fine one (measured 1.08 times slower)."""
    cfg = dict(kind="mlp", d=48, E=16, width=648, n_blocks=5, K=K, L=14, act_terms=2)
    _, p, _ = oracle_setup(cfg)
    ctx = runtime.open_ctx(cfg, p, seed=0, chains=48)
    rows = []
    for pieces in (True, False):
        ctx.use_window_pieces(pieces)
        ctx.profile_enable(True)
        ctx.set_seed(6)
        ctx.sample(torch.empty((48, K + 1, 48), device=DEV))
        torch.cuda.synchronize()
        rows.append(ctx.profile_rows()[1])
    ctx.close()
    assert (rows[0] < rows[1]) == taken and rows[0] <= rows[1]


@pytest.mark.parametrize("d, C, L, K, chains, adaptive", [
    (1, 1, 1, 3, 2, False),           # nothing but a step
    (2, 4, 8, 40, 5, False),
    (3, 7, 5, 30, 300, True),         # lanes without a component; two chains a workgroup
    (5, 40, 16, 40, 4, False),        # two blocks of coordinates, the second mostly padding
    (9, 16, 3, 25, 600, False),       # three; windows shorter than the lanes' slots; three chains a workgroup
    (16, 8, 17, 50, 3, True),         # two lanes a slot
    (13, 5, 64, 70, 3, False),        # a lane a slot; windows nearly as long as the chain
    (4, 6, 12, 1000, 2100, False),    # as many chains a workgroup as LDS holds
])
def test_samples_of_a_wavefront_per_chain(d, C, L, K, chains, adaptive):
    """Whole samples of mixtures of a few numbers against the oracle, chain by chain (1e-4, the bar of fp32 denoisers)."""
    cfg = dict(kind="gmm", d=d, C=C, K=K, L=L, var=0.25)
    T, p, model = oracle_setup(cfg)
    ctx = runtime.open_ctx(cfg, p, seed=8, chains=chains)
    assert ctx.resident_active()
    ctx.use_adaptive_window(adaptive)
    traj = torch.full((chains, K + 1, d), float("nan"), device=DEV)
    rounds = torch.zeros(chains, dtype=torch.int32, device=DEV)
    n = ctx.sample(traj, rounds)
    y0 = traj[:, 0].clone()
    given = torch.full_like(traj, float("nan"))
    assert ctx.sample(given, None, y0) == n == int(rounds.max())
    ctx.close()
    assert bool(torch.isfinite(traj).all()) and torch.equal(traj, given)
    for c in sorted({0, 1, chains // 2, chains - 1}):
        f = H.follow_chain(cfg, T, model, 8, c, traj[c].cpu().numpy(), 1e-4, adaptive=adaptive)
        assert H.rel_err(traj[c].cpu().numpy(), f["y"]) <= 1e-4
        assert int(rounds[c]) == f["R"]


@pytest.mark.parametrize("d, C, L, K, chains, adaptive, empty", [
    (3, 300, 2, 9, 2, False, 0),      # more tiles of components than wavefronts
    (20, 66, 9, 25, 2, False, 16),    # a tile of components that weigh nothing
    (64, 128, 17, 40, 3, True, 0),    # one tile of rows, full
    (70, 129, 18, 60, 3, False, 33),  # two, the second of one row; a thread has no coordinate, one component alone in a tile
    (33, 97, 64, 90, 2, False, 0),    # logits through LDS, a ring of one window's noise
    (128, 20, 33, 150, 2, False, 0),  # ... and logits that stay in registers
    (260, 8, 5, 21, 2, False, 0),     # more coordinates than threads
])
def test_samples_of_a_workgroup_per_chain(d, C, L, K, chains, adaptive, empty):
    """The same for mixtures a workgroup holds; the first components may weigh nothing (the oracle leaves them out)."""
    cfg = dict(kind="gmm", d=d, C=C, K=K, L=L, var=0.25)
    T, p, _ = oracle_setup(cfg)
    model = gmm_model(T, dict(p, means=p["means"][empty:], log_w=p["log_w"][empty:]))
    p["log_w"][:empty] = -np.inf
    ctx = runtime.open_ctx(cfg, p, seed=8, chains=chains)
    assert ctx.resident_active()
    ctx.use_adaptive_window(adaptive)
    traj = torch.full((chains, K + 1, d), float("nan"), device=DEV)
    rounds = torch.zeros(chains, dtype=torch.int32, device=DEV)
    n = ctx.sample(traj, rounds)
    ctx.close()
    assert bool(torch.isfinite(traj).all()) and n == int(rounds.max())
    for c in range(chains):
        f = H.follow_chain(cfg, T, model, 8, c, traj[c].cpu().numpy(), 1e-4, adaptive=adaptive)
        assert H.rel_err(traj[c].cpu().numpy(), f["y"]) <= 1e-4
        assert int(rounds[c]) == f["R"]


@pytest.mark.parametrize("d, E, width, blocks, chains, terms, eps", [
    (8, 24, 64, 1, 3, 2, False),         # an embedding longer than the row; one tile of 16 rows
    (40, 8, 512, 2, 100, 1, True),       # ragged columns, tiles of 32 rows, a noise-predicting network
    (104, 16, 520, 1, 1100, 2, False),   # the tiles of many rows
    (64, 16, 2304, 1, 5, 2, True),       # sums in parts, added in registers
    (72, 16, 2560, 1, 64, 1, False),     # ... and in a launch of their own (few rows of the output layer)
    (2560, 8, 2560, 1, 64, 2, False),    # ... the output layer's too
])
def test_sequential_steps_of_a_network(d, E, width, blocks, chains, terms, eps):
    """The step taken by the output layer against windows of one slot, whose draft call and draft kernel take it on their
    own: the same chains bit for bit."""
    cfg = dict(kind="mlp", d=d, E=E, width=width, n_blocks=blocks, K=7, L=1, act_terms=terms)
    _, p, _ = oracle_setup(cfg)
    p["predict_eps"] = eps
    ctx = runtime.open_ctx(cfg, p, seed=5, chains=chains)
    one, seq = (torch.full((chains, cfg["K"] + 1, d), float("nan"), device=DEV) for _ in range(2))
    ctx.sample(one)
    ctx.sample_sequential(seq)
    ctx.close()
    assert bool(torch.isfinite(one).all()) and torch.equal(one, seq)


@pytest.mark.parametrize("d, C, n", [
    (1000, 4000, 1001),     # a quarter of the last slab of d; whole slabs of C
    (516, 1060, 5000),      # an eighth of the last slab of d and of C; a row, column and component tile with four in it
    (512, 2052, 4100),      # whole slabs of d
    (2052, 516, 2000),
])
def test_mixture_sums_padded_to_whole_slabs(d, C, n):
    """d or C no multiple of 16: fp16 terms, their sums padded to whole slabs, against the oracle (the bound of the tiled kernels
    above) and against its 64 bits summed over the call: an fp32 sum of K products in K / 16 steps or more, each rounded by 2^-24
    of a partial sum, errs by 2^-24 sqrt(K / 16) of it or so, twice as the two sums meet, and the logits' errors reach the
    weights times their size, a few tens here.  A call does not depend on the rows behind it."""
    cfg = dict(kind="gmm", d=d, C=C, K=50, L=16, var=0.25)
    on, want = _denoise(cfg, n, tiled=True, split=True)
    off, _ = _denoise(cfg, n, keep=n, tiled=True, split=False)
    for got in (on, off):
        assert H.rel_err(got, want) <= 3e-5
        assert np.linalg.norm(got - want) / np.linalg.norm(want) <= 2.0 ** -24 * np.sqrt(max(d, C) / 16) * 4
    assert not np.array_equal(on, off)
    first, _ = _denoise(cfg, n, keep=n - 130, tiled=True, split=True)
    assert np.array_equal(first, on[:n - 130])


@pytest.mark.parametrize("d, C", [(100, 400), (60, 516), (36, 2052)])
def test_mixtures_no_call_of_which_is_padded_hold_no_terms(d, C):
    """Ragged sizes whose sums are faster on fp32 tiles at any number of rows: nothing to switch on."""
    cfg = dict(kind="gmm", d=d, C=C, K=50, L=16, var=0.25)
    _, p, _ = oracle_setup(cfg)
    ctx = runtime.open_ctx(cfg, p, chains=750)
    ctx.use_split_gemm(True)
    assert not ctx.split_gemm_active()
    ctx.close()


@pytest.mark.parametrize("change", ["component", "coordinate"])
def test_mixtures_of_mixed_size_stay_on_fp32(change):
    """One component, or one coordinate, a millionth of the others: fp16 terms that share a scale would keep a few of its bits
    only.  The context has none to switch on, and the call is the one with the switch off, bit for bit."""
    def shrink(m):
        m = m.copy()
        m[(17 if change == "component" else slice(None)), (slice(None) if change == "component" else 5)] *= 1e-6
        return m
    cfg = dict(kind="gmm", d=516, C=1060, K=50, L=16, var=0.25)
    _, p, _ = oracle_setup(cfg)
    ctx = runtime.open_ctx(cfg, dict(p, means=shrink(p["means"])), chains=-(-5000 // 16))
    ctx.use_split_gemm(True)
    assert not ctx.split_gemm_active()
    ctx.close()
    got, want = _denoise(cfg, 5000, tiled=True, change=shrink)
    off, _ = _denoise(cfg, 5000, keep=5000, tiled=True, split=False, change=shrink)
    assert H.rel_err(got, want) <= 3e-5 and np.array_equal(got, off)


@pytest.mark.parametrize("d, C", [(516, 1060), (96, 1056)])
def test_rows_near_the_largest_float_on_split_operands(d, C):
    """Points of up to 1e36 among ordinary ones: their terms are scaled into fp16's range like any other's, and what the model
    adds to c_x' x is lost in its rounding."""
    cfg = dict(kind="gmm", d=d, C=C, K=50, L=16, var=0.25)
    T, p, _ = oracle_setup(cfg)
    n, far = 4100, [0, 1, 130, 4099]
    ctx = runtime.open_ctx(cfg, p, chains=-(-n // 16))
    ctx.use_few_rows(False)
    assert ctx.split_gemm_active()
    x = np.random.default_rng(4).standard_normal((n, d)).astype(np.float32)
    near = x.copy()
    x[far] *= np.array([1e34, 6e34, 1e35, 2e35], dtype=np.float32)[:, None]
    tau = np.full(n, 25, dtype=np.int32)
    outs = []
    for rows in (x, near):
        out = torch.full((n, d), float("nan"), dtype=torch.float32, device=DEV)
        ctx.denoise(torch.from_numpy(rows).to(DEV), torch.from_numpy(tau).to(DEV), out)
        outs.append(out.cpu().numpy())
    ctx.close()
    ab = T["abar"][25]
    cx = np.sqrt(ab) * p["var"] / (ab * p["var"] + 1 - ab)
    want = cx * x[far].astype(np.float64)
    assert np.abs(outs[0][far] - want).max() <= 1e-6 * np.abs(want).max() and np.isfinite(outs[0]).all()
    keep = np.setdiff1d(np.arange(n), far)
    assert np.array_equal(outs[0][keep], outs[1][keep])


def test_samples_of_a_ragged_mixture_on_split_operands():
    """Whole samples whose verify calls take padded fp16 terms, on fewer rows than there may be once windows are cut and chains
    end, against the oracle chain by chain (1e-4, the bar of fp32 denoisers)."""
    cfg = dict(kind="gmm", d=300, C=1000, K=70, L=32, var=0.25)
    T, p, model = oracle_setup(cfg)
    chains = 256
    ctx = runtime.open_ctx(cfg, p, seed=9, chains=chains)
    traj, rounds = torch.full((chains, 71, 300), float("nan"), device=DEV), torch.zeros(chains, dtype=torch.int32, device=DEV)
    ctx.profile_enable(True)
    n = ctx.sample(traj, rounds)
    taken = ctx.profile_read(binding.PROF["GMM_SOFTMAX"], 1)[0]
    ctx.close()
    assert taken >= n and bool(torch.isfinite(traj).all())
    for c in (0, 100, chains - 1):
        f = H.follow_chain(cfg, T, model, 9, c, traj[c].cpu().numpy(), 1e-4)
        assert H.rel_err(traj[c].cpu().numpy(), f["y"]) <= 1e-4
        assert int(rounds[c]) == f["R"]
