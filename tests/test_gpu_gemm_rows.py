"""The bf16 projections at the row counts where another tile takes over, and with shapes whose
column tiles, K splits and row tails are ragged, against the CPU oracle."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import dpara_oracle as O  # noqa: E402
from paper_2609_27396_amd import synth  # noqa: E402

pytestmark = pytest.mark.gpu

TOL = 2e-2  # the bf16 bar of test_gpu_parity
# K of a fusion is 3 * hidden: 384 (three 128-deep steps) and 960 (no multiple of 128)
ROWS = [64, 65, 128, 129, 192, 193, 320, 321, 385, 513]


def _say(*a):
    print(*a, file=sys.stderr, flush=True)


def _shape(hidden, ffn, vocab, gamma, layers=1):
    return synth.DrafterShape(n_layers=layers, hidden=hidden, n_q_heads=4, n_kv_heads=2, head_dim=128, ffn=ffn,
                              vocab=vocab, gamma=gamma, ar_rank=64, qk_norm=True, dtype="bf16")


@pytest.mark.parametrize("hidden", [128, 320])
def test_fused_features_around_tile_edges(hidden):
    from paper_2609_27396_amd import dpara as D
    s = _shape(hidden, 256, 500, 4)
    wf = synth.make_fusion_weights(s, n_feat=3, seed=21, gain_jitter=0.1)
    fus = D.DeviceFusion(s, wf, 3)
    for n in ROWS:
        _say("case fuse", hidden, n)
        hid = synth.make_target_hidden(s, n, n_feat=3, seed=22 + n)
        out = torch.empty((n, hidden), dtype=torch.bfloat16, device="cuda")
        ws = torch.empty(D.dpara_fuse_workspace_bytes(fus.cfg, n, 3), dtype=torch.uint8, device="cuda")
        D.fuse_features(fus, torch.from_numpy(hid).to(device="cuda", dtype=torch.bfloat16), out, ws)
        torch.cuda.synchronize()
        ref = O.fuse_features(s, wf, hid, "bf16")
        # one bf16 rounding, and the float32 summation error of a 3H-term projection near zero
        assert np.all(np.abs(out.float().cpu().numpy() - ref) <= 2.0 ** -7 * np.abs(ref) + 1e-4), n


# two row tiles over K split eight ways (29 units of 128, dealt unevenly); the last column tile is half full
@pytest.mark.parametrize("n", [192, 193, 289, 319, 320, 321])
def test_fused_features_of_two_row_tiles(n):
    from paper_2609_27396_amd import dpara as D
    s = _shape(1856, 256, 500, 4)
    wf = synth.make_fusion_weights(s, n_feat=2, seed=31, gain_jitter=0.1)
    fus = D.DeviceFusion(s, wf, 2)
    _say("case fuse 1856", n)
    hid = synth.make_target_hidden(s, n, n_feat=2, seed=32 + n)
    out = torch.empty((n, s.hidden), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(D.dpara_fuse_workspace_bytes(fus.cfg, n, 2), dtype=torch.uint8, device="cuda")
    D.fuse_features(fus, torch.from_numpy(hid).to(device="cuda", dtype=torch.bfloat16), out, ws)
    torch.cuda.synchronize()
    ref = O.fuse_features(s, wf, hid, "bf16")
    # one bf16 rounding, and the float32 summation error of a 2H-term projection near zero
    assert np.all(np.abs(out.float().cpu().numpy() - ref) <= 2.0 ** -7 * np.abs(ref) + 1e-4), n


# requests of 17 block rows: 68, 119 | 136, 187 | 204, 255 | 272, 306 | 323, 391 rows.  hidden 384 is
# three 128-deep K steps; ffn 640 and vocab 3001 leave ragged column tiles at every tile width
@pytest.mark.parametrize("batch", [4, 7, 8, 11, 12, 15, 16, 18, 19, 23])
def test_target_rows_around_tile_edges(batch):
    from paper_2609_27396_amd import dpara as D
    from paper_2609_27396_amd.harness import upload_cache
    s = _shape(384, 640, 3001, 16, layers=2)
    lens = [(29 * i) % 70 for i in range(batch)]
    _say("case target rows", batch * 17)
    w = synth.make_target_weights(s, seed=7, gain_jitter=0.1)
    k, v = synth.make_target_cache(s, lens, seed=8)
    block = np.random.default_rng(batch).integers(0, s.vocab, (batch, 17)).astype(np.int32)
    t = D.DeviceTarget(s, w)
    ctx = D.DeviceContext(s, batch, 128)
    upload_cache(ctx, k, v, lens, torch.bfloat16)
    ws = D.Workspace(t.cfg, batch, 128, target=True)
    lf = torch.empty((batch, 17, s.vocab), dtype=torch.float32, device="cuda")
    lb = torch.empty_like(lf, dtype=torch.bfloat16)
    D.target_forward(t, ctx, torch.from_numpy(block).cuda(), lf, ws)
    D.target_forward(t, ctx, torch.from_numpy(block).cuda(), lb, ws)
    torch.cuda.synchronize()
    for b in sorted({0, batch // 2, batch - 1}):
        ref = O.target_forward(s, w, [k[l][b] for l in range(2)], [v[l][b] for l in range(2)], block[b], "bf16")
        assert np.abs(lf[b].cpu().numpy() - ref).max() <= TOL, b
    # bf16 logits are the float32 logits rounded once
    np.testing.assert_allclose(lb.float().cpu().numpy(), lf.cpu().numpy(), rtol=2 ** -8, atol=0)


def candidates_are_the_plain_head(batch, gamma, hidden):
    from paper_2609_27396_amd import dpara as D
    s = _shape(hidden, 256, 3000, gamma)
    _say("case candidate rows", batch * (gamma + 1) * gamma)
    w = synth.make_weights(s, seed=6, gain_jitter=0.1, ar_w_std=0.005, ar_e_std=0.02)
    dd = D.DeviceDrafter(s, w)
    ws = D.Workspace(dd.cfg, batch, 64)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(batch)
    reps = torch.empty((batch, gamma + 1, gamma, s.hidden), dtype=torch.float32, device="cuda").normal_(generator=gen)
    rng = np.random.default_rng(gamma)
    acc = torch.from_numpy(rng.integers(0, gamma + 1, batch).astype(np.int32)).cuda()
    bon = torch.from_numpy(rng.integers(0, s.vocab, batch).astype(np.int32)).cuda()

    def outs():
        return (torch.empty((batch, gamma, s.hidden), dtype=torch.float32, device="cuda"),
                torch.empty((batch, gamma), dtype=torch.int32, device="cuda"),
                torch.empty((batch, gamma + 1), dtype=torch.int32, device="cuda"),
                torch.empty((batch, gamma), dtype=torch.float32, device="cuda"))

    a, b = outs(), outs()
    D.select_and_head(dd, reps, acc, bon, *a, ws)
    torch.cuda.synchronize()
    assert ws.status() == 0 and ws.head_fallback() == 0
    cand = D.branch_candidates_buffer(dd, batch)
    D.branch_candidates(dd, reps, cand, ws)
    D.select_and_head_cand(dd, reps, cand, acc, bon, *b, ws)
    torch.cuda.synchronize()
    assert ws.status() == 0 and ws.head_fallback() == 0
    for x, y in zip(a, b):
        assert torch.equal(x, y)


# branch rows batch * (gamma + 1) * gamma: 72, 126 | 144, 180 | 198, 252 | 270, 320 | 360
@pytest.mark.parametrize("batch,gamma", [(6, 3), (3, 6), (2, 8), (9, 4), (1, 13), (6, 6), (3, 9), (16, 4), (4, 9)])
def test_candidate_rows_around_tile_edges(batch, gamma):
    """Candidates of every branch row, then the serial step: where every step is proven, bit for
    bit the plain head (whose rows are at most 64 here and take another kernel)."""
    candidates_are_the_plain_head(batch, gamma, 256)


def append_is_its_short_appends(layers, starts, counts, n_max, cap, step, hidden):
    from paper_2609_27396_amd import dpara as D
    B = len(starts)
    assert B * n_max > 320 and B * step <= 320
    s = synth.DrafterShape(n_layers=layers, hidden=hidden, n_q_heads=4, n_kv_heads=2, head_dim=128, ffn=256, vocab=500,
                           gamma=4, ar_rank=64, qk_norm=True, dtype="bf16")
    _say("case prompt append", layers, B, n_max)
    dd = D.DeviceDrafter(s, synth.make_weights(s, seed=31, gain_jitter=0.1))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(layers)
    feats = torch.empty((B, n_max, s.hidden), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)

    def run(step):
        ctx = D.DeviceContext(s, B, cap)
        ctx.k.fill_(7.0)
        ctx.v.fill_(-7.0)
        ctx.ctx_len.copy_(torch.tensor(starts, dtype=torch.int32))
        ws = D.Workspace(dd.cfg, B, cap)
        for c0 in range(0, n_max, step):
            n = min(step, n_max - c0)
            new = torch.tensor([c if c < 0 else min(max(c - c0, 0), n) for c in counts], dtype=torch.int32, device="cuda")
            D.ctx_append(dd, ctx, feats[:, c0:c0 + n].contiguous(), new, ws)
        torch.cuda.synchronize()
        return ctx, ws.status()

    one, status = run(n_max)
    ref, ref_status = run(step)
    assert status == ref_status
    assert torch.equal(one.ctx_len, ref.ctx_len)
    for a, b, mark in ((one.k, ref.k, 7.0), (one.v, ref.v, -7.0)):
        assert torch.equal(a == mark, b == mark)
        a, b = a.float(), b.float()
        assert bool(((a - b).abs() <= 2.0 ** -7 * b.abs() + 1e-5).all())


# rows of one append: just above 320, row tiles of padding only, two layer groups, an append past the
# cache's end, and more rows than one launch takes
@pytest.mark.parametrize("layers,starts,counts,n_max,cap,step", [
    (2, [0, 3, 0], [107, 1, 106], 107, 128, 53),
    (9, [5, 0, 70, 9], [700, 0, 133, -2], 700, 640, 70),
    (1, [1, 64], [9000, 4097], 9000, 9088, 160),
])
def test_prompt_append_is_its_short_appends(layers, starts, counts, n_max, cap, step):
    """A prompt's rows appended at once (one projection that writes the caches) against the same
    rows in appends of at most 320 rows (projection, then a store pass): lengths equal, entries
    nobody appended untouched, the others within one bf16 rounding (float32 sums in another order)."""
    append_is_its_short_appends(layers, starts, counts, n_max, cap, step, 384)


# more than 320 rows, rows x columns at most 800 (K - 300): K split into planes, over all rows at once; an append past the cache's end, and two layer groups
@pytest.mark.parametrize("layers,starts,counts,n_max,cap,step,hidden", [
    (1, [0, 3, 0], [200, 1, 190], 200, 256, 100, 1024),
    (2, [5, 0, 70], [190, 0, 188], 190, 256, 53, 1024),
    (9, [0, 3], [250, -2], 250, 256, 125, 4096),
])
def test_append_of_few_columns_is_its_short_appends(layers, starts, counts, n_max, cap, step, hidden):
    append_is_its_short_appends(layers, starts, counts, n_max, cap, step, hidden)


# batch * gamma rows: 15, 64 | 66, 128 | 135, 192 | 198, 256 | 260, 320
@pytest.mark.parametrize("batch,gamma", [(3, 5), (16, 4), (11, 6), (16, 8), (15, 9), (16, 12), (18, 11), (16, 16), (20, 13),
                                         (20, 16)])
def test_sampled_scores_around_tile_edges(batch, gamma):
    """Draft scores of the sampled head where every step is proven, rank 256, a vocabulary that is no
    multiple of four: (h . E_v + E(y_prev) . W_v) / T against float64."""
    from paper_2609_27396_amd import dpara as D
    s = synth.DrafterShape(n_layers=1, hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=128, ffn=256, vocab=3001,
                           gamma=gamma, ar_rank=256, qk_norm=True, dtype="bf16")
    _say("case sampled scores", batch * gamma)
    w = synth.make_weights(s, seed=6, gain_jitter=0.1, ar_w_std=0.005, ar_e_std=0.02)
    dd = D.DeviceDrafter(s, w)
    ws = D.Workspace(dd.cfg, batch, 64)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(batch)
    reps = torch.empty((batch, gamma + 1, gamma, s.hidden), dtype=torch.float32, device="cuda").normal_(generator=gen)
    rng = np.random.default_rng(gamma)
    acc = torch.from_numpy(rng.integers(0, gamma + 1, batch).astype(np.int32)).cuda()
    bon = torch.from_numpy(rng.integers(0, s.vocab, batch).astype(np.int32)).cuda()
    drafts = torch.empty((batch, gamma), dtype=torch.int32, device="cuda")
    nsp = torch.empty((batch, gamma + 1), dtype=torch.int32, device="cuda")
    scores = torch.full((batch, gamma, s.vocab), float("nan"), dtype=torch.float32, device="cuda")
    D.select_and_head_sampled(dd, reps, acc, bon, None, drafts, nsp, None, 0.7, 11, scores, ws)
    torch.cuda.synchronize()
    assert ws.status() == 0 and ws.head_fallback() == 0
    bf = lambda x: torch.from_numpy(np.asarray(x, np.float32)).to(torch.bfloat16).double()  # noqa: E731
    h = torch.stack([reps[b, int(acc[b])] for b in range(batch)]).cpu().double()
    prev = nsp[:, :gamma].cpu().long()
    ref = (h @ bf(w["embed"]).T + bf(w["ar_E"])[prev] @ bf(w["ar_W"]).T) / 0.7
    # h as bf16 hi + lo parts: 2^-16 of the products' magnitudes (256 of about 0.8 * 0.016)
    assert (scores.cpu().double() - ref).abs().max() <= 1e-3


# hidden and ffn that are multiples of 64 but not of the K stages of the kernels for few rows: the
# gate/up product of at most 64 rows takes 128-deep stages, the two-plane head 256-deep ones up to
# 16 rows and 128-deep ones up to 32.  Block rows 25, 50 | 147, head rows 4, 8 | 18
@pytest.mark.parametrize("hidden,ffn,gamma,ctx", [(64, 64, 4, [20]), (128, 320, 4, [20, 0]), (320, 576, 4, [70]),
                                                  (320, 320, 6, [0, 77, 30]), (384, 640, 4, [70, 5])])
def test_rounds_of_every_hidden_multiple_of_64(hidden, ffn, gamma, ctx):
    from test_gpu_parity import check_head, check_verify, run_full
    s = synth.DrafterShape(n_layers=2, hidden=hidden, n_q_heads=4, n_kv_heads=2, head_dim=64, ffn=ffn, vocab=3001,
                           gamma=gamma, ar_rank=64, qk_norm=True, dtype="bf16")
    _say("case round", hidden, ffn, gamma, ctx)
    wl = synth.Workload("multiple_of_64", s, batch=len(ctx), ctx_min=0, ctx_max=0, p_reject=0.3, seed_in=7)
    w = synth.make_weights(s, seed=3, gain_jitter=0.1, ar_e_std=1.0)
    ri = synth.make_round(wl, ctx_lens=ctx)
    dr = run_full(wl, w, ri)
    check_verify(ri, dr)
    for b in range(len(ctx)):
        ref = O.backbone_all_boundaries(s, w, ri.ctx_feats[b], ri.spine[b], "bf16")["reps"]
        assert np.abs(dr.reps[b].cpu().numpy() - ref).max() <= TOL, b
        check_head(s, w, dr, "bf16", b)


# more than 1024 rows of products the persistent kernel does not take (K = 64 mod 128): 128 x 128
# tiles; whole rounds of 256 x 256 and a second launch for the last columns; 256 x 256; 192 x 256
@pytest.mark.parametrize("hidden,n", [(320, 1025), (4160, 4096), (2880, 4096), (8128, 2400)])
def test_fused_features_above_1024_rows(hidden, n):
    from paper_2609_27396_amd import dpara as D
    s = _shape(hidden, 256, 500, 4)
    wf = synth.make_fusion_weights(s, n_feat=1, seed=41, gain_jitter=0.1)
    fus = D.DeviceFusion(s, wf, 1)
    _say("case fuse above 1024", hidden, n)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(hidden)
    hid = torch.empty((n, hidden), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    out = torch.empty((n, hidden), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(D.dpara_fuse_workspace_bytes(fus.cfg, n, 1), dtype=torch.uint8, device="cuda")
    D.fuse_features(fus, hid, out, ws)
    x = hid.double() @ torch.from_numpy(wf["fc"]).cuda().double().T
    ref = x / torch.sqrt((x * x).mean(-1, keepdim=True) + s.rms_eps) * torch.from_numpy(wf["fc_norm"]).cuda().double()
    assert bool(((out.double() - ref).abs() <= 2.0 ** -7 * ref.abs() + 1e-4).all())


# block rows 1152 and 2601 of shapes the persistent kernel does not take: K = 64 mod 128 (the second
# with 192-row tiles for Q|K|V and a gate/up product in two launches), one 128-wide and two 64-wide
# KV heads; then of shapes it takes: its Q|K|V epilogue over 1152, 1183 and 2601 rows (last row tiles of
# 128, 159 or 31 and 41 rows), and below that split-K planes of Q|K|V (338 rows, K 1024) and 64-row
# tiles for Q|K|V and gate/up (338 and 1014 rows, K 256)
@pytest.mark.parametrize("hidden,ffn,nq,nkv,hd,gamma,batch", [
    (192, 320, 4, 2, 128, 11, 8), (192, 3136, 14, 2, 128, 16, 9), (256, 384, 3, 1, 128, 11, 8), (256, 384, 4, 2, 64, 11, 8),
    (256, 384, 4, 2, 128, 11, 8), (384, 640, 4, 2, 128, 12, 7), (256, 384, 4, 2, 128, 16, 9),
    (1024, 512, 4, 2, 128, 12, 2), (256, 384, 4, 2, 128, 12, 2), (256, 384, 4, 2, 128, 12, 6)])
def test_backbone_rows(hidden, ffn, nq, nkv, hd, gamma, batch):
    from paper_2609_27396_amd.harness import DeviceRound
    s = synth.DrafterShape(n_layers=1, hidden=hidden, n_q_heads=nq, n_kv_heads=nkv, head_dim=hd, ffn=ffn, vocab=1000,
                           gamma=gamma, ar_rank=64, qk_norm=True, dtype="bf16")
    _say("case backbone rows", hidden, ffn, nq, nkv, hd)
    ctx = [(61 * i + 5) % 190 for i in range(batch)]
    wl = synth.Workload("rows", s, batch=batch, ctx_min=0, ctx_max=0, p_reject=0.3, seed_in=7)
    w = synth.make_weights(s, seed=3, gain_jitter=0.1)
    ri = synth.make_round(wl, ctx_lens=ctx)
    dr = DeviceRound(s, w, ri)
    dr.backbone()
    assert dr.status() == 0
    for b in (0, batch // 2, batch - 1):
        ref = O.backbone_all_boundaries(s, w, ri.ctx_feats[b], ri.spine[b], "bf16")["reps"]
        assert np.abs(dr.reps[b].cpu().numpy() - ref).max() <= TOL, b


# candidates and the plain head where K is no multiple of 128; branch rows 252 (one 256-row tile), 360,
# 1620 (256 x 256 tiles); head rows 36, 36, 162 (one 256-row tile of two planes)
@pytest.mark.parametrize("batch,gamma", [(6, 6), (4, 9), (18, 9)])
def test_candidates_with_hidden_192(batch, gamma):
    candidates_are_the_plain_head(batch, gamma, 192)


# requests of 42 branch rows: one at a time they are ranked by the kernel for at most 64 rows, which
# inserts a key for every logit; 84, 168, 252 | 294, 336 rows take the three largest values of a tile by
# medians first
@pytest.mark.parametrize("batch", [2, 4, 6, 7, 8])
def test_candidates_with_ties_and_values_that_are_not_finite(batch):
    """Equal leaders (two and three equal embedding rows in one full 128-column tile, equal rows in two
    tiles, a tile and a row of zeros), infinities and NaN: every row's candidates and bound are bit for
    bit those of its request alone."""
    from paper_2609_27396_amd import dpara as D
    gamma, V = 6, 3000
    s = _shape(256, 256, V, gamma)
    _say("case ties", batch)
    w = synth.make_weights(s, seed=6, gain_jitter=0.1, ar_w_std=0.005, ar_e_std=0.02)
    E = w["embed"]
    E[700], E[703], E[701] = E[650], E[650], E[651]  # columns 640 .. 767: three, and two
    E[131], E[1500] = E[130], E[130]                 # two in one tile, the third in another
    E[2304:2432] = 0                                 # one whole tile
    dd = D.DeviceDrafter(s, w)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(batch)
    reps = torch.empty((batch, gamma + 1, gamma, s.hidden), dtype=torch.float32, device="cuda").normal_(generator=gen)
    Ed = torch.from_numpy(E).cuda()
    flat = reps.view(batch, (gamma + 1) * gamma, s.hidden)
    for b in range(batch):
        for i, v in enumerate((650, 651, 130)):  # their logits lead
            flat[b, (5 * b + i) % 42] += 300 * Ed[v]
        flat[b, (5 * b + 7) % 42] = 0  # every logit 0
        flat[b, (5 * b + 9) % 42, 3] = float("inf")
        flat[b, (5 * b + 11) % 42, 5] = float("-inf")
        flat[b, (5 * b + 13) % 42, 7] = float("nan")
        flat[b, (5 * b + 15) % 42] = 3e38  # products that overflow
    ref_rows = []
    ws = D.Workspace(dd.cfg, batch, 64)

    def rows_of(x):
        cand = D.branch_candidates_buffer(dd, x.shape[0])
        D.branch_candidates(dd, x, cand, ws)
        torch.cuda.synchronize()
        return cand[4096:].view(torch.int64).view(x.shape[0], 42, -1).cpu()

    got = rows_of(reps)
    for b in range(batch):
        ref_rows.append(rows_of(reps[b:b + 1].contiguous())[0])
    ref = torch.stack(ref_rows)
    assert torch.equal(got, ref)
    col = 0xFFFFFFFF - (got[:, :, :17] & 0xFFFFFFFF)
    assert bool((col[:, :, :2] < V).all())
    for b in range(batch):  # the lowest of equal columns leads
        for i, lead in enumerate(((650, 700), (651, 701), (130, 131))):
            assert tuple(col[b, (5 * b + i) % 42, :2].tolist()) == lead


# 102, 170, 238 and 272 rows over more than 32768 columns (wide tiles), where four columns are one store and
# where they are not
@pytest.mark.parametrize("batch,vocab", [(6, 33000), (10, 33001), (14, 33000), (16, 33001)])
def test_target_over_a_wide_vocabulary(batch, vocab):
    from paper_2609_27396_amd import dpara as D
    from paper_2609_27396_amd.harness import upload_cache
    s = _shape(256, 256, vocab, 16)
    lens = [(29 * i) % 70 for i in range(batch)]
    _say("case target vocabulary", batch * 17, vocab)
    w = synth.make_target_weights(s, seed=7, gain_jitter=0.1)
    k, v = synth.make_target_cache(s, lens, seed=8)
    block = np.random.default_rng(batch).integers(0, vocab, (batch, 17)).astype(np.int32)
    t = D.DeviceTarget(s, w)
    ctx = D.DeviceContext(s, batch, 128)
    upload_cache(ctx, k, v, lens, torch.bfloat16)
    ws = D.Workspace(t.cfg, batch, 128, target=True)
    lf = torch.empty((batch, 17, vocab), dtype=torch.float32, device="cuda")
    lb = torch.empty_like(lf, dtype=torch.bfloat16)
    D.target_forward(t, ctx, torch.from_numpy(block).cuda(), lf, ws)
    D.target_forward(t, ctx, torch.from_numpy(block).cuda(), lb, ws)
    torch.cuda.synchronize()
    for b in (0, batch - 1):
        ref = O.target_forward(s, w, [k[0][b]], [v[0][b]], block[b], "bf16")
        assert np.abs(lf[b].cpu().numpy() - ref).max() <= TOL, b
    np.testing.assert_allclose(lb.float().cpu().numpy(), lf.cpu().numpy(), rtol=2 ** -8, atol=0)
