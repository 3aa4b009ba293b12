"""GPU parity of the training-side "single user, multiple items" forward (Sec. 3.2): histories and
candidates as one packed set of rows under the SUMI mask, no cache kept, against the oracle's packed
definition (the (L+M) x (L+M) mask written out) on the same seeded inputs; tolerance 2e-2 max-abs."""
import numpy as np
import pytest

import workloads as W
from harness import GpuStack, launches, max_abs, oracle, oracle_stack_config, say

pytestmark = pytest.mark.gpu


def run_forward(spec, users, want_hist=True, flags=0):
    import torch
    say(f"[case] forward {spec.name} layers={spec.n_layers} d={spec.d_model} B={spec.B} L={spec.L} sub={spec.sub_len} "
        f"causal={spec.causal} flags={flags} y_hist={want_hist}")
    w = W.make_stack(spec)
    g = GpuStack(w, flags=flags)
    P = g.P
    T = int(w["tok_off"][-1])
    # scratch cache: one layer is all the packed forward needs
    one = P.Config(n_layers=1, d_model=spec.d_model, n_heads=spec.H, d_head=spec.dh, d_ffn=spec.d_ffn,
                   n_scen=spec.n_scen, n_beh=spec.n_beh, sub_len=spec.sub_len, dtype=P.BF16, flags=g.cfg.flags,
                   qk_scale=spec.qk_scale, rms_eps=spec.rms_eps)
    buf = torch.empty(P.climber_kv_cache_bytes(one, g.padded), dtype=torch.uint8, device="cuda:0")
    scratch = P.climber_kv_cache_create(one, [int(x) for x in w["hist_len"]], g.padded, buf)
    ws = torch.empty(P.climber_workspace_bytes(g.cfg, T + g.m_total), dtype=torch.uint8, device="cuda:0")
    y_c = torch.full((max(g.m_total, 1), spec.d_model), float("nan"), dtype=torch.float32, device="cuda:0")
    y_h = torch.full((T, spec.d_model), float("nan"), dtype=torch.float32, device="cuda:0") if want_hist else None
    P.climber_sumi_forward(g.cfg, g.layers, g.tau, g.x_hist, g.scen, g.beh, g.x_cand, g.cand_off, g.m_total,
                           g.m_max, g.cscen, g.cbeh, scratch, y_h, y_c, ws)
    torch.cuda.synchronize()
    yc = y_c.cpu().numpy()
    yh = y_h.cpu().numpy() if want_hist else None
    cfg = oracle_stack_config(spec)
    ec = eh = 0.0
    sq, cnt = 0.0, 0
    for b in users:
        t0, Lb = int(w["tok_off"][b]), int(w["hist_len"][b])
        c0, c1 = int(w["cand_off"][b]), int(w["cand_off"][b + 1])
        rh, rc = oracle.stack_packed(cfg, w["layers"], w["tau"], w["x_hist"][t0:t0 + Lb], w["scen"][t0:t0 + Lb],
                                     w["beh"][t0:t0 + Lb], w["x_cand"][c0:c1], w["cscen"][c0:c1], w["cbeh"][c0:c1])
        ec = max(ec, max_abs(yc[c0:c1], rc))
        sq, cnt = sq + float((rh ** 2).sum() + (rc ** 2).sum()), cnt + rh.size + rc.size
        if want_hist and Lb:
            eh = max(eh, max_abs(yh[t0:t0 + Lb], rh))
    # the bar is 2e-2 for outputs at unit scale; a stack whose hidden states are larger is held to the
    # same relative figure
    rms = (sq / max(cnt, 1)) ** 0.5
    tol = 2e-2 * max(1.0, rms)
    say(f"  packed forward: y_cand max-abs {ec:.3e}" + (f", y_hist max-abs {eh:.3e}" if want_hist else "") +
        f" (|y| rms {rms:.3f}, tol {tol:.2e})")
    assert np.isfinite(yc[:g.m_total]).all() and ec < tol and eh < tol
    return w, g, yc


def test_packed_forward_small_ragged_both_masks():
    spec = W.StackSpec("fwd-ragged", B=4, L=384, sub_len=128, M=0, n_layers=3, d_model=128, H=2, dh=64, d_ffn=256,
                       n_scen=8, n_beh=4, seed=91, hist_lens=(384, 77, 300, 129), cand_counts=(37, 5, 0, 130),
                       nan_padding=True)
    run_forward(spec, users=(0, 1, 2, 3))
    run_forward(spec, users=(0, 1, 3), want_hist=False)
    # keys / values through rows (one projection launch over both kinds of rows) instead of straight
    # into the scratch cache
    run_forward(spec, users=(0, 1, 2, 3), flags=4)
    run_forward(spec, users=(0, 1, 3), want_hist=False, flags=4)
    spec = W.StackSpec("fwd-causal", B=2, L=256, sub_len=128, M=50, n_layers=3, d_model=128, H=2, dh=64, d_ffn=256,
                       n_scen=8, n_beh=4, seed=92, hist_lens=(256, 200), causal=True, w_std=0.04)
    run_forward(spec, users=(0, 1))
    run_forward(spec, users=(0, 1), flags=2)
    run_forward(spec, users=(0, 1), flags=4)


def test_packed_forward_equals_encode_then_score_within_rounding():
    spec = W.StackSpec("fwd-vs-serving", B=3, L=256, sub_len=128, M=70, n_layers=2, d_model=128, H=2, dh=64,
                       d_ffn=256, n_scen=8, n_beh=4, seed=93, hist_lens=(256, 130, 203))
    w, g, yc = run_forward(spec, users=(0, 1, 2), want_hist=False)
    g.encode()
    ys = g.score()
    e = max_abs(yc[:g.m_total], ys)
    say(f"  packed forward vs encode + score: max-abs {e:.3e}")
    assert e < 2e-2
    # with the keys / values going straight into the cache on both sides the two are the same kernels
    # on the same rows: equal bits
    if not (g.cfg.flags & 4):
        assert np.array_equal(yc[:g.m_total], ys)


def test_packed_forward_config4_full_size_sampled_users():
    # full size (B=32, L=1024, M=256, 4 layers): 41k rows per projection launch; four users against
    # the oracle's packed definition (one user's 1280 x 1280 mask per layer and head)
    run_forward(W.CONFIG4, users=(0, 9, 22, 31), want_hist=False)


def test_randomized_stack_shapes_and_routes():
    # seeded sweep over small stacks: 1..3 layers, d_model 128 / 256, ragged histories (down to none)
    # padded to 64 or 128, candidate counts across the query-tile and GEMM-tile sizes (down to none),
    # both masks, every route (flags 0, 2, 4, 6), NaN padding; encode + score or the packed forward
    from test_gpu_stack import run
    rng = np.random.Generator(np.random.Philox(25020988))
    for i in range(40):
        B = int(rng.integers(1, 5))
        d = int(rng.choice([128, 256]))
        hist = tuple(int(x) for x in rng.integers(0, 420, size=B))
        if max(hist) == 0:
            hist = (50,) + hist[1:]
        cands = tuple(int(x) for x in rng.choice([0, 1, 5, 37, 128, 129, 200, 260], size=B))
        if sum(cands) == 0:
            cands = (9,) + cands[1:]
        spec = W.StackSpec(f"stack-sweep-{i}", B=B, L=0, sub_len=int(rng.choice([0, 128, 256])), M=0,
                           n_layers=int(rng.integers(1, 4)), d_model=d, H=d // 64, dh=64, d_ffn=int(rng.choice([256, 512])),
                           n_scen=int(rng.integers(1, 9)), n_beh=int(rng.integers(1, 5)), seed=9000 + i,
                           pad_to=int(rng.choice([64, 128])), hist_lens=hist, cand_counts=cands,
                           nan_padding=bool(rng.integers(0, 2)), causal=bool(rng.integers(0, 2)))
        users = tuple(b for b in range(B) if cands[b] > 0)
        flags = int(rng.choice([0, 2, 4, 6]))
        if rng.integers(0, 2):
            run(spec, users=users, flags=flags)
        else:
            run_forward(spec, users=users, want_hist=bool(rng.integers(0, 2)), flags=flags)


@pytest.mark.parametrize("d, F, m", [(512, 256, 5), (512, 256, 4200), (512, 256, 8300), (512, 128, 12400), (256, 256, 4200),
                                     (384, 256, 3500), (384, 256, 11000), (384, 256, 43600)])
def test_residual_joins_the_finished_sum(d, F, m):
    # every route of the two residual projections: a wave per block, the one-launch tail with its four kernels, and the 64 x 128, 128 x 128 and 256 x 128 tiles.  Residual rows of 4096 (ulp 2^-11) and products of which 16, what one
    # matrix instruction adds, make a quarter of that ulp: summed onto the residual each would be lost, summed first
    # they are d 2^-17 and d_ffn 2^-17, whole ulps, and every sum on the way is exact in fp32.
    import torch
    import paper_2502_09888_amd as P
    say(f"[case] residual d={d} F={F} m={m}")
    dev, bf = "cuda:0", torch.bfloat16
    cfg = P.Config(n_layers=1, d_model=d, n_heads=d // 64, d_head=64, d_ffn=F, dtype=P.BF16)
    w = {k: torch.zeros(*s, dtype=bf, device=dev) for k, s in
         (("g1", (d,)), ("wqkv", (d, 3 * d)), ("wo", (d, d)), ("g2", (d,)), ("w1", (d, F)), ("w2", (F, d)))}
    w["g1"].fill_(1), w["g2"].fill_(1)
    w["wqkv"][0, 2 * d:] = 1          # values: 1 (no history: a candidate's output is its own value)
    w["wo"].fill_(2.0 ** -17)
    w["w1"][0] = 16                   # hidden: GELU(16) = 16
    w["w2"].fill_(2.0 ** -21)
    buf = torch.empty(P.climber_kv_cache_bytes(cfg, [64]), dtype=torch.uint8, device=dev)
    cache = P.climber_kv_cache_create(cfg, [0], [64], buf)
    x = torch.full((m, d), 4096.0, device=dev)
    y = torch.full((m, d), float("nan"), device=dev)
    ids, off = torch.zeros(m, dtype=torch.int32, device=dev), torch.tensor([0, m], dtype=torch.int32, device=dev)
    ws = torch.empty(P.climber_workspace_bytes(cfg, m), dtype=torch.uint8, device=dev)
    P.climber_layer_forward(cfg, w, torch.ones(1, 1, device=dev), 0, P.MODE_CANDIDATE, cache, x, y, ids, ids, off, m, m, ws)
    torch.cuda.synchronize()
    assert bool((y == 4096.0 + (d + F) * 2.0 ** -17).all())


@pytest.mark.parametrize("d, F, m", [(512, 512, 5), (512, 512, 4200), (512, 512, 8300), (512, 384, 12400), (256, 256, 4200),
                                     (384, 384, 4000), (384, 384, 11000), (384, 384, 44000)])
def test_gelu_keeps_its_relative_error_in_the_tail(d, F, m):
    # every route of the up-projection (as above): hidden unit j gets the pre-activation z_j in every row and w2 hands it
    # out as column j, 2^24 times.  Against formula 7.1.26 of Abramowitz & Stegun in double precision: the bf16 rounding
    # of the hidden (eight bits: 2^-8) and 1e-5 for its evaluation in fp32 (the exponent of up to 26 to half an ulp: 1e-6 of the
    # value; a reciprocal, an exponential and ten more operations: 1.5e-6), the rounding of 1 + 2^24 u (2^-24 / 0.1).
    import torch
    import paper_2502_09888_amd as P
    say(f"[case] gelu d={d} F={F} m={m}")
    dev, bf = "cuda:0", torch.bfloat16
    cfg = P.Config(n_layers=1, d_model=d, n_heads=d // 64, d_head=64, d_ffn=F, dtype=P.BF16, rms_eps=1e-12)
    z = torch.linspace(-6, 2, F, dtype=torch.float64).to(bf)
    w = {k: torch.zeros(*s, dtype=bf, device=dev) for k, s in
         (("g1", (d,)), ("wqkv", (d, 3 * d)), ("wo", (d, d)), ("g2", (d,)), ("w1", (d, F)), ("w2", (F, d)))}
    w["g1"].fill_(1), w["g2"].fill_(1)
    w["w1"][0] = z.to(dev)
    w["w2"].fill_diagonal_(2.0 ** 24)
    buf = torch.empty(P.climber_kv_cache_bytes(cfg, [64]), dtype=torch.uint8, device=dev)
    cache = P.climber_kv_cache_create(cfg, [0], [64], buf)
    x, y = torch.ones(m, d, device=dev), torch.full((m, d), float("nan"), device=dev)
    ids, off = torch.zeros(m, dtype=torch.int32, device=dev), torch.tensor([0, m], dtype=torch.int32, device=dev)
    ws = torch.empty(P.climber_workspace_bytes(cfg, m), dtype=torch.uint8, device=dev)
    P.climber_layer_forward(cfg, w, torch.ones(1, 1, device=dev), 0, P.MODE_CANDIDATE, cache, x, y, ids, ids, off, m, m, ws)
    torch.cuda.synchronize()
    assert torch.equal(y, y[:1].expand_as(y))
    a, zz = z.double().abs().numpy(), z.double().numpy()
    t = 1 / (1 + 0.3275911 * a / np.sqrt(2))
    poly = t * (0.254829592 + t * (-0.284496736 + t * (1.421413741 + t * (-1.453152027 + t * 1.061405429))))
    want = np.maximum(zz, 0) - a * 0.5 * poly * np.exp(-a * a / 2)
    got = (y[0, :F].double().cpu().numpy() - 1) / 2.0 ** 24
    err = np.abs(got - want) / np.abs(want).clip(1e-12)
    say(f"largest relative error {err.max():.2e} at z = {zz[err.argmax()]:.3f}")
    assert err.max() < 2.0 ** -8 + 1e-5


@pytest.mark.parametrize("d, F, m", [(256, 256, 4200), (512, 256, 4200), (512, 256, 8300), (512, 128, 12400)])
def test_layer_output_over_its_own_input(d, F, m):
    # x_out apart from x_in, the same rows, and rows shifted by less than their number in either direction: the same bits
    import torch
    import paper_2502_09888_amd as P
    say(f"[case] in and out d={d} F={F} m={m}")
    dev, bf = "cuda:0", torch.bfloat16
    gen = torch.Generator(device=dev)
    gen.manual_seed(m)
    cfg = P.Config(n_layers=1, d_model=d, n_heads=d // 64, d_head=64, d_ffn=F, dtype=P.BF16)
    w = {k: (torch.randn(*s, generator=gen, device=dev) * 0.05).to(bf) for k, s in
         (("g1", (d,)), ("wqkv", (d, 3 * d)), ("wo", (d, d)), ("g2", (d,)), ("w1", (d, F)), ("w2", (F, d)))}
    buf = torch.empty(P.climber_kv_cache_bytes(cfg, [64]), dtype=torch.uint8, device=dev)
    cache = P.climber_kv_cache_create(cfg, [0], [64], buf)
    ids, off = torch.zeros(m, dtype=torch.int32, device=dev), torch.tensor([0, m], dtype=torch.int32, device=dev)
    ws = torch.empty(P.climber_workspace_bytes(cfg, m), dtype=torch.uint8, device=dev)
    x = torch.randn(m, d, generator=gen, device=dev)
    outs = []
    for at_in, at_out in ((0, 2 * m), (0, 0), (0, 100), (100, 0), (0, m)):
        rows = torch.zeros(3 * m, d, device=dev)
        rows[at_in:at_in + m] = x
        P.climber_layer_forward(cfg, w, torch.ones(1, 1, device=dev), 0, P.MODE_CANDIDATE, cache, rows[at_in:], rows[at_out:], ids,
                                ids, off, m, m, ws)
        outs.append(rows[at_out:at_out + m].clone())
    torch.cuda.synchronize()
    assert all(torch.equal(o, outs[0]) for o in outs[1:])


@pytest.mark.parametrize("users, m", [(10, 1), (10, 33), (10, 95), (30, 1), (30, 95), (115, 33), (115, 127)])
def test_projection_kernels_for_few_and_many_rows_give_the_same_bits(users, m):
    # the packed forward runs users x 384 history rows and the candidates through one launch, at a width without a
    # one-launch tail: 3840 rows 64 x 128 tiles, 11520 rows 128 x 128, 44160 rows 256 x 128, up-projection (tiled store)
    # and both residual ones; the scoring call runs the candidates alone (16 rows x 64 columns a workgroup): a row's bits do
    # not depend on which; candidate counts at the edges of 32 rows, one of them the smallest launch there is
    spec = W.StackSpec(f"fwd-tiles-{users}-{m}", B=users, L=384, sub_len=128, M=0, n_layers=2, d_model=384, H=6, dh=64, d_ffn=768,
                       n_scen=8, n_beh=4, seed=95 + m, hist_lens=(384,) * users, cand_counts=(m,) + (0,) * (users - 1))
    w, g, yc = run_forward(spec, users=(0,), want_hist=True)
    g.encode()
    assert np.array_equal(yc[:g.m_total], g.score())


@pytest.mark.parametrize("d_model, d_ffn, users, m", [(512, 128, 33, 33), (512, 384, 33, 95), (512, 256, 22, 63),
                                                         (512, 512, 22, 2), (512, 256, 11, 31), (512, 768, 19, 1), (256, 128, 11, 1),
                                                         (256, 256, 11, 64)])
def test_layer_tail_in_one_launch_gives_the_bits_of_three(d_model, d_ffn, users, m):
    # users x 384 history rows and the candidates in one launch: more rows than the single-launch tail asks for, the
    # candidates alone fewer.  One, two and three chunks of the hidden; tiles of 64 and 32 rows, the last one with 1
    # to all of them.
    spec = W.StackSpec(f"fwd-tail-{d_model}-{d_ffn}", B=users, L=384, sub_len=128, M=0, n_layers=2, d_model=d_model,
                       H=d_model // 64, dh=64, d_ffn=d_ffn, n_scen=8, n_beh=4, seed=140 + m, hist_lens=(384,) * users,
                       cand_counts=(m,) + (0,) * (users - 1))
    w, g, yc = run_forward(spec, users=(0,), want_hist=True)
    g.encode()
    assert np.array_equal(yc[:g.m_total], g.score())


@pytest.mark.parametrize("d_ffn, users, m", [(256, 11, 1), (512, 11, 32), (2048, 12, 33), (256, 16, 2048), (1024, 16, 2047)])
def test_layer_tail_with_weights_requested_ahead_gives_the_bits_of_three(d_ffn, users, m):
    # 32-row tiles at d_model 512, from 4097 to 8192 rows: one to eight chunks of the hidden, the fewest and the most
    # workgroups that share out the requests; the candidates alone by separate launches
    spec = W.StackSpec(f"fwd-ahead-{d_ffn}-{m}", B=users, L=384, sub_len=128, M=0, n_layers=2, d_model=512, H=8, dh=64, d_ffn=d_ffn,
                       n_scen=8, n_beh=4, seed=240 + m, hist_lens=(384,) * users, cand_counts=(m,) + (0,) * (users - 1))
    w, g, yc = run_forward(spec, users=(1,), want_hist=True)
    g.encode()
    assert np.array_equal(yc[:g.m_total], g.score())


@pytest.mark.parametrize("d_ffn, m", [(1024, 2049), (2048, 2305), (1280, 4096)])
def test_down_projection_on_a_longer_ring_gives_the_bits_of_the_tail(d_ffn, m):
    # candidates alone by 64 x 128 tiles, whose ring is six k-tiles long where K is 1024 and more, the last row's tile nearly empty;
    # with the history's rows in the tail's one launch
    spec = W.StackSpec(f"fwd-ring-{d_ffn}", B=11, L=384, sub_len=128, M=0, n_layers=2, d_model=512, H=8, dh=64, d_ffn=d_ffn, n_scen=8, n_beh=4,
                       seed=440 + m, hist_lens=(384,) * 11, cand_counts=(m,) + (0,) * 10)
    w, g, yc = run_forward(spec, users=(1,), want_hist=True)
    g.encode()
    assert np.array_equal(yc[:g.m_total], g.score())
    import torch
    y = torch.empty(m, 512, device="cuda:0")
    run = launches(lambda: g.P.climber_sumi_score(g.cfg, g.layers, g.tau, g.cache, g.x_cand, g.cand_off, m, m, g.cscen, g.cbeh, y, g.ws))
    assert any("gemm_bf16_kernelILi2ELi1ELi2ELi6E" in k.kernel for k in run)


@pytest.mark.parametrize("d_model, d_ffn, m, rows", [
    (384, 128, 1, 1), (384, 384, 15, 1), (384, 640, 17, 1), (512, 768, 31, 1), (512, 1536, 33, 1), (512, 2048, 16, 1), (512, 512, 129, 1),
    (512, 2048, 512, 1), (512, 2048, 513, 2), (512, 1024, 2017, 2), (512, 1024, 2048, 2), (384, 896, 1313, 2), (768, 640, 353, 2), (768, 256, 385, 2)])
def test_few_rows_give_the_bits_of_the_macro_tiles(d_model, d_ffn, m, rows):
    # candidates alone in blocks of 16 (rows 1) or 32 (rows 2) rows, against the tiles that they share with 11520 rows of history; K a multiple of 128,
    # 256 or 512 only, one chunk of it and an odd number of chunks; the last block with 1 to all of its rows; both sides of the line between 16 and 32 rows
    # and the largest launch of the residual projections
    spec = W.StackSpec(f"fwd-few-{d_model}-{d_ffn}-{m}", B=30, L=384, sub_len=128, M=0, n_layers=2, d_model=d_model, H=d_model // 64, dh=64,
                       d_ffn=d_ffn, n_scen=8, n_beh=4, seed=540 + m, hist_lens=(384,) * 30, cand_counts=(m,) + (0,) * 29)
    w, g, yc = run_forward(spec, users=(1,), want_hist=True)
    g.encode()
    assert np.array_equal(yc[:g.m_total], g.score())
    import torch
    y = torch.empty(m, d_model, device="cuda:0")
    run = launches(lambda: g.P.climber_sumi_score(g.cfg, g.layers, g.tau, g.cache, g.x_cand, g.cand_off, m, m, g.cscen, g.cbeh, y, g.ws))
    assert any(f"gemm_small_kernelILi2ELi{rows}E" in k.kernel for k in run)


@pytest.mark.parametrize("d_model, layers, lens, cands, sums", [(512, 1, (64,), (1,), True), (256, 2, (1, 64), (15, 2), True), (512, 3, (130, 60), (129, 31), True),
                                                                (256, 2, (560, 0, 40), (672, 0, 0), True), (512, 2, (1024,), (1024,), True),
                                                                (512, 2, (1025,), (1025,), False), (256, 2, (1984, 1), (2048, 0), True),
                                                                (384, 2, (100,), (33,), False)])
def test_first_projection_of_few_rows_makes_their_sums_and_copies(d_model, layers, lens, cands, sums):
    # few rows of 256 or 512 columns: the first layer's projection forms the sums of squares and the fp32 residual rows itself, in
    # blocks of 16 or 32 rows for candidates, of 32 into the cache; against the packed forward and the encode by way of rows, which have a launch
    # for them: one row to the most there are, and one block more; NaN in the padding
    spec = W.StackSpec(f"fwd-sums-{d_model}-{sum(cands)}", B=len(lens), L=0, sub_len=128, M=0, n_layers=layers, d_model=d_model, H=d_model // 64, dh=64,
                       d_ffn=512, n_scen=8, n_beh=4, seed=640 + sum(cands), pad_to=64, hist_lens=lens, cand_counts=cands, nan_padding=True)
    w, g, yc = run_forward(spec, users=(0,), want_hist=True)
    other = GpuStack(w, flags=4)
    other.encode()
    assert np.array_equal(yc[:g.m_total], other.score())
    g.encode()
    assert np.array_equal(yc[:g.m_total], g.score())
    import torch
    y = torch.empty(g.m_total, d_model, device="cuda:0")
    for call in (g.encode, lambda: g.P.climber_sumi_score(g.cfg, g.layers, g.tau, g.cache, g.x_cand, g.cand_off, g.m_total, g.m_max, g.cscen, g.cbeh, y, g.ws)):
        assert any("row_prep_kernel" in k.kernel for k in launches(call)) != sums


@pytest.mark.parametrize("d_ffn, m, head", [(128, 1, True), (384, 31, True), (1024, 33, True), (1024, 1024, True), (1024, 1025, False),
                                            (2048, 500, True), (256, 4096, True)])
def test_projection_and_hidden_in_one_launch_give_the_bits_of_two(d_ffn, m, head):
    # d_model 256: candidates alone in at most a workgroup per CU of 32 rows x 128 columns of the hidden, against all rows in the
    # tail's one launch; one to 16 parts of the hidden, the last rows' block in part, the most workgroups and one block more
    spec = W.StackSpec(f"fwd-head-{d_ffn}-{m}", B=11, L=384, sub_len=128, M=0, n_layers=2, d_model=256, H=4, dh=64, d_ffn=d_ffn, n_scen=8,
                       n_beh=4, seed=340 + m, hist_lens=(384,) * 11, cand_counts=(m,) + (0,) * 10)
    w, g, yc = run_forward(spec, users=(1,), want_hist=True)
    g.encode()
    assert np.array_equal(yc[:g.m_total], g.score())
    import torch
    y = torch.empty(m, 256, device="cuda:0")
    run = launches(lambda: g.P.climber_sumi_score(g.cfg, g.layers, g.tau, g.cache, g.x_cand, g.cand_off, m, m, g.cscen, g.cbeh, y, g.ws))
    assert any("layer_head_kernel" in k.kernel for k in run) == head


@pytest.mark.parametrize("d, F, layers", [(128, 128, 1), (256, 384, 5), (384, 128, 4), (512, 2048, 2)])
def test_packed_weights_are_the_operand_fragments(d, F, layers):
    # 16 bytes (column block nb, k step ks, lane): rows 16 ks + 8 (lane / 32) + 0..7 of column 32 nb + lane % 32, the gains of the
    # two projections behind a norm multiplied in and rounded once; the five-layer stack takes two launches
    import torch
    import paper_2502_09888_amd as P
    say(f"[case] packed weights d={d} F={F} layers={layers}")
    dev, bf = "cuda:0", torch.bfloat16
    gen = torch.Generator(device=dev)
    gen.manual_seed(d + F)
    cfg = P.Config(n_layers=layers, d_model=d, n_heads=d // 64, d_head=64, d_ffn=F, dtype=P.BF16)
    ws = [{k: torch.randn(*s, generator=gen, device=dev).to(bf) for k, s in
           (("g1", (d,)), ("wqkv", (d, 3 * d)), ("wo", (d, d)), ("g2", (d,)), ("w1", (d, F)), ("w2", (F, d)))} for _ in range(layers)]
    packed = torch.full((P.climber_packed_weights_bytes(cfg) // 2,), float("nan"), dtype=bf, device=dev)
    P.climber_pack_weights(cfg, ws, packed)
    torch.cuda.synchronize()
    got = packed.view(layers, -1)
    for l, w in enumerate(ws):
        at = 0
        for k, gain in (("wqkv", "g1"), ("wo", None), ("w1", "g2"), ("w2", None)):
            x = w[k].float() * w[gain].float()[:, None] if gain else w[k].float()
            K, N = x.shape
            want = x.to(bf).view(K // 16, 2, 8, N // 32, 32).permute(3, 0, 1, 4, 2).reshape(-1)
            assert torch.equal(got[l, at:at + K * N], want), (l, k)
            at += K * N


@pytest.mark.parametrize("layers, flags", [(1, 0), (3, 0), (1, 4), (2, 4)])
def test_packed_forward_candidates_with_and_without_history_outputs(layers, flags):
    # the first layer's inputs where they are (flags 0) or copied behind one another (CLIMBER_QKV_VIA_ROWS); the candidates'
    # rows written by the last layer, or copied out behind the history's: the same bits
    spec = W.StackSpec(f"fwd-outputs-{layers}-{flags}", B=2, L=0, sub_len=128, M=0, n_layers=layers, d_model=256, H=4, dh=64, d_ffn=256,
                       n_scen=8, n_beh=4, seed=300 + layers, pad_to=64, hist_lens=(130, 63), cand_counts=(33, 7), nan_padding=True)
    a = run_forward(spec, users=(0, 1), want_hist=False, flags=flags)[2]
    b = run_forward(spec, users=(0, 1), want_hist=True, flags=flags)[2]
    assert np.array_equal(a[:40], b[:40])


@pytest.mark.parametrize("d, F, layers, lens, cands, flags", [
    (512, 256, 3, (384, 77, 300, 129, 512, 64, 1) * 6, 8200, 0),     # histories and candidates, each more than 8192 rows
    (512, 256, 1, (384, 130) * 17, 4133, 0), (256, 128, 1, (384,) * 11, 4097, 0),  # one layer: the inputs are its residual
    (512, 768, 2, (448,) * 19, 127, 0),                              # a uniform batch, few candidates
    (512, 256, 3, (512, 500, 449) * 21, 65, 0),                      # encode: two turns of tiles, every tail of it with a projection
    (512, 384, 3, (500, 33) * 15, 33, 0),                            # no kernel with a projection at this d_ffn: launches of their own
    (256, 128, 3, (200, 31, 0, 96, 130) * 9, 4161, 0), (256, 384, 2, (320,) * 14, 1, 1), (256, 256, 3, (320, 65) * 12, 31, 4)])
def test_projection_behind_the_tail_gives_the_bits_of_separate_launches(d, F, layers, lens, cands, flags):
    # a batch large enough for the tail that makes the next layer's projection (and for the projection of resident rows) against
    # single users, which take the launches for few rows: caches of all layers, scores, packed forward with and without
    # history outputs.  Lengths at and off the edges of blocks, NaN in the padding rows
    import torch
    import paper_2502_09888_amd as P
    say(f"[case] chain d={d} F={F} users={len(lens)} cands={cands} flags={flags}")
    dev, bf, H = "cuda:0", torch.bfloat16, d // 64
    gen = torch.Generator(device=dev)
    gen.manual_seed(d + F + cands)
    cfg = P.Config(n_layers=layers, d_model=d, n_heads=H, d_head=64, d_ffn=F, n_scen=2, n_beh=2, sub_len=128, flags=flags, dtype=P.BF16,
                   qk_scale=0.02)  # (every row stays in one form of the softmax)
    w = [{k: (torch.randn(*s, generator=gen, device=dev) * 0.05 + (k[0] == "g")).to(bf) for k, s in
          (("g1", (d,)), ("wqkv", (d, 3 * d)), ("wo", (d, d)), ("g2", (d,)), ("w1", (d, F)), ("w2", (F, d)))} for _ in range(layers)]
    tau = torch.rand(layers, 2, 2, generator=gen, device=dev) + 0.5
    pads = [max(64, (n + 63) // 64 * 64) for n in lens]
    t0 = [sum(pads[:i]) for i in range(len(lens) + 1)]
    counts = [cands // len(lens) + (i < cands % len(lens)) for i in range(len(lens))]
    c0 = [sum(counts[:i]) for i in range(len(lens) + 1)]
    x = torch.randn(t0[-1], d, generator=gen, device=dev).to(bf)
    for i, n in enumerate(lens):
        x[t0[i] + n:t0[i + 1]] = float("nan")
    xc = torch.randn(cands, d, generator=gen, device=dev).to(bf)
    ids = torch.randint(0, 2, (2, t0[-1]), generator=gen, device=dev, dtype=torch.int32)
    cids = torch.randint(0, 2, (2, cands), generator=gen, device=dev, dtype=torch.int32)

    def run(users):
        hist, pad, m = [lens[i] for i in users], [pads[i] for i in users], [counts[i] for i in users]
        rows, a, b = sum(pad), t0[users[0]], c0[users[0]]
        buf = torch.full((P.climber_kv_cache_bytes(cfg, pad),), 0x7f, dtype=torch.uint8, device=dev)
        cache = P.climber_kv_cache_create(cfg, hist, pad, buf)
        ws = torch.empty(P.climber_workspace_bytes(cfg, rows + sum(m)), dtype=torch.uint8, device=dev)
        s, be, cs, cb = (t[k:k + n].clone() for t, k, n in ((ids[0], a, rows), (ids[1], a, rows), (cids[0], b, sum(m)), (cids[1], b, sum(m))))
        xh, xq = x[a:a + rows].clone(), xc[b:b + sum(m)].clone()
        off = torch.tensor([0] + [sum(m[:i + 1]) for i in range(len(m))], dtype=torch.int32, device=dev)
        P.climber_history_encode(cfg, w, tau, xh, s, be, cache, ws)
        ys = [torch.zeros(sum(m), d, device=dev) for _ in range(3)]
        yh = torch.zeros(rows, d, device=dev)
        P.climber_sumi_score(cfg, w, tau, cache, xq, off, sum(m), max(m), cs, cb, ys[0], ws)
        kv = buf[-layers * rows * d * 4:].view(layers, rows, d * 4).clone()
        for y, h in ((ys[1], None), (ys[2], yh)):
            P.climber_sumi_forward(cfg, w, tau, xh, s, be, xq, off, sum(m), max(m), cs, cb, cache, h, y, ws)
        torch.cuda.synchronize()
        return kv, ys, yh

    kv, ys, yh = run(list(range(len(lens))))
    assert torch.equal(ys[0], ys[1]) and torch.equal(ys[0], ys[2]) and not ys[0].isnan().any()
    for i in (0, 1, len(lens) - 1):
        kv1, ys1, yh1 = run([i])
        assert torch.equal(kv1, kv[:, t0[i]:t0[i + 1]]) and torch.equal(ys1[0], ys[0][c0[i]:c0[i + 1]])
        assert torch.equal(yh1[:lens[i]], yh[t0[i]:t0[i] + lens[i]])


@pytest.mark.parametrize("F, layers, lens, cands, flags", [
    (256, 3, (384, 77, 300, 129, 512, 64, 1) * 3, 1, 0),      # just above 4096 rows with the history, ragged
    (512, 2, (448,) * 18, 65, 0),                             # a uniform batch, 8129 rows: encode with 8064
    (256, 4, (200, 31, 0, 96, 130) * 3, 5377, 0),             # candidates alone from where their own launch begins a third turn, empty histories
    (2048, 2, (64, 1, 40), 7649, 0), (512, 2, (64, 0), 8128, 0), (256, 2, (320, 65) * 10, 31, 4)])
def test_projection_behind_tails_of_32_rows_gives_the_bits_of_separate_launches(F, layers, lens, cands, flags):
    # as above from 4097 to 8192 rows, where a ninth wave requests this projection's weights as well
    test_projection_behind_the_tail_gives_the_bits_of_separate_launches(512, F, layers, lens, cands, flags)


@pytest.mark.parametrize("users, cands, encode, forward, score", [(5, 4, 3, 3, 0), (7, 600, 3, 3, 0), (8, 0, 3, 3, 0), (8, 672, 3, 3, 0), (8, 673, 3, 3, 3),
                                                                 (8, 960, 3, 3, 3), (8, 961, 3, 3, 3), (8, 1024, 3, 3, 3), (8, 1025, 3, 0, 0)])
def test_tails_of_32_rows_make_the_next_projection_where_that_was_measured_to_be_faster(users, cands, encode, forward, score):
    # four layers, d_model 512: how many tails of an encode, a packed forward and a scoring call do
    import torch
    import paper_2502_09888_amd as P
    cfg, dev = P.Config(n_layers=4, n_heads=8, d_ffn=256, n_scen=1, n_beh=1, sub_len=256), "cuda:0"
    lens, rows, m = [1024] * users, 1024 * users, cands * users
    w = [{k: torch.zeros(s, dtype=torch.bfloat16, device=dev) for k, s in
          (("g1", 512), ("wqkv", (512, 1536)), ("wo", (512, 512)), ("g2", 512), ("w1", (512, 256)), ("w2", (256, 512)))} for _ in range(4)]
    buf = torch.empty(P.climber_kv_cache_bytes(cfg, lens), dtype=torch.uint8, device=dev)
    cache = P.climber_kv_cache_create(cfg, lens, lens, buf)
    ws = torch.empty(P.climber_workspace_bytes(cfg, rows + m), dtype=torch.uint8, device=dev)
    x, xc, y = (torch.zeros(n, 512, dtype=t, device=dev) for n, t in ((rows, torch.bfloat16), (max(m, 1), torch.bfloat16), (max(m, 1), torch.float32)))
    (ids, cids), tau = (torch.zeros(n, dtype=torch.int32, device=dev) for n in (rows, max(m, 1))), torch.ones(4, 1, 1, device=dev)
    off = torch.arange(users + 1, dtype=torch.int32, device=dev) * cands

    def tails(call):
        names = [k.kernel for k in launches(call)]
        say(names)
        return sum("layer_tail_kernelILi512E" in n and ("ELi8ELi8ELi1ELb1E" in n or "ELi8ELi8ELi0ELb1E" in n) for n in names)

    assert tails(lambda: P.climber_history_encode(cfg, w, tau, x, ids, ids, cache, ws)) == encode
    assert tails(lambda: P.climber_sumi_forward(cfg, w, tau, x, ids, ids, xc, off, m, cands, cids, cids, cache, None, y, ws)) == forward
    if m:
        assert tails(lambda: P.climber_sumi_score(cfg, w, tau, cache, xc, off, m, cands, cids, cids, y, ws)) == score


@pytest.mark.parametrize("d, m", [(512, 4225), (256, 4225), (512, 200)])
def test_one_layer_scores_written_over_its_inputs(d, m):
    # outputs that begin inside the candidates' rows, before them, and apart from them: the same bits
    import torch
    import paper_2502_09888_amd as P
    say(f"[case] outputs over inputs d={d} m={m}")
    dev, bf = "cuda:0", torch.bfloat16
    gen = torch.Generator(device=dev)
    gen.manual_seed(d + m)
    cfg = P.Config(n_layers=1, d_model=d, n_heads=d // 64, d_head=64, d_ffn=256, dtype=P.BF16, qk_scale=0.02)
    w = [{k: (torch.randn(*s, generator=gen, device=dev) * 0.05).to(bf) for k, s in
          (("g1", (d,)), ("wqkv", (d, 3 * d)), ("wo", (d, d)), ("g2", (d,)), ("w1", (d, 256)), ("w2", (256, d)))}]
    buf = torch.empty(P.climber_kv_cache_bytes(cfg, [64]), dtype=torch.uint8, device=dev)
    cache = P.climber_kv_cache_create(cfg, [0], [64], buf)
    ids, off = torch.zeros(m, dtype=torch.int32, device=dev), torch.tensor([0, m], dtype=torch.int32, device=dev)
    ws = torch.empty(P.climber_workspace_bytes(cfg, m), dtype=torch.uint8, device=dev)
    x = torch.randn(m, d, generator=gen, device=dev).to(bf)
    outs = []
    for at_y in (0, m // 2 * d, m * d, 3 * m * d):  # in bf16 values; the candidates' rows begin at m * d
        mem = torch.zeros(5 * m * d, dtype=bf, device=dev)
        mem[m * d:2 * m * d] = x.flatten()
        at_y = at_y // 64 * 64
        y = mem[at_y:at_y + 2 * m * d].view(torch.float32).view(m, d)
        P.climber_sumi_score(cfg, w, torch.ones(1, 1, 1, device=dev), cache, mem[m * d:2 * m * d], off, m, m, ids, ids, y, ws)
        outs.append(y.clone())
    torch.cuda.synchronize()
    assert all(torch.equal(o, outs[-1]) for o in outs) and outs[-1].abs().max() > 0


@pytest.mark.parametrize("users, cands, encode, forward", [(9, 8, 1, 3), (16, 0, 1, 1), (17, 8, 1, 0), (19, 8, 1, 3), (24, 0, 1, 1), (31, 0, 3, 3), (33, 8, 1, 3),
                                                           (40, 0, 1, 1), (44, 0, 3, 3)])
def test_tails_make_the_next_projection_where_that_was_measured_to_be_faster(users, cands, encode, forward):
    # four layers, d_model 512, 16 tiles a user: how many tails of an encode and of a packed forward (without candidates: the same) do.
    # Keys and values only (encode's last) always; whole layers by how full the last turn of 256 tiles is
    import torch
    import paper_2502_09888_amd as P
    cfg, dev = P.Config(n_layers=4, n_heads=8, d_ffn=256, n_scen=1, n_beh=1, sub_len=256), "cuda:0"
    lens, rows, m = [1024] * users, 1024 * users, cands * users
    w = [{k: torch.zeros(s, dtype=torch.bfloat16, device=dev) for k, s in
          (("g1", 512), ("wqkv", (512, 1536)), ("wo", (512, 512)), ("g2", 512), ("w1", (512, 256)), ("w2", (256, 512)))} for _ in range(4)]
    buf = torch.empty(P.climber_kv_cache_bytes(cfg, lens), dtype=torch.uint8, device=dev)
    cache = P.climber_kv_cache_create(cfg, lens, lens, buf)
    ws = torch.empty(P.climber_workspace_bytes(cfg, rows + m), dtype=torch.uint8, device=dev)
    x, xc, y = (torch.zeros(n, 512, dtype=t, device=dev) for n, t in ((rows, torch.bfloat16), (max(m, 1), torch.bfloat16), (max(m, 1), torch.float32)))
    (ids, cids), tau = (torch.zeros(n, dtype=torch.int32, device=dev) for n in (rows, max(m, 1))), torch.ones(4, 1, 1, device=dev)
    off = torch.arange(users + 1, dtype=torch.int32, device=dev) * cands

    def tails(call):
        names = [k.kernel for k in launches(call)]
        say(names)
        return sum("layer_tail_kernelILi512ELi2ELi8ELi8ELi0ELb1E" in n for n in names)

    assert tails(lambda: P.climber_history_encode(cfg, w, tau, x, ids, ids, cache, ws)) == encode
    assert tails(lambda: P.climber_sumi_forward(cfg, w, tau, x, ids, ids, xc, off, m, cands, cids, cids, cache, None, y, ws)) == forward
