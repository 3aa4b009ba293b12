"""GPU parity of the relative attention bias (Eq. (3): R = Q K^T + f_b, divided by the temperature):
the bias entry points of the C ABI against the oracle's *_bias functions on the same seeded inputs.
Bucket decisions are integer arithmetic on both sides, so they agree exactly; tolerances as for the
bias-free attention (1e-4 fp32, 2e-2 bf16)."""
import numpy as np
import pytest

import workloads as W
from harness import GpuAttention, launches, max_abs, oracle, say, valid_rows

pytestmark = pytest.mark.gpu
TOL = {"f32": 1e-4, "bf16": 2e-2}


class GpuBias(GpuAttention):
    def __init__(self, w, causal=False):
        super().__init__(w, causal=causal)
        t = self.torch
        dev = "cuda:0"
        for n in ("hist_pos", "hist_ts", "cand_pos", "cand_ts", "pos_table", "time_table"):
            setattr(self, n, t.from_numpy(w[n]).to(dev).contiguous())
        self.rb = self.P.rel_bias(self.pos_table, self.time_table, self.hist_pos, self.hist_ts, self.cand_pos,
                                  self.cand_ts)

    def history_bias(self):
        t = self.torch
        o = t.full((self.qh.shape[0], self.d), float("nan"), dtype=self.dt, device="cuda:0")
        self.P.climber_attn_history_bias(self.cfg, self.tau, self.qh, self.kh, self.vh, self.scen, self.beh,
                                         self.cache, 0, o, self.rb)
        t.cuda.synchronize()
        return o.float().cpu().numpy()

    def sumi_bias(self):
        m_total = int(self.w["cand_off"][-1])
        o = self.torch.full((max(m_total, 1), self.d), float("nan"), dtype=self.dt, device="cuda:0")
        self.launch_sumi_bias(o)
        self.torch.cuda.synchronize()
        return o[:m_total].float().cpu().numpy()

    def launch_sumi_bias(self, o):
        w = self.w
        m_total = int(w["cand_off"][-1])
        m_max = int(np.diff(w["cand_off"]).max()) if m_total else 0
        self.P.climber_attn_sumi_bias(self.cfg, self.tau, self.cache, 0, self.qc, self.kc, self.vc, self.cand_off,
                                      m_total, m_max, self.cscen, self.cbeh, o, self.rb)


def oracle_hist_bias(w, causal=False):
    s = w["spec"]
    return oracle.attn_history_bias(w["tok_off"], w["hist_len"], w["qh"], w["kh"], w["vh"], w["scen"], w["beh"],
                                    w["tau"], s.qk_scale, w["hist_pos"], w["hist_ts"], w["pos_table"],
                                    w["time_table"], sub_len=s.sub_len, causal=causal)


def oracle_sumi_bias(w):
    s = w["spec"]
    return oracle.attn_sumi_bias(w["tok_off"], w["hist_len"], w["cand_off"], w["kh"], w["vh"], w["qc"], w["kc"],
                                 w["vc"], w["cscen"], w["cbeh"], w["tau"], s.qk_scale, w["hist_pos"], w["hist_ts"],
                                 w["cand_pos"], w["cand_ts"], w["pos_table"], w["time_table"])


def check_bias(w, causal=False):
    spec = w["spec"]
    say(f"[case] bias {spec.name} dtype={spec.dtype} B={spec.B} L={spec.L} sub={spec.sub_len} M={spec.M} H={spec.H} "
        f"qk_scale={spec.qk_scale} causal={causal} n_pos={w['pos_table'].shape[3]} n_time={w['time_table'].shape[3]}")
    g = GpuBias(w, causal=causal)
    tol = TOL[spec.dtype]
    oh = g.history_bias()
    ok = valid_rows(w)
    e = max_abs(oh[ok], oracle_hist_bias(w, causal=causal)[ok])
    say(f"  history+bias max-abs {e:.3e}")
    assert np.isfinite(oh[ok]).all() and e < tol and np.all(oh[~ok] == 0)
    os_ = g.sumi_bias()
    ref = oracle_sumi_bias(w)
    e = max_abs(os_, ref)
    # the bias must matter in the case: without it the result is far from the reference
    plain = g.sumi()
    say(f"  sumi+bias max-abs {e:.3e} (bias-free kernel output differs from it by {max_abs(plain, ref):.2e})")
    assert np.isfinite(os_).all() and e < tol
    assert max_abs(plain, ref) > 5 * tol
    return g, os_


def test_fp32_bias_both_masks_ragged():
    spec = W.shrink(W.CONFIG1, name="f32-bias", B=3, L=90, L_min=10, M=11, M_min=1, sub_len=32, pad_to=8,
                    nan_padding=True, dh=48, H=3, seed=81)
    w = W.add_bias_inputs(W.make_attention(spec), n_pos=15, n_time=9)
    check_bias(w)
    check_bias(w, causal=True)
    check_bias(W.add_bias_inputs(W.make_attention(W.CONFIG1)))


def test_bf16_bias_multi_tile_ragged_both_masks():
    spec = W.shrink(W.CONFIG5, name="bf16-bias-ragged", B=4, L=700, L_min=1, sub_len=256, M=200, M_min=1, H=2,
                    seed=82)
    w = W.add_bias_inputs(W.make_attention(spec))
    check_bias(w)
    check_bias(w, causal=True)
    spec = W.shrink(W.CONFIG2, name="bf16-bias-onesub", B=2, L=333, L_min=77, sub_len=0, M=70, H=1,
                    nan_padding=True, seed=83)
    check_bias(W.add_bias_inputs(W.make_attention(spec), n_pos=5, n_time=3))


def test_bf16_bias_single_bucket_tables_and_edges():
    # n_pos = n_time = 1: one entry per (scenario, behaviour, head), i.e. a constant along every row,
    # which softmax ignores: the result equals the bias-free one; and timestamps at the int32 ends
    spec = W.shrink(W.CONFIG2, name="bf16-bias-const", B=2, L=256, sub_len=128, M=60, H=2, seed=84)
    w = W.add_bias_inputs(W.make_attention(spec), n_pos=1, n_time=1, table_std=3.0)
    w["hist_ts"][::7] = -2_000_000_000
    w["cand_ts"][::5] = 2_000_000_000
    g = GpuBias(w)
    g.history(want_output=False)
    ref = oracle_sumi_bias(w)
    e = max_abs(g.sumi_bias(), ref)
    say(f"[case] bias {spec.name}: sumi+bias max-abs {e:.3e}; vs bias-free oracle "
        f"{max_abs(ref, oracle.attn_sumi(w['tok_off'], w['hist_len'], w['cand_off'], w['kh'], w['vh'], w['qc'], w['kc'], w['vc'], w['cscen'], w['cbeh'], w['tau'], spec.qk_scale)):.1e}")
    assert e < 2e-2


def test_bias_buckets_at_the_ends_of_the_int32_range():
    # positions and time stamps at and near the ends of int32: differences that overflow 32-bit
    # subtraction, every one of the 32 possible log2 buckets of |ts_i - ts_j| has a table entry of its own
    ends = np.array([-2**31, -2**31 + 1, -2**30, -3, -1, 0, 1, 2, 2**30, 2**31 - 2, 2**31 - 1], dtype=np.int64)
    for dtype, tol_key in (("f32", "f32"), ("bf16", "bf16")):
        base = W.CONFIG1 if dtype == "f32" else W.CONFIG2
        spec = (W.shrink(base, name="f32-bias-ends", B=2, L=192, sub_len=64, M=33, seed=88) if dtype == "f32" else
                W.shrink(base, name="bf16-bias-ends", B=2, L=256, sub_len=128, M=70, H=2, seed=89))
        w = W.add_bias_inputs(W.make_attention(spec), n_pos=7, n_time=34, table_std=1.0)
        rng = np.random.default_rng(5)
        for n in ("hist_pos", "hist_ts", "cand_pos", "cand_ts"):
            pick = rng.random(w[n].shape) < 0.5
            w[n][pick] = rng.choice(ends, size=int(pick.sum())).astype(np.int32)
        check_bias(w)


def test_bf16_bias_large_logits_take_the_running_maximum_pass():
    spec = W.shrink(W.CONFIG2, name="bf16-bias-biglogits", B=2, L=256, sub_len=128, M=100, H=2, qk_scale=12.0,
                    seed=85)
    check_bias(W.add_bias_inputs(W.make_attention(spec), table_std=20.0))


def test_bf16_bias_zero_tables_reproduce_the_bias_free_result():
    # zero tables: the bias variant computes the bias-free attention (it keeps the query exact and
    # scales the logits in fp32 where the plain kernel folds the scale into the query, so the two agree
    # to rounding, not bit for bit); both against the bias-free oracle
    spec = W.shrink(W.CONFIG2, name="bf16-bias-zero", B=2, L=384, sub_len=128, M=100, H=2, seed=86)
    w = W.add_bias_inputs(W.make_attention(spec))
    w["pos_table"][:] = 0
    w["time_table"][:] = 0
    g = GpuBias(w)
    g.history(want_output=False)
    ref = oracle.attn_sumi(w["tok_off"], w["hist_len"], w["cand_off"], w["kh"], w["vh"], w["qc"], w["kc"], w["vc"],
                           w["cscen"], w["cbeh"], w["tau"], spec.qk_scale)
    with_zero, plain = g.sumi_bias(), g.sumi()
    say(f"[case] bias {spec.name}: zero tables vs bias-free kernel {max_abs(with_zero, plain):.3e}, vs bias-free oracle "
        f"{max_abs(with_zero, ref):.3e} (bias-free kernel: {max_abs(plain, ref):.3e})")
    assert max_abs(with_zero, ref) < 2e-2 and max_abs(with_zero, plain) < 2e-2


def test_bias_at_config2_and_config3_shapes():
    for spec in (W.CONFIG2, W.CONFIG3):
        w = W.add_bias_inputs(W.make_attention(spec))
        say(f"[case] bias {spec.name} full size")
        g = GpuBias(w)
        oh = g.history_bias()
        ok = valid_rows(w)
        e = max_abs(oh[ok], oracle_hist_bias(w)[ok])
        say(f"  history+bias max-abs {e:.3e}")
        assert e < 2e-2
        e = max_abs(g.sumi_bias(), oracle_sumi_bias(w))
        say(f"  sumi+bias max-abs over all users {e:.3e}")
        assert e < 2e-2


def test_randomized_shapes_scales_masks_with_bias():
    # seeded sweep: ragged histories and candidate counts, paddings of 64 / 128, any subsequence length the
    # API admits, 1..4 heads, logit scales from the unit-scale benchmark to far beyond, both masks,
    # table sizes from one bucket to more buckets than distances
    rng = np.random.Generator(np.random.Philox(2502098))
    done = 0
    for i in range(60):
        L = int(rng.integers(1, 1400))
        M = int(rng.choice([1, 2, 31, 33, 64, 127, 128, 129, 255, 256, 257, 300, 513]))
        spec = W.shrink(W.CONFIG2, name=f"bias-sweep-{i}", B=int(rng.integers(1, 6)), L=L, L_min=int(rng.integers(1, L + 1)),
                        sub_len=int(rng.choice([0, 128, 256, 384, 512])), M=M, M_min=int(rng.integers(1, M + 1)),
                        H=int(rng.integers(1, 5)), pad_to=int(rng.choice([64, 128])), nan_padding=bool(rng.integers(0, 2)),
                        n_scen=int(rng.integers(1, 9)), n_beh=int(rng.integers(1, 5)),
                        qk_scale=float(rng.choice([0.125, 0.125, 0.3, 0.7, 1.5, 6.0])), seed=7000 + i)
        w = W.add_bias_inputs(W.make_attention(spec), n_pos=int(rng.choice([1, 5, 33])), n_time=int(rng.choice([1, 7, 34])),
                              table_std=float(rng.choice([0.3, 1.0])))
        causal = bool(rng.integers(0, 2))
        g = GpuBias(w, causal=causal)
        oh = g.history_bias()
        ok = valid_rows(w)
        e1 = max_abs(oh[ok], oracle_hist_bias(w, causal=causal)[ok])
        e2 = max_abs(g.sumi_bias(), oracle_sumi_bias(w))
        say(f"[case] {spec.name} B={spec.B} L={spec.L} sub={spec.sub_len} M={spec.M} H={spec.H} qk_scale={spec.qk_scale} "
            f"causal={causal}: history+bias {e1:.3e}, sumi+bias {e2:.3e}")
        assert np.isfinite(oh[ok]).all() and np.all(oh[~ok] == 0) and e1 < 2e-2 and e2 < 2e-2
        done += 1
    assert done == 60


@pytest.mark.parametrize("n_pos,n_time,L,sub,causal,shuffled", [
    (33, 12, 2300, 0, False, False),     # more than 64 blocks of 32 keys: classified in two turns, the second one ragged
    (33, 12, 2300, 0, True, True),       # coordinates in no order: hardly any block has one bucket
    (201, 40, 300, 256, False, False),   # more time buckets than an int32 distance has octaves; table rows longer than a wave
    (1, 2, 97, 128, False, False),       # one position bucket, two of time: hardly any block is mixed
    (129, 20, 700, 128, True, False),
    (3, 31, 65, 0, False, True)])
def test_bf16_bias_uniform_and_mixed_blocks(n_pos, n_time, L, sub, causal, shuffled):
    spec = W.shrink(W.CONFIG2, name=f"bias-blocks-{n_pos}-{n_time}-{L}", B=2, L=L, L_min=L - 40, sub_len=sub, M=150, M_min=20, H=2,
                    nan_padding=True, seed=900 + n_pos + L)
    w = W.add_bias_inputs(W.make_attention(spec), n_pos=n_pos, n_time=n_time)
    if shuffled:
        rng = np.random.Generator(np.random.Philox(5))
        w["hist_pos"] = rng.permutation(w["hist_pos"]).astype(np.int32)
        w["hist_ts"] = rng.permutation(w["hist_ts"]).astype(np.int32)
    check_bias(w, causal=causal)


def test_bf16_bias_running_maximum_over_two_turns_of_blocks():
    spec = W.shrink(W.CONFIG2, name="bias-safe-long", B=1, L=2200, sub_len=0, M=140, H=2, qk_scale=12.0, seed=941)
    check_bias(W.add_bias_inputs(W.make_attention(spec)))


@pytest.mark.parametrize("half", [2 ** 22 - 1, 2 ** 22, 2 ** 23, 2 ** 24])
def test_bf16_bias_position_tables_of_any_length(half):
    # every query at the positive clip of a long table, whose last entry puts all weight on the history and whose first
    # would take it away: distances at and beyond what a block's class holds
    spec = W.shrink(W.CONFIG2, name=f"bias-long-table-{half}", B=1, L=97, sub_len=0, M=40, H=1, n_scen=1, n_beh=1, seed=960)
    w = W.add_bias_inputs(W.make_attention(spec), n_pos=3, n_time=12)
    w["pos_table"] = np.zeros((1, 1, 1, 2 * half + 1), np.float32)
    w["pos_table"][..., -1], w["pos_table"][..., 0] = 4.0, -4.0
    w["cand_pos"] = np.full_like(w["cand_pos"], 2 ** 30)
    check_bias(w)


@pytest.mark.parametrize("qk_scale", [0.125, 12.0])  # (12: the running-maximum pass)
@pytest.mark.parametrize("L,sub,causal", [(97, 0, False), (161, 128, True), (300, 256, True)])
@pytest.mark.parametrize("n_pos", [3, 65])           # (3: blocks of later keys fall into one bucket; 65: they do not)
def test_bf16_bias_entries_of_unseen_keys_do_not_matter(L, sub, causal, qk_scale, n_pos):
    # the entries for negative distances are selected by keys that no row sees: later behaviours under the causal
    # flag, slots past a history's end.  Whatever they hold, the outputs are the same bits.
    spec = W.shrink(W.CONFIG2, name=f"bias-unseen-{L}-{n_pos}", B=2, L=L, L_min=L - 30, sub_len=sub, M=40, H=2, nan_padding=True,
                    qk_scale=qk_scale, seed=970 + L)
    w = W.add_bias_inputs(W.make_attention(spec), n_pos=n_pos, n_time=12)
    for b in range(2):
        w["hist_pos"][w["tok_off"][b] + w["hist_len"][b]:w["tok_off"][b + 1]] = 2 ** 30
    outs = []
    for fill in (0.0, np.nan, np.inf):
        w["pos_table"] = w["pos_table"].copy()
        w["pos_table"][..., :(n_pos - 1) // 2] = fill
        g = GpuBias(w, causal=causal)
        outs.append(((g.history_bias() if causal else None), (g.history(want_output=False), g.sumi_bias())[1]))
    for oh, oc in outs[1:]:
        assert np.array_equal(oc, outs[0][1])
        assert oh is None or np.array_equal(oh, outs[0][0])
    assert np.isfinite(outs[0][1]).all()


@pytest.mark.parametrize("L", [40, 300])
def test_bf16_bias_few_and_many_candidates_give_the_same_bits(L):
    # 128-query tiles up to 512 workgroups, 256-query tiles beyond: 33000 candidates of two heads in one call, 700 of them
    spec = W.shrink(W.CONFIG2, name=f"bias-tiles-{L}", B=1, L=L, sub_len=0, M=33000, H=2, pad_to=64, nan_padding=True, seed=980 + L)
    w = W.add_bias_inputs(W.make_attention(spec), n_pos=33, n_time=12)
    g = GpuBias(w)
    g.history(want_output=False)
    full = g.sumi_bias()
    part = dict(w)
    for n in ("qc", "kc", "vc", "cscen", "cbeh", "cand_pos", "cand_ts"):
        part[n] = np.ascontiguousarray(w[n][:700])
    part["cand_off"] = np.array([0, 700], np.int32)
    g = GpuBias(part)
    g.history(want_output=False)
    got = g.sumi_bias()
    assert np.array_equal(got, full[:700])
    assert max_abs(got, oracle_sumi_bias(part)) < TOL["bf16"]


def check_one_launch_writes_the_bits_of_two(spec, n_pos, n_time, causal):
    """Outputs and the whole cache of the history pass, over what was in both before."""
    import torch
    w = W.add_bias_inputs(W.make_attention(spec), n_pos=n_pos, n_time=n_time)
    say(f"[case] {spec.name} causal={causal}")
    out = []
    for flags in (0, 2):
        g = GpuBias(w, causal=causal)
        g.cfg.flags |= flags
        payload = int(w["tok_off"][-1]) * spec.H * 256
        g.buf[-payload:].fill_(77)
        oh, ok = g.history_bias(), valid_rows(w)
        assert np.isfinite(oh[ok]).all() and np.all(oh[~ok] == 0)
        out.append((oh, g.buf[-payload:].clone()))
    assert np.array_equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert max_abs(out[0][0][ok], oracle_hist_bias(w, causal=causal)[ok]) < TOL["bf16"]


@pytest.mark.parametrize("L,L_min,sub,H,qk_scale", [(1, 1, 0, 1, 0.125), (65, 0, 0, 2, 0.125), (129, 64, 384, 1, 0.125), (300, 1, 256, 3, 0.125),
                                                    (700, 200, 128, 2, 0.125), (500, 300, 512, 2, 12.0), (2200, 1900, 0, 2, 0.125)])
@pytest.mark.parametrize("causal", [False, True])
def test_bf16_bias_history_from_rows_writes_the_bits_of_two_launches(L, L_min, sub, H, qk_scale, causal):
    # tiles of padding only, NaN in the padding, histories of more than the 64 blocks that are classified at a time; 12: the
    # running-maximum pass
    spec = W.shrink(W.CONFIG2, name=f"bias-rows-{L}-{sub}", B=3, L=L, L_min=L_min, sub_len=sub, M=1, H=H, pad_to=64, nan_padding=True,
                    qk_scale=qk_scale, seed=990 + L)
    check_one_launch_writes_the_bits_of_two(spec, 33, 12, causal)


@pytest.mark.parametrize("B,L,H,n_scen,n_beh,n_pos", [(44, 300, 8, 1, 1, 483), (44, 300, 8, 1, 1, 497), (5, 255, 2, 8, 4, 257), (5, 256, 2, 8, 4, 257)])
@pytest.mark.parametrize("causal", [False, True])
def test_bf16_bias_history_from_rows_by_tables_and_workgroups(B, L, H, n_scen, n_beh, n_pos, causal):
    # 1056 workgroups: three per CU with tables of 503 entries, two with 517; tables beyond LDS: from rows with walks below
    # 256 keys or the causal flag, else two launches either way
    spec = W.shrink(W.CONFIG2, name=f"bias-rows-by-{n_pos}-{L}", B=B, L=L, L_min=L - 60, sub_len=0, M=1, H=H, pad_to=64, nan_padding=True,
                    n_scen=n_scen, n_beh=n_beh, seed=1100 + n_pos)
    check_one_launch_writes_the_bits_of_two(spec, n_pos, 20, causal)


@pytest.mark.parametrize("n_scen,n_beh,n_pos,n_time", [(8, 4, 195, 13), (1, 1, 6645, 12), (8, 4, 129, 20)])
def test_bf16_bias_tables_up_to_and_beyond_what_lds_holds(n_scen, n_beh, n_pos, n_time):
    # as many entries a head as are copied into LDS (6656), one more (looked up in global memory), and a usual size in between;
    # both passes, 128- and 256-query tiles
    for B, M in ((2, 130), (20, 520)):
        spec = W.shrink(W.CONFIG2, name=f"bias-lds-{n_pos}-{B}", B=B, L=300, L_min=200, sub_len=256, M=M, H=8, n_scen=n_scen, n_beh=n_beh,
                        pad_to=64, seed=1000 + n_pos)
        check_bias(W.add_bias_inputs(W.make_attention(spec), n_pos=n_pos, n_time=n_time))


@pytest.mark.parametrize("n_pos", [2791, 2793])
@pytest.mark.parametrize("causal", [False, True])
def test_bf16_bias_history_with_tables_that_just_leave_room_for_three_workgroups(n_pos, causal):
    # 1056 workgroups, two rings: 42496 bytes and the entries, and four flags behind them, in 53760 (a third of what LDS gives out), and 4 more
    spec = W.shrink(W.CONFIG2, name=f"bias-rows-three-{n_pos}", B=44, L=300, L_min=240, sub_len=0, M=1, H=8, pad_to=64, nan_padding=True,
                    n_scen=1, n_beh=1, seed=1200)
    check_one_launch_writes_the_bits_of_two(spec, n_pos, 20, causal)


@pytest.mark.parametrize("B,M,n_pos,n_time", [(33, 300, 65, 12), (24, 512, 65, 12), (32, 512, 33, 12), (33, 300, 97, 20), (33, 129, 33, 12),
                                              (24, 512, 257, 20), (33, 300, 257, 20)])
def test_bf16_bias_candidate_tiles_by_the_share_of_the_busiest_cu(B, M, n_pos, n_time):
    # tiles of 128 where they leave the busiest CU fewer queries or fill better (tables that leave room for three workgroups per CU, 65 + 12
    # entries, and that do not, 97 + 20; beyond LDS, 257 + 20), of 256 else (512 of 32; 129 of 33), against single users, which take 128: the same bits.  Histories of
    # one to five tiles of 64 keys: both rings' ends
    spec = W.shrink(W.CONFIG2, name=f"bias-share-{B}-{M}", B=B, L=320, L_min=20, sub_len=128, M=M, H=8, pad_to=64, nan_padding=True, seed=1300 + M)
    w = W.add_bias_inputs(W.make_attention(spec), n_pos=n_pos, n_time=n_time)
    g = GpuBias(w)
    g.history(want_output=False)
    full = g.sumi_bias()
    assert np.isfinite(full).all() and max_abs(full, oracle_sumi_bias(w)) < TOL["bf16"]
    for b in (0, B // 2, B - 1):
        part, c = dict(w), slice(int(w["cand_off"][b]), int(w["cand_off"][b + 1]))
        for n in ("qc", "kc", "vc", "cscen", "cbeh", "cand_pos", "cand_ts"):
            part[n] = np.ascontiguousarray(w[n][c])
        part["cand_off"] = np.array([0] * (b + 1) + [c.stop - c.start] * (B - b), np.int32)
        g = GpuBias(part)
        g.history(want_output=False)
        assert np.array_equal(g.sumi_bias(), full[c])


@pytest.mark.parametrize("B,M,M_min,n_pos,three", [(24, 512, None, 257, True), (33, 300, None, 257, True), (30, 300, 75, 257, False), (8, 512, None, 257, False),
                                                   (24, 512, None, 33, True), (33, 300, None, 33, True), (16, 512, None, 33, False), (33, 300, None, 129, False)])
def test_bf16_bias_candidates_have_the_third_workgroup_that_the_choice_of_tiles_counts_on(B, M, M_min, n_pos, three):
    # 128-query tiles because three workgroups of them fit a CU, with the tables in LDS (33 + 12 entries of 32 rows) and beyond it (257 + 12): then
    # registers (512 a SIMD) and LDS (160 KiB a CU, given out by 1280 bytes) hold three.  No more than two a CU, or tables that leave room
    # for two (129 + 12): the instance for two
    spec = W.shrink(W.CONFIG2, name=f"bias-three-{B}-{M}-{n_pos}", B=B, L=64, L_min=64, sub_len=0, M=M, M_min=M_min, H=8, pad_to=64, seed=1400 + M)
    g = GpuBias(W.add_bias_inputs(W.make_attention(spec), n_pos=n_pos, n_time=12))
    g.history(want_output=False)
    o = g.torch.empty((int(g.w["cand_off"][-1]), g.d), dtype=g.dt, device="cuda:0")
    run = launches(lambda: g.launch_sumi_bias(o))
    say([tuple(k) for k in run])
    assert len(run) == 1 and "attn_bias_kernelILi1ELb1" in run[0].kernel
    assert run[0].kernel.split("EEEv")[0].endswith("Li3" if three else "Li2")
    if three:
        assert run[0].regs <= 168 and (run[0].lds + 1279) // 1280 * 1280 * 3 <= 160 * 1024


@pytest.mark.parametrize("causal", [False, True])
def test_bf16_bias_history_from_the_cache_beyond_lds_takes_the_third_workgroup_under_the_causal_flag(causal):
    # (what a call that asks for two launches, or puts its outputs over the keys or values, takes; without the flag two per CU)
    spec = W.shrink(W.CONFIG2, name="bias-cached-three", B=5, L=300, L_min=200, sub_len=0, M=1, H=8, pad_to=64, seed=1500)
    g = GpuBias(W.add_bias_inputs(W.make_attention(spec), n_pos=257, n_time=12), causal=causal)
    g.cfg.flags |= 2
    o = g.torch.empty((g.qh.shape[0], g.d), dtype=g.dt, device="cuda:0")
    run = launches(lambda: g.P.climber_attn_history_bias(g.cfg, g.tau, g.qh, g.kh, g.vh, g.scen, g.beh, g.cache, 0, o, g.rb))
    say([tuple(k) for k in run])
    k = next(k for k in run if "attn_bias_kernel" in k.kernel)
    assert k.kernel.split("EEEv")[0].endswith("Li3" if causal else "Li2") and (k.regs <= 168 or not causal)
