"""GPU parity of the bit-wise gating fusion module (Sec. 3.1.4, Eq. (4)) and of the paper-faithful
multi-block scoring it closes: one block (own weights, own cache) per subsequence, the candidate scored
against each block on its own, the N_b block outputs fused into a score.  Reference: the oracle's bgf()
and its stack functions, same seeded inputs; tolerance 2e-2 max-abs (unit-scale values)."""
import re

import numpy as np
import pytest

import workloads as W
from harness import GpuStack, launches, max_abs, oracle, oracle_stack_config, say, stack_config

pytestmark = pytest.mark.gpu
GIVEN_F32 = re.compile(r"gemm_small_kernelI\w*Li2EEEv")   # (its last template argument)


def gpu_bgf(P, torch, cfg, w, e, run=None):
    """Y and scores; run: a list that receives the mangled names of the kernels launched."""
    dev, bf = "cuda:0", torch.bfloat16
    m, nb, dg = e.shape[0], w["n_blocks"], w["d_gate"]
    atl = {n.lower(): torch.from_numpy(w["atl"][n]).to(dev).to(bf).contiguous() for n in ("g1", "Wqkv", "Wo", "g2", "W1", "W2")}
    wd = torch.from_numpy(w["w_down"]).to(dev).to(bf).contiguous()
    wu = torch.from_numpy(w["w_up"]).to(dev).to(bf).contiguous()
    wh = torch.from_numpy(w["w_head"]).to(dev)
    ts = torch.from_numpy(w["tau_scen"]).to(dev)
    et = torch.from_numpy(np.ascontiguousarray(e, np.float32)).to(dev)
    sc = torch.from_numpy(w["scen"]).to(dev)
    ws = torch.empty(P.climber_bgf_workspace_bytes(cfg, nb, dg, m), dtype=torch.uint8, device=dev)
    y = torch.full(et.shape, float("nan"), dtype=torch.float32, device=dev)
    score = torch.full((m,), float("nan"), dtype=torch.float32, device=dev)
    P.climber_bgf_score(cfg, atl, wd, wu, wh, ts, float(w["b_head"]), nb, dg, et, sc, m, y, score, ws)
    # the same without the optional output
    score2 = torch.empty_like(score)
    P.climber_bgf_score(cfg, atl, wd, wu, wh, ts, float(w["b_head"]), nb, dg, et, sc, m, None, score2, ws)
    torch.cuda.synchronize()
    assert torch.equal(score, score2)
    if run is not None:
        run += [k.kernel for k in launches(lambda: P.climber_bgf_score(cfg, atl, wd, wu, wh, ts, float(w["b_head"]), nb, dg, et, sc, m, y, score, ws))]
    return y.cpu().numpy(), score.cpu().numpy()


def check_bgf(spec, nb, dg, m):
    import torch
    import paper_2502_09888_amd as P
    say(f"[case] bgf {spec.name} d={spec.d_model} F={spec.d_ffn} n_blocks={nb} d_gate={dg} m={m}")
    w = W.make_bgf(spec, nb, dg, m)
    cfg = stack_config(spec)
    y, sc = gpu_bgf(P, torch, cfg, w, w["e"])
    _, yr, scr = oracle.bgf(oracle_stack_config(spec), w["atl"], w["tau_scen"], w["w_down"], w["w_up"], w["w_head"],
                            w["b_head"], w["e"], w["scen"])
    ey, es = max_abs(y, yr), max_abs(sc, scr)
    say(f"  fused Y max-abs {ey:.3e} (|Y| rms {np.sqrt((yr ** 2).mean()):.3f}), score max-abs {es:.3e} "
        f"(score std {scr.std():.3f})")
    assert np.isfinite(y).all() and ey < 2e-2 and es < 2e-2


def test_bgf_small_and_odd_counts():
    spec = W.StackSpec("bgf-small", B=1, L=128, sub_len=0, M=1, n_layers=1, d_model=128, H=2, dh=64, d_ffn=256,
                       n_scen=8, n_beh=4, seed=51)
    check_bgf(spec, nb=4, dg=128, m=301)
    check_bgf(spec, nb=1, dg=128, m=7)
    check_bgf(spec, nb=3, dg=256, m=64)
    # many blocks: the attention kernel is instantiated per block count up to 16
    check_bgf(spec, nb=16, dg=128, m=45)
    check_bgf(spec, nb=7, dg=128, m=130)


def test_bgf_config4_width():
    spec = W.StackSpec("bgf-cfg4", B=1, L=128, sub_len=0, M=1, n_layers=1, d_model=512, H=8, dh=64, d_ffn=2048,
                       n_scen=8, n_beh=4, seed=52)
    check_bgf(spec, nb=4, dg=256, m=1024)


def test_multi_block_scoring_end_to_end():
    # Sec. 3.1.2 + 3.1.4: N_b = 2 blocks with weights of their own; block k encodes subsequence k only and
    # scores every candidate against it; the two block outputs per candidate are fused into a score
    import torch
    import paper_2502_09888_amd as P
    nb, sub, B, M = 2, 128, 3, 40
    specs = [W.StackSpec(f"block{k}", B=B, L=sub, sub_len=0, M=M, n_layers=2, d_model=128, H=2, dh=64, d_ffn=256,
                         n_scen=8, n_beh=4, seed=60 + k, hist_lens=(128, 77, 100)) for k in range(nb)]
    say(f"[case] multi-block: {nb} blocks of {sub} tokens, B={B}, M={M}")
    ws_ = [W.make_stack(s) for s in specs]
    # the candidates (embeddings and ids) are the same for every block
    for w in ws_[1:]:
        for n in ("x_cand", "cscen", "cbeh", "cand_off"):
            w[n] = ws_[0][n]
    e_gpu, e_ref = [], []
    for spec, w in zip(specs, ws_):
        g = GpuStack(w)
        g.encode()
        e_gpu.append(g.score())
        cfg = oracle_stack_config(spec)
        kc, vc, _ = oracle.stack_encode(cfg, w["layers"], w["tau"], w["tok_off"], w["hist_len"],
                                        np.nan_to_num(w["x_hist"]), w["scen"], w["beh"])
        e_ref.append(oracle.stack_score(cfg, w["layers"], w["tau"], w["tok_off"], w["hist_len"], kc, vc,
                                        w["cand_off"], w["x_cand"], w["cscen"], w["cbeh"]))
    e_gpu, e_ref = np.stack(e_gpu, axis=1), np.stack(e_ref, axis=1)      # [m, n_blocks, d]
    assert max_abs(e_gpu, e_ref) < 2e-2
    fw = W.make_bgf(specs[0], nb, 128, e_gpu.shape[0])
    fw["scen"] = ws_[0]["cscen"]
    _, sc = gpu_bgf(P, torch, stack_config(specs[0]), fw, e_gpu)
    _, _, scr = oracle.bgf(oracle_stack_config(specs[0]), fw["atl"], fw["tau_scen"], fw["w_down"], fw["w_up"],
                           fw["w_head"], fw["b_head"], e_ref, fw["scen"])
    e = max_abs(sc, scr)
    say(f"  block outputs max-abs {max_abs(e_gpu, e_ref):.3e}, final scores max-abs {e:.3e} (std {scr.std():.3f})")
    assert e < 2e-2


@pytest.mark.parametrize("d, nb, dg, m, part", [(512, 4, 128, 2049, 33), (512, 3, 256, 2731, 1), (256, 8, 128, 1025, 16), (256, 2, 256, 4129, 40),
                                                (256, 3, 256, 2095, 64), (256, 1, 128, 1500, 9), (512, 5, 256, 6001, 32)])
def test_few_and_many_candidates_give_the_same_bits(d, nb, dg, m, part):
    # 4000 rows or more of 2 to 8 blocks: projection and attention are one launch, above 4096 rows the tail is, from the lines of the gate on it is,
    # the last 32 candidates of it in part; few candidates: launches of their own
    few_against_many(d, nb, dg, m, part)


def few_against_many(d, nb, dg, m, part):
    """Both calls' launches, after a comparison of their bits."""
    import torch
    import paper_2502_09888_amd as P
    spec = W.StackSpec(f"bgf-many-{d}", B=1, L=128, sub_len=0, M=1, n_layers=1, d_model=d, H=d // 64, dh=64, d_ffn=256, n_scen=8, n_beh=4,
                       seed=57)
    say(f"[case] {spec.name} n_blocks={nb} m={m}")
    w = W.make_bgf(spec, nb, dg, m)
    cfg = stack_config(spec)
    many, ran = [], []
    y, sc = gpu_bgf(P, torch, cfg, w, w["e"], many)
    for lo in (0, m - part):
        few = dict(w, scen=np.ascontiguousarray(w["scen"][lo:lo + part]))
        y1, sc1 = gpu_bgf(P, torch, cfg, few, w["e"][lo:lo + part], ran)
        assert np.isfinite(y1).all() and np.array_equal(y1, y[lo:lo + part]) and np.array_equal(sc1, sc[lo:lo + part])
    return ran, many


def ran_among(run, part):
    return any(part in k for k in run)


@pytest.mark.parametrize("d, nb, dg, m, part", [(512, 9, 128, 913, 1), (512, 9, 256, 911, 40), (512, 16, 128, 521, 33), (512, 1, 256, 8193, 64), (256, 16, 128, 513, 5),
                                                (256, 1, 128, 8257, 9), (256, 9, 256, 1000, 300)])
def test_projection_of_many_fp32_rows_makes_their_sums(d, nb, dg, m, part):
    # one block or more than eight, more than 8192 rows: the projection with its rows in LDS rounds them and forms their sums, the last 64 of them in part,
    # and the attention is a launch of its own; against calls of few rows, whose projection is another kernel
    few, many = few_against_many(d, nb, dg, m, part)
    assert ran_among(many, f"gemm_resident_kernelILi{d}E") and ran_among(many, f"bgf_attention_kernelILi{nb}E") and not ran_among(many, "row_prep_kernel")
    assert not ran_among(few, "gemm_resident_kernel")


@pytest.mark.parametrize("d, nb, dg, m, part", [(512, 4, 256, 3425, 33), (512, 7, 256, 6017, 1), (256, 5, 256, 2717, 28), (512, 3, 128, 2815, 31), (512, 7, 128, 3210, 40),
                                                (512, 4, 256, 2401, 17), (256, 5, 256, 2699, 3), (512, 7, 128, 2101, 35)])
def test_one_launch_of_a_wide_gate_gives_the_bits_of_three(d, nb, dg, m, part):
    # from its lines on, the last 32 candidates in part, an even and an odd number of steps; the last three are one launch with Y alone, so that their scores
    # come from both ways
    few, many = few_against_many(d, nb, dg, m, part)
    assert ran_among(many, f"bgf_gate_kernelILi{dg}E") and ran_among(few, "bgf_gate_head_kernel") and not ran_among(few, "bgf_gate_kernel")


@pytest.mark.parametrize("d, nb, m, part", [(512, 4, 300, 1), (512, 4, 300, 9), (512, 4, 300, 256), (512, 3, 700, 113), (512, 8, 600, 128), (256, 4, 600, 5),
                                            (256, 4, 600, 512), (256, 1, 2100, 673), (256, 9, 300, 227)])
def test_first_projection_of_few_fp32_rows_makes_their_sums(d, nb, m, part):
    # the fusion layer's projection of few rows forms the sums of squares of its fp32 rows, in blocks of 16 or 32 of them, the last in part, up
    # to the most rows there are; against a call of more, which has a launch for that before, or (4800 rows of 8 blocks) one launch to the attention
    few, many = few_against_many(d, nb, 128, m, part)
    own = lambda run: any("gemm_small_kernel" in k and GIVEN_F32.search(k) for k in run)
    assert own(few) and not ran_among(few, "row_prep_kernel")
    assert not own(many) and ran_among(many, "row_prep_kernel") != ran_among(many, "bgf_front_kernel")


@pytest.mark.parametrize("d, nb, m", [(512, 2, 2001), (256, 2, 2063), (512, 3, 2049), (256, 3, 2069), (512, 4, 1000), (256, 4, 1017), (512, 5, 1229),
                                      (256, 5, 1235), (512, 6, 667), (256, 6, 675), (512, 7, 572), (256, 7, 577), (512, 8, 500), (256, 8, 509)])
def test_projection_and_attention_in_one_launch_give_the_bits_of_two(d, nb, m):
    # two blocks a workgroup of as many whole candidates as 32 lanes hold, the last of them with one or a few: against calls
    # for few candidates, which take a launch each.  A candidate of NaN and one of infinities reach no other's rows.
    import torch
    import paper_2502_09888_amd as P
    spec = W.StackSpec(f"bgf-front-{d}-{nb}", B=1, L=128, sub_len=0, M=1, n_layers=1, d_model=d, H=d // 64, dh=64, d_ffn=256, n_scen=8, n_beh=4, seed=61)
    say(f"[case] {spec.name} m={m}")
    w = W.make_bgf(spec, nb, 128, m)
    cfg, dev, bf = stack_config(spec), "cuda:0", torch.bfloat16
    atl = {n.lower(): torch.from_numpy(w["atl"][n]).to(dev).to(bf).contiguous() for n in ("g1", "Wqkv", "Wo", "g2", "W1", "W2")}
    wd, wu = (torch.from_numpy(w[n]).to(dev).to(bf).contiguous() for n in ("w_down", "w_up"))
    wh, ts, scen = (torch.from_numpy(w[n]).to(dev) for n in ("w_head", "tau_scen", "scen"))
    e = torch.from_numpy(w["e"]).to(dev)
    e[5], e[m - 2] = float("nan"), float("inf")
    ws = torch.empty(P.climber_bgf_workspace_bytes(cfg, nb, 128, m), dtype=torch.uint8, device=dev)

    def call(lo, n):
        y, score, part, sc = torch.zeros(n, nb, d, device=dev), torch.zeros(n, device=dev), e[lo:lo + n].clone(), scen[lo:lo + n].clone()
        return lambda: P.climber_bgf_score(cfg, atl, wd, wu, wh, ts, 0.25, nb, 128, part, sc, n, y, score, ws), y, score

    go, y, score = call(0, m)
    run = launches(go)
    assert any("bgf_front_kernel" in k.kernel for k in run) and not any("bgf_attention_kernel" in k.kernel for k in run)
    go()
    for lo, n in ((0, 5), (6, 34), (m - 40, 38), (m - 1, 1)):
        few, y1, score1 = call(lo, n)
        few()
        assert y1.isfinite().all() and torch.equal(y1, y[lo:lo + n]) and torch.equal(score1, score[lo:lo + n])
    assert score[[5, m - 2]].isnan().all()


@pytest.mark.parametrize("d, nb, dg, m, one", [(512, 4, 256, 2048, False), (512, 4, 256, 3399, False), (512, 4, 256, 3400, True), (256, 3, 256, 2048, False), (256, 3, 256, 2049, True),
                                               (512, 2, 256, 2699, False), (256, 7, 256, 2700, True), (512, 8, 256, 5999, False), (512, 8, 256, 6000, True),
                                               (512, 8, 128, 1499, False), (512, 8, 128, 3199, False), (512, 8, 128, 3200, True), (512, 16, 128, 4999, False), (512, 16, 128, 5000, True)])
def test_the_gate_is_one_launch_where_that_was_measured_to_be_faster(d, nb, dg, m, one, with_y=False):
    import torch
    import paper_2502_09888_amd as P
    spec = W.StackSpec("bgf-launches", B=1, L=128, sub_len=0, M=1, n_layers=1, d_model=d, H=d // 64, dh=64, d_ffn=256, n_scen=8, n_beh=4, seed=59)
    cfg, bf = stack_config(spec), dict(dtype=torch.bfloat16, device="cuda:0")
    atl = {k: torch.zeros(s, **bf) for k, s in (("g1", d), ("wqkv", (d, 3 * d)), ("wo", (d, d)), ("g2", d), ("w1", (d, 256)), ("w2", (256, d)))}
    wd, wu = torch.zeros(nb * d, dg, **bf), torch.zeros(dg, nb * d, **bf)
    wh, ts, e = torch.zeros(nb * d, device="cuda:0"), torch.ones(8, device="cuda:0"), torch.ones(m, nb, d, device="cuda:0")
    sc, score = torch.zeros(m, dtype=torch.int32, device="cuda:0"), torch.empty(m, device="cuda:0")
    ws = torch.empty(P.climber_bgf_workspace_bytes(cfg, nb, dg, m), dtype=torch.uint8, device="cuda:0")
    run = launches(lambda: P.climber_bgf_score(cfg, atl, wd, wu, wh, ts, 0.5, nb, dg, e, sc, m, torch.empty_like(e) if with_y else None, score, ws))
    say([tuple(k)[:2] for k in run])
    assert (score == 0.5).all()
    assert any("bgf_gate_kernel" in k.kernel for k in run) == one and any("bgf_gate_head_kernel" in k.kernel for k in run) != one


@pytest.mark.parametrize("d, nb, dg, m, one", [(512, 4, 256, 2399, False), (512, 4, 256, 2400, True), (512, 2, 256, 2399, False), (256, 7, 256, 2400, True),
                                               (256, 3, 256, 2049, True), (512, 8, 256, 5999, False), (512, 7, 128, 2099, False), (512, 7, 128, 2100, True),
                                               (512, 8, 128, 3199, False), (512, 8, 128, 3200, True), (512, 6, 128, 2799, False)])
def test_the_gate_with_its_rows_out_is_one_launch_from_fewer_candidates_on(d, nb, dg, m, one):
    test_the_gate_is_one_launch_where_that_was_measured_to_be_faster(d, nb, dg, m, one, with_y=True)


@pytest.mark.parametrize("d, nb, m, one", [(512, 2, 1499, False), (512, 2, 1500, True), (256, 5, 2799, False), (256, 5, 2800, True), (512, 6, 2799, False), (512, 6, 2800, True)])
def test_the_narrow_gate_is_three_launches_further_on_with_rows_of_1280_to_3072(d, nb, m, one):
    test_the_gate_is_one_launch_where_that_was_measured_to_be_faster(d, nb, 128, m, one)
