"""GPU parity of sc_encoder_attn_stack (QKV GEMM, sparse attention, scores,
pruning, Wo GEMM, residual + LayerNorm, layer after layer) against the CPU
oracle, compared layer by layer: each oracle layer starts from the GPU's
previous-layer output (re-sync), so that one legitimate near-threshold flip
cannot cascade through the later layers' geometry.  On every layer and
sequence, the hidden rows of every token that both sides keep are compared,
matched by the token's index in the layer input; kept-list differences are
allowed only for tokens whose oracle score lies within 1e-6 of the threshold,
and their count is asserted and recorded."""
import numpy as np
import pytest
import torch

import oracle
import sc_inputs as si
from gpu_helpers import DEV, NEAR_THETA, check_out, dev_i32, log, record

import paper_2310_07109_amd as sc

pytestmark = pytest.mark.gpu


def bf16_dev(a_bits):
    return torch.from_numpy(np.ascontiguousarray(a_bits).view(np.int16)).to(DEV).view(torch.bfloat16)


def to_f64(t, lens=None):
    """Device bf16 tensor [B, n, D] -> float64; with lens, rows at or beyond lens[b] (never written by a
    compacting call) are zeroed instead of converted."""
    a = t.float().cpu().numpy()
    if lens is not None:
        for b in range(a.shape[0]):
            a[b, int(lens[b]):] = 0.0
    return a.astype(np.float64)


def run_layer(x_t, wq_t, wo_t, vl, gp, H, window, alpha, theta, w1_t=None, w2_t=None):
    B, n, D = x_t.shape
    d = sc.Desc(B, n, H, window, dev_i32(vl), dev_i32(gp), alpha, sc.SC_BF16)
    if w1_t is None:
        y, fl, orig, kpl = sc.sc_encoder_attn_stack(d, x_t, [wq_t], [wo_t], [theta])
    else:
        y, fl, orig, kpl = sc.sc_encoder_stack(d, x_t, [wq_t], [wo_t], [w1_t], [w2_t], [theta], windows=[window])
    torch.cuda.synchronize()
    return y, fl.cpu().numpy(), orig.cpu().numpy()


def remap_globals(gp, orig, new_len):
    """Global positions after pruning (globals are kept): their index in the compacted sequence."""
    out = np.full_like(gp, -1)
    for b in range(gp.shape[0]):
        pos = {int(o): j for j, o in enumerate(orig[b, :new_len[b]])}
        new = sorted(pos[int(p)] for p in gp[b] if p >= 0 and int(p) in pos)
        out[b, :len(new)] = new
    return out


def layerwise(x_bits, wq_bits, wo_bits, vl, gp, H, window, alpha, thetas, seqs=None, tag="", w1_bits=None,
              w2_bits=None, windows=None):
    """Run the stack one layer at a time on the GPU; check each layer against the oracle on `seqs` (default:
    every sequence).  w1_bits / w2_bits: feed-forward weights per layer (full layers); windows: one per layer."""
    x_t = bf16_dev(x_bits)
    seqs = list(range(x_bits.shape[0])) if seqs is None else seqs
    excluded_total = flips_total = rows_checked = 0
    beyond = [0]
    for l, theta in enumerate(thetas):
        wq_t, wo_t = bf16_dev(wq_bits[l]), bf16_dev(wo_bits[l])
        win = windows[l] if windows is not None else window
        ffn = {}
        if w1_bits is not None:
            ffn = dict(w1=si.bf16_bits_to_f64(w1_bits[l]), w2=si.bf16_bits_to_f64(w2_bits[l]))
            y_t, nl, orig = run_layer(x_t, wq_t, wo_t, vl, gp, H, win, alpha, theta, bf16_dev(w1_bits[l]),
                                      bf16_dev(w2_bits[l]))
        else:
            y_t, nl, orig = run_layer(x_t, wq_t, wo_t, vl, gp, H, win, alpha, theta)
        x64 = to_f64(x_t, vl)[seqs]
        ry, rk, rnl, rngp, rs = oracle.encoder_layer(x64, si.bf16_bits_to_f64(wq_bits[l]),
                                                     si.bf16_bits_to_f64(wo_bits[l]), vl[seqs], gp[seqs], H, win,
                                                     alpha, theta, **ffn)
        y = to_f64(y_t, nl)
        for i, b in enumerate(seqs):
            L = int(vl[b])
            g = {int(p) for p in gp[b] if 0 <= p < L}
            near = {k for k in range(L) if abs(float(rs[i, k]) - theta) <= NEAR_THETA} - g
            kept_gpu = [int(k) for k in orig[b, :nl[b]]]
            kept_ref = [int(k) for k in rk[i, :rnl[i]]]
            flips = set(kept_gpu) ^ set(kept_ref)
            excluded_total += len(near)
            flips_total += len(flips)
            assert flips <= near, f"layer {l} seq {b}: kept sets differ outside the near-threshold band"
            # hidden rows of the tokens both sides keep, matched by index in the layer input
            row_ref = {k: j for j, k in enumerate(kept_ref)}
            both = [(j, row_ref[k]) for j, k in enumerate(kept_gpu) if k in row_ref]
            if both:
                jg, jr = (np.array(v) for v in zip(*both))
                check_out(y[b, jg], ry[i, jr], "bf16", what=f"layer {l} seq {b} hidden", bf16_step=True,
                          count_beyond=beyond)
                rows_checked += len(both)
        assert flips_total <= excluded_total
        log(f"{tag} layer {l}: theta {theta:.5f} kept {nl.tolist()}")
        gp = remap_globals(gp, orig, nl)
        vl = nl.astype(np.int32)
        x_t = y_t
    record(f"{tag}: {len(thetas)} layers, {len(seqs)} sequences through the oracle, {rows_checked} hidden rows "
           f"compared ({beyond[0]} elements one bf16 step beyond 2e-2), near-theta excluded {excluded_total}, "
           f"kept-list flips {flips_total}")
    return x_t, vl


def test_small_stack_layerwise_and_chained():
    cfg = si.StackConfig("small", 21, 3, 300, 2, 64, 4, 64, (120, 300), 1, 0.05, 0.012)
    inp = si.make_stack_inputs(cfg)
    inp["valid_len"][1] = 1  # a one-token sequence
    inp["global_pos"] = si.global_positions(cfg.seed, inp["valid_len"], 1, "first")
    thetas = [0.0, 0.004, 0.008, 0.012]
    xl, vl_final = layerwise(inp["x"], inp["wqkv"], inp["wo"], inp["valid_len"], inp["global_pos"], cfg.H,
                             cfg.window, cfg.alpha, thetas, tag="small")
    # the multi-layer call equals the chain of single-layer calls, bit for bit
    d = sc.Desc(cfg.B, cfg.n, cfg.H, cfg.window, dev_i32(inp["valid_len"]), dev_i32(inp["global_pos"]), cfg.alpha,
                sc.SC_BF16)
    y, fl, orig, kpl = sc.sc_encoder_attn_stack(d, bf16_dev(inp["x"]), [bf16_dev(w) for w in inp["wqkv"]],
                                                [bf16_dev(w) for w in inp["wo"]], thetas)
    fl = fl.cpu().numpy()
    assert np.array_equal(fl, vl_final)
    assert np.array_equal(kpl.cpu().numpy()[-1], fl)
    for b in range(cfg.B):
        assert torch.equal(y[b, :fl[b]].view(torch.int16), xl[b, :fl[b]].view(torch.int16))
        o = orig.cpu().numpy()[b]
        assert np.all(o[fl[b]:] == -1) and np.all(np.diff(o[:fl[b]]) > 0)


def test_stack_no_pruning_keeps_all():
    cfg = si.StackConfig("nop", 22, 2, 130, 2, 64, 3, 32, (100, 130), 1, 0.05, 0.0)
    inp = si.make_stack_inputs(cfg)
    d = sc.Desc(cfg.B, cfg.n, cfg.H, cfg.window, dev_i32(inp["valid_len"]), dev_i32(inp["global_pos"]), cfg.alpha,
                sc.SC_BF16)
    y, fl, orig, kpl = sc.sc_encoder_attn_stack(d, bf16_dev(inp["x"]), [bf16_dev(w) for w in inp["wqkv"]],
                                                [bf16_dev(w) for w in inp["wo"]], [-1.0] * 3)
    assert np.array_equal(fl.cpu().numpy(), inp["valid_len"])
    for b in range(cfg.B):
        assert list(orig.cpu().numpy()[b, :inp["valid_len"][b]]) == list(range(inp["valid_len"][b]))
    ry, rfl, roi, rkpl = oracle.encoder_stack(inp["x64"], inp["wqkv64"], inp["wo64"], inp["valid_len"],
                                              inp["global_pos"], cfg.H, cfg.window, cfg.alpha, [-1.0] * 3)
    yy = to_f64(y, inp["valid_len"])
    for b in range(cfg.B):
        L = int(inp["valid_len"][b])
        check_out(yy[b, :L], ry[b, :L], "bf16", what="unpruned stack", bf16_step=True)


def test_config3_stack_all_sequences():
    """RoBERTa-shaped 12-layer stack, B16 n2048, every sequence through the oracle, layer by layer."""
    cfg = si.STACK_CONFIG
    log("config 3: generating inputs")
    inp = si.make_stack_inputs(cfg)
    vl = inp["valid_len"]
    log(f"config 3: lengths {vl.tolist()}")
    layerwise(inp["x"], inp["wqkv"], inp["wo"], vl, inp["global_pos"], cfg.H, cfg.window, cfg.alpha,
              cfg.thresholds(), tag="config 3 stack")


def test_small_full_stack_layerwise_and_chained():
    """Full layers (GELU feed-forward block) with a window per layer, layer by layer against the oracle; the
    multi-layer call equals the chain of single-layer calls bit for bit."""
    cfg = si.StackConfig("small full", 23, 3, 300, 2, 64, 4, 64, (120, 300), 1, 0.05, 0.012, ffn_dim=512,
                         windows=(8, 32, 64, 600))
    inp = si.make_stack_inputs(cfg)
    inp["valid_len"][2] = 1
    inp["global_pos"] = si.global_positions(cfg.seed, inp["valid_len"], 1, "first")
    thetas = [0.0, 0.004, 0.008, 0.012]
    xl, vl_final = layerwise(inp["x"], inp["wqkv"], inp["wo"], inp["valid_len"], inp["global_pos"], cfg.H,
                             cfg.window, cfg.alpha, thetas, tag="small full", w1_bits=inp["w1"], w2_bits=inp["w2"],
                             windows=inp["windows"])
    d = sc.Desc(cfg.B, cfg.n, cfg.H, cfg.window, dev_i32(inp["valid_len"]), dev_i32(inp["global_pos"]), cfg.alpha,
                sc.SC_BF16)
    dv = lambda ws: [bf16_dev(w) for w in ws]  # noqa: E731
    y, fl, orig, kpl = sc.sc_encoder_stack(d, bf16_dev(inp["x"]), dv(inp["wqkv"]), dv(inp["wo"]), dv(inp["w1"]),
                                           dv(inp["w2"]), thetas, windows=inp["windows"])
    fl = fl.cpu().numpy()
    assert np.array_equal(fl, vl_final)
    for b in range(cfg.B):
        assert torch.equal(y[b, :fl[b]].view(torch.int16), xl[b, :fl[b]].view(torch.int16))


def test_full_stack_unpruned_against_oracle_stack():
    cfg = si.StackConfig("nop full", 24, 2, 130, 2, 64, 3, 32, (100, 130), 1, 0.05, 0.0, ffn_dim=256,
                         windows=(16, 48, 32))
    inp = si.make_stack_inputs(cfg)
    d = sc.Desc(cfg.B, cfg.n, cfg.H, cfg.window, dev_i32(inp["valid_len"]), dev_i32(inp["global_pos"]), cfg.alpha,
                sc.SC_BF16)
    dv = lambda ws: [bf16_dev(w) for w in ws]  # noqa: E731
    y, fl, orig, kpl = sc.sc_encoder_stack(d, bf16_dev(inp["x"]), dv(inp["wqkv"]), dv(inp["wo"]), dv(inp["w1"]),
                                           dv(inp["w2"]), [-1.0] * 3, windows=inp["windows"])
    assert np.array_equal(fl.cpu().numpy(), inp["valid_len"])
    ry, rfl, roi, rkpl = oracle.encoder_stack(inp["x64"], inp["wqkv64"], inp["wo64"], inp["valid_len"],
                                              inp["global_pos"], cfg.H, inp["windows"], cfg.alpha, [-1.0] * 3,
                                              w1_list=inp["w1_64"], w2_list=inp["w2_64"])
    yy = to_f64(y, inp["valid_len"])
    for b in range(cfg.B):
        L = int(inp["valid_len"][b])
        check_out(yy[b, :L], ry[b, :L], "bf16", what="unpruned full stack", bf16_step=True)


def test_full_encoder_config_all_sequences():
    """RoBERTa-base-shaped full encoder (FFN 3072, windows 64..512), B16 n2048, every sequence through the
    oracle, layer by layer."""
    cfg = si.STACK_FULL_CONFIG
    log("full encoder: generating inputs")
    inp = si.make_stack_inputs(cfg)
    vl = inp["valid_len"]
    log(f"full encoder: lengths {vl.tolist()}")
    layerwise(inp["x"], inp["wqkv"], inp["wo"], vl, inp["global_pos"], cfg.H, cfg.window, cfg.alpha,
              cfg.thresholds(), tag="full encoder", w1_bits=inp["w1"], w2_bits=inp["w2"], windows=inp["windows"])


def test_split_reduction_full_layers():
    """RoBERTa-base widths (D 768, FFN 3072) on few short sequences: the surviving rows fill at most seven
    128-row tiles, so the output and second feed-forward products split their 768- and 3072-long reductions
    into float32 slabs that the residual LayerNorm adds in a fixed order.  Layer by layer against the oracle,
    and the two-layer call equals the chain of single-layer calls bit for bit (the split is deterministic)."""
    cfg = si.StackConfig("split full", 25, 4, 300, 12, 64, 2, 64, (120, 300), 1, 0.02, 0.004, ffn_dim=3072,
                         windows=(32, 96))
    inp = si.make_stack_inputs(cfg)
    inp["valid_len"][1] = 7
    inp["valid_len"][2] = 0  # an empty sequence between live ones: no tiles, the plan's offsets skip it
    inp["global_pos"] = si.global_positions(cfg.seed, inp["valid_len"], 1, "first")
    thetas = [0.0, 0.004]
    xl, vl_final = layerwise(inp["x"], inp["wqkv"], inp["wo"], inp["valid_len"], inp["global_pos"], cfg.H,
                             cfg.window, cfg.alpha, thetas, tag="split full", w1_bits=inp["w1"], w2_bits=inp["w2"],
                             windows=inp["windows"])
    d = sc.Desc(cfg.B, cfg.n, cfg.H, cfg.window, dev_i32(inp["valid_len"]), dev_i32(inp["global_pos"]), cfg.alpha,
                sc.SC_BF16)
    dv = lambda ws: [bf16_dev(w) for w in ws]  # noqa: E731
    y, fl, orig, kpl = sc.sc_encoder_stack(d, bf16_dev(inp["x"]), dv(inp["wqkv"]), dv(inp["wo"]), dv(inp["w1"]),
                                           dv(inp["w2"]), thetas, windows=inp["windows"])
    fl = fl.cpu().numpy()
    assert np.array_equal(fl, vl_final)
    for b in range(cfg.B):
        assert torch.equal(y[b, :fl[b]].view(torch.int16), xl[b, :fl[b]].view(torch.int16))
    # run to run: the partial sums are added in a fixed order
    y2, fl2, orig2, kpl2 = sc.sc_encoder_stack(d, bf16_dev(inp["x"]), dv(inp["wqkv"]), dv(inp["wo"]),
                                               dv(inp["w1"]), dv(inp["w2"]), thetas, windows=inp["windows"])
    assert np.array_equal(fl2.cpu().numpy(), fl) and torch.equal(orig2, orig) and torch.equal(kpl2, kpl)
    for b in range(cfg.B):
        assert torch.equal(y2[b, :fl[b]].view(torch.int16), y[b, :fl[b]].view(torch.int16))


@pytest.mark.parametrize("H,F,lens", [
    (2, 128, (1,)),                      # one row; products of two K stages
    (2, 384, (63, 1, 0, 65)),            # 129 rows: one past two 64-row tiles; six K stages
    (4, 512, (64, 64)),                  # whole tiles
    (4, 192, (200, 130, 3)),             # N = 192: not a multiple of 128, the unpacked product
    (12, 3072, (33, 31)),                # RoBERTa widths on one tile: the widest split
    (12, 3072, (700, 650, 640)),         # several items per workgroup
    (6, 768, (1024, 1023, 1000, 1025)),  # more than 4096 padded rows: the three-workgroup product
    (4, 256, (800, 700)),                # one and two ranges of W2's reduction (and of Wo's) are priced alike
    (2, 512, (800, 700)),                # two and four ranges of W2's
    (6, 2304, (1000, 990, 980, 970)),    # W1 has too many tiles for the few-row product, the others not
])
def test_products_of_few_rows(H, F, lens):
    """One unpruned full layer at the edges of the small products' tiles, splits and row limit."""
    B, n = len(lens), max(lens)
    cfg = si.StackConfig("rows", 41, B, n, H, 64, 1, 32, (n, n), 1, 0.04, 0.0, ffn_dim=F, windows=(32,))
    inp = si.make_stack_inputs(cfg)
    vl = np.array(lens, np.int32)
    gp = si.global_positions(41, vl, 1, "first")
    d = sc.Desc(B, n, H, 32, dev_i32(vl), dev_i32(gp), cfg.alpha, sc.SC_BF16)
    dv = lambda ws: [bf16_dev(w) for w in ws]  # noqa: E731
    y, fl, _, _ = sc.sc_encoder_stack(d, bf16_dev(inp["x"]), dv(inp["wqkv"]), dv(inp["wo"]), dv(inp["w1"]),
                                      dv(inp["w2"]), [-1.0], windows=[32])
    assert np.array_equal(fl.cpu().numpy(), vl)
    ry, _, _, _ = oracle.encoder_stack(inp["x64"], inp["wqkv64"], inp["wo64"], vl, gp, H, [32], cfg.alpha, [-1.0],
                                       w1_list=inp["w1_64"], w2_list=inp["w2_64"])
    yy = to_f64(y, vl)
    for b, L in enumerate(lens):
        check_out(yy[b, :L], ry[b, :L], "bf16", what=f"sequence {b}", bf16_step=True)


@pytest.mark.parametrize("H,F", [(3, 0), (3, 256), (1, 0), (1, 192)])
def test_pruned_layers_of_odd_width(H, F):
    """Two pruned layers whose width (64 H) is no multiple of 128: the output projection takes the unpacked product,
    which reads the kept rows through keep_idx (as the residual LayerNorm does, without slabs).  Ragged lengths, with
    sequences of one token and none."""
    lens = (190, 1, 0, 147)
    cfg = si.StackConfig("odd", 53, len(lens), 190, H, 64, 2, 32, (190, 190), 1, 0.08, 0.0, ffn_dim=F,
                         windows=(32, 64) if F else None)
    inp = si.make_stack_inputs(cfg)
    vl = np.array(lens, np.int32)
    gp = si.global_positions(53, vl, 1, "first")
    ffn = dict(w1_bits=inp["w1"], w2_bits=inp["w2"], windows=[32, 64]) if F else {}
    _, left = layerwise(inp["x"], inp["wqkv"], inp["wo"], vl, gp, H, 32, cfg.alpha, [0.0055, 0.009],
                        tag=f"odd width H{H} F{F}", **ffn)
    assert 1 < left[0] < 190 and 1 < left[3] < 147, "the thresholds prune some tokens and keep some"
