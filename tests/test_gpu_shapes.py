"""The routes that sizes choose, at the sizes where they can go wrong, against the oracle: products of few
rows (LayerNorm inside the projection, weights straight to registers), large fp32 products through three
bf16 parts, the encoder of a ragged batch without its padding, its bf16 attention, wide beams."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1906_11024_amd import workloads as wl
from tests import harness as hz
from tests import rules
from tests.test_gpu_parity import BF16_TOL, F32_TOL, _compaction_schedule


def _cfg(**kw):
    cfg = dict(n_enc=1, n_dec=3, d=64, H=4, F=128, V=1004, dtype="f32", batch=1, beam=1, src_len=(3, 9), steps=4,
               self_pi=[2, 1], encdec_pi=[1, 2], self_kind="dot", name="shapes")
    cfg.update(kw)
    return cfg


def _tol(cfg):
    return F32_TOL if cfg["dtype"] == "f32" else BF16_TOL


def _lockstep(cfg, share="A", loop=None, seed=31, **kw):
    w = wl.make_weights(cfg, seed=seed, sharp=4.0)
    w["w_out"] = w["w_out"] * np.float32(8.0)
    if cfg["dtype"] == "bf16":
        w["w_out"] = wl.round_to_bf16(w["w_out"])
    src, lens = wl.make_source(cfg, seed)
    gpu = hz.make_gpu(cfg, w, share=share, **kw)
    ls = hz.Lockstep(gpu, hz.make_oracle(cfg, w, share=share), src, lens, cfg["beam"], loop=loop)
    for _ in range(cfg["steps"]):
        ls.step(logit_tol=_tol(cfg))
    return ls


_FEW = {
    # one row; fewer 64-byte units of k (4, bf16: 2) than the eight waves that share them; ragged vocabulary.  (F = 128: one
    # launch a step.)
    "one_row": dict(),
    "one_row_f192": dict(F=192),
    "one_row_bf16": dict(dtype="bf16", F=64),
    # the last row count of the products of few rows, and the first beyond it
    "rows16": dict(batch=4, beam=4, d=512, H=8, F=1024, V=16388),
    "rows17": dict(batch=17, d=512, H=8, F=1024, V=16388),
    # general route, LayerNorm rows that leave lanes of their one wave idle
    "rows20_d320": dict(batch=5, beam=4, d=320, H=5, F=192),
    "rows20_d320_bf16": dict(dtype="bf16", batch=5, beam=4, d=320, H=5, F=192),
    # widths and row counts around the steps of the kernel's shares
    "rows15_d576_share_s": dict(batch=3, beam=5, d=576, H=9, F=832, share="S"),
    "rows9_d1024": dict(batch=3, beam=3, d=1024, H=16, F=1088, self_pi=[1, 2], encdec_pi=[3]),
    "rows16_d1024_bf16": dict(dtype="bf16", batch=2, beam=8, d=1024, H=16, F=4096, V=16388),
    "rows6_d832_bf16_share_s": dict(dtype="bf16", batch=3, beam=2, d=832, H=13, F=320, share="S", encdec_pi=[3]),
    # wider than any projection with a LayerNorm inside
    "rows4_d1088": dict(batch=2, beam=2, d=1088, H=17, F=256),
    "rows12_aan": dict(batch=3, beam=4, self_kind="aan", self_pi=[1, 1, 1]),
}


@pytest.mark.parametrize("loop", [None, "cands"])
@pytest.mark.parametrize("case", sorted(_FEW))
def test_few_rows_match_oracle(case, loop):
    cfg = _cfg(**_FEW[case])
    share = cfg.pop("share", "A")
    ls = _lockstep(cfg, share, loop)
    assert (ls.gpu.last_launch_count == 1) == (case == "one_row")
    if loop is None:
        assert max(ls.log["logit_err"]) <= _tol(cfg), max(ls.log["logit_err"])
    ls.gpu.close()


# Steps with the LayerNorms inside the projections, at the last row count of each width that takes them (few = 1), and at
# the next, which runs the general launches with products of few rows where those are faster: both kinds of block, one
# LayerNorm or two per projection, split weights shared or not, vocabularies on both sides of the output layer's lines.
@pytest.mark.parametrize("loop", [None, "cands"])
@pytest.mark.parametrize("dtype,d,batch,beam,few,kw", [
    ("f32", 64, 1, 1, 0, {}), ("f32", 128, 1, 4, 1, {}), ("f32", 128, 5, 1, 0, {}), ("f32", 256, 2, 4, 1, dict(V=18436)),
    ("f32", 256, 3, 3, 0, dict(V=18428)), ("f32", 512, 3, 4, 1, dict(F=1088, V=18436)), ("f32", 512, 13, 1, 0, dict(F=1088, V=16388)),
    ("f32", 576, 2, 2, 1, dict(share="S")), ("f32", 768, 4, 1, 1, dict(F=2048, encdec_pi=[3])), ("f32", 768, 5, 1, 0, dict(F=3072)),
    ("f32", 1024, 1, 1, 0, dict(F=2048)), ("bf16", 256, 1, 4, 1, dict(V=18428)), ("bf16", 512, 2, 3, 1, dict(F=2048, V=18436)),
    ("bf16", 512, 7, 1, 0, dict(F=2048)), ("bf16", 1024, 1, 4, 1, dict(F=4096, self_pi=[1, 2], encdec_pi=[3])),
    ("bf16", 832, 2, 2, 1, dict(share="S")), ("bf16", 1024, 5, 1, 0, dict(F=4096)),
    ("bf16", 512, 3, 4, 0, dict(F=2048, self_kind="aan", self_pi=[1, 1, 1]))])
def test_few_rows_on_both_sides_of_the_rule(dtype, d, batch, beam, few, kw, loop):
    L, dt, rows = rules.lib(), 1 if dtype == "bf16" else 0, batch * beam
    if kw.get("self_kind") != "aan":
        assert L.few_rows(dt, rows, d) == few
    cfg = _cfg(dtype=dtype, d=d, H=d // 64, F=kw.get("F", 320), batch=batch, beam=beam, steps=3)
    cfg.update({k: v for k, v in kw.items() if k != "share"})
    ls = _lockstep(cfg, kw.get("share", "A"), loop)
    if loop is None:
        assert max(ls.log["logit_err"]) <= _tol(cfg), max(ls.log["logit_err"])
    ls.gpu.close()


# The two LayerNorms of an Eq. 5 follower in one launch, each with the k split of the product in front of it: a kernel for
# every pair that the products come with, one for the others (16, 4), by one wave (d <= 512) and by several.
@pytest.mark.parametrize("dtype,d,rows,block,splits", [
    ("f32", 64, 17, 2, (1, 1)), ("f32", 128, 17, 2, (2, 2)), ("f32", 256, 17, 2, (4, 4)), ("f32", 512, 17, 2, (8, 8)),
    ("f32", 512, 72, 4, (8, 4)), ("f32", 512, 130, 6, (8, 2)), ("f32", 512, 520, 4, (4, 1)), ("f32", 256, 520, 4, (4, 2)),
    ("bf16", 256, 520, 4, (2, 1)), ("bf16", 512, 17, 2, (4, 4)), ("f32", 576, 17, 2, (8, 8)), ("f32", 768, 17, 6, (8, 4)),
    ("bf16", 640, 17, 2, (4, 4)), ("bf16", 768, 72, 6, (4, 2)), ("f32", 1024, 72, 4, (8, 2)), ("f32", 1024, 17, 4, (16, 4))])
def test_layer_norms_over_split_products(dtype, d, rows, block, splits):
    _layer_norms(dtype, d, rows, block, splits, 64)


# F = 192: no one-workgroup decoder, the LayerNorms are launches.
@pytest.mark.parametrize("d,splits", [(64, (1, 1)), (128, (2, 2))])
def test_layer_norms_over_split_products_of_narrow_models(d, splits):
    assert _layer_norms("f32", d, 17, 2, splits, 192) > 10


def _layer_norms(dtype, d, rows, block, splits, F):
    dt = 1 if dtype == "bf16" else 0
    assert (rules.lib().pick_ksplit(rows, d, d, dt), rules.lib().pick_ksplit(rows, block * d, d, dt)) == splits
    cfg = _cfg(dtype=dtype, d=d, H=d // 64, F=F, V=260, batch=rows, n_dec=block, self_pi=[block], encdec_pi=[block], steps=2)
    w = wl.make_weights(cfg, seed=8, sharp=4.0)
    src, lens = wl.make_source(cfg, 8)
    gpu = hz.make_gpu(cfg, w)
    ls = hz.Lockstep(gpu, hz.make_oracle(cfg, w), src, lens, 1, subset=np.array([0, rows // 2, rows - 1]))
    for _ in range(cfg["steps"]):
        ls.step(logit_tol=_tol(cfg))
    assert max(ls.log["logit_err"]) <= _tol(cfg), max(ls.log["logit_err"])
    launches = gpu.last_launch_count
    gpu.close()
    return launches


# a wide vocabulary whose last column tile has 4 live columns, k = 192 (an odd number of chunk pairs) and 256; wm: tiles
# of 64 wm rows (100 rows of 128, 185 of 192, 256 two full tiles of 128, 300 two of 192, the second ragged).
# debug = 2: the fp32 instructions instead.
@pytest.mark.parametrize("loop", [None, "cands"])
@pytest.mark.parametrize("batch,beam,d,debug,wm", [(25, 4, 192, 0, 2), (32, 4, 256, 0, 2), (37, 5, 192, 0, 3), (64, 4, 192, 0, 2),
                                                   (300, 1, 192, 0, 3), (64, 4, 192, 2, 2)])
def test_large_fp32_products_match_oracle(batch, beam, d, debug, wm, loop):
    assert rules.lib().split_wm(batch * beam, 25604, d, 1, 1) == wm
    ls = _lockstep(_cfg(batch=batch, beam=beam, d=d, H=d // 64, V=25604, steps=2, n_dec=1, self_pi=[1], encdec_pi=[1]), loop=loop, debug=debug)
    if loop is None:
        assert max(ls.log["logit_err"]) <= F32_TOL, max(ls.log["logit_err"])
    ls.gpu.close()


def _logits_of(cfg, row, w_out, debug):
    """Logits of a one-step decode whose decoder output is `row` for every hypothesis: the last LayerNorm has gain 0
    and bias `row`."""
    w = wl.make_weights(cfg, seed=4)
    w["dec0.ln3.g"] = np.zeros_like(w["dec0.ln3.g"])
    w["dec0.ln3.b"] = row
    w["w_out"] = w_out
    src, lens = wl.make_source(cfg, 4)
    gpu = hz.make_gpu(cfg, w, debug=debug)
    logits = torch.empty((cfg["batch"], cfg["V"]), dtype=torch.float32, device="cuda")
    gpu.encode(torch.from_numpy(src).cuda(), torch.from_numpy(lens).cuda())
    gpu.decode_step(torch.full((cfg["batch"],), wl.BOS_ID, dtype=torch.int32, device="cuda"), logits)
    out = logits.cpu().numpy()
    gpu.close()
    return out


@pytest.mark.parametrize("batch", [128, 185])
@pytest.mark.parametrize("operands", ["normal", "spread", "relu", "one_live", "below_half_step", "signed_half_step"])
def test_split_products_are_no_further_from_64_bits(operands, batch):
    """fp32 products through bf16 parts against the fp32 instructions (debug = 2), both against 64 bits: rows of random
    values, of values spread over e^+-8, of non-negative ones (a ReLU's output), a single live value, and operands whose
    bf16 parts are as large as they get, with one sign and with random ones."""
    V, d = 32000, 512
    assert rules.lib().split_wm(batch, V, d, 1, 1) == (2 if batch == 128 else 3)
    rng = np.random.default_rng(11)
    row, w_out = rng.normal(size=d), 0.02 * rng.normal(size=(V, d))
    step = np.nextafter(np.float32(1.00390625), np.float32(0))          # 1 + 2^-8, less one unit of the 24th bit
    if operands == "spread":
        row, w_out = row * np.exp(rng.uniform(-8, 8, d)), w_out * np.exp(rng.uniform(-8, 8, (V, d)))
    elif operands == "relu":
        row = np.maximum(row, 0)
    elif operands == "one_live":
        row[np.arange(d) != 77] = 0
    elif operands == "below_half_step":
        row, w_out = np.full(d, step), np.full((V, d), step)
    elif operands == "signed_half_step":
        row, w_out = step * np.sign(row), step * np.sign(w_out)
    row, w_out = row.astype(np.float32), w_out.astype(np.float32)
    cfg = _cfg(batch=batch, d=d, H=8, F=64, V=V, n_dec=1, self_pi=[1], encdec_pi=[1])
    exact = w_out.astype(np.float64) @ row.astype(np.float64)
    err = []
    for debug in (0, 2):
        got = _logits_of(cfg, row, w_out, debug)
        assert np.array_equal(got, np.broadcast_to(got[0], got.shape))
        err.append(np.linalg.norm(got[0] - exact) / np.linalg.norm(exact))
    # 1 % for the two roundings of the last addition, where that is all there is
    assert err[0] <= 1.01 * err[1], err
    # one rounding of the running sum per 16 products, one for joining the two sums: sqrt(d / 16 + 1) of them at 2^-25
    # rms each add up like this when they are independent; 4 times that covers sums that are larger than the result
    assert err[0] <= 4 * np.sqrt(d / 16 + 1) * 2.0 ** -25, err


def test_infinite_weight_keeps_its_logits():
    """An infinite output weight makes its word's logits infinite with the sign of the activation it meets, as
    fp32 products do; split into bf16 parts it would make them NaN."""
    cfg = _cfg(batch=64, beam=4, d=192, H=3, V=25604, n_dec=1, self_pi=[1], encdec_pi=[1])
    w = wl.make_weights(cfg, seed=5)
    src, lens = wl.make_source(cfg, 5)
    tokens = torch.full((256,), wl.BOS_ID, dtype=torch.int32, device="cuda")
    rows = []
    for value in (1.0, np.inf):
        w["w_out"] = w["w_out"].copy()
        w["w_out"][7] = 0.0
        w["w_out"][7, 3] = value
        gpu = hz.make_gpu(cfg, w)
        logits = torch.empty((256, cfg["V"]), dtype=torch.float32, device="cuda")
        gpu.encode(torch.from_numpy(src).cuda(), torch.from_numpy(lens).cuda())
        gpu.decode_step(tokens, logits)
        rows.append(logits.cpu().numpy())
        gpu.close()
    x3 = rows[0][:, 7]
    assert np.array_equal(rows[1][:, 7], np.where(x3 > 0, np.inf, -np.inf).astype(np.float32))
    others = np.delete(np.arange(cfg["V"]), 7)
    assert np.allclose(rows[0][:, others], rows[1][:, others], rtol=0, atol=1e-4 * np.abs(rows[0][:, others]).max())


@pytest.mark.parametrize("value", [np.inf, -np.inf, 3.4e38, 1e6])
def test_activations_too_large_to_split(value):
    """A bias of the last LayerNorm that is infinite, rounds to infinity in bf16 or is merely large: the logits are what
    the fp32 instructions give, infinite with the weight's sign or finite."""
    cfg = _cfg(batch=256, d=192, H=3, V=25604, n_dec=1, self_pi=[1], encdec_pi=[1])
    assert rules.lib().split_wm(256, 25604, 192, 1, 1) > 0
    rng = np.random.default_rng(6)
    row, w_out = rng.normal(size=192).astype(np.float32), (1e-3 * rng.normal(size=(25604, 192))).astype(np.float32)
    row[5] = value
    got = _logits_of(cfg, row, w_out, 0)
    if np.isinf(value):
        assert np.array_equal(got, np.broadcast_to(np.sign(value) * np.sign(w_out[:, 5]) * np.float32(np.inf), got.shape))
    else:
        assert np.isfinite(got).all()
    assert np.array_equal(got, _logits_of(cfg, row, w_out, 2))


@pytest.mark.parametrize("dtype,batch,max_src,share,enc_pi,d,H", [("f32", 40, 61, "A", None, 128, 4), ("bf16", 33, 70, "S", None, 128, 4),
                                                                  ("f32", 20, 30, "A", [2, 1], 128, 4), ("f32", 1030, 5, "A", None, 128, 4),
                                                                  # few long streams: each is split over four waves
                                                                  ("f32", 6, 104, "A", None, 128, 4), ("bf16", 6, 104, "S", None, 128, 4),
                                                                  ("f32", 5, 130, "A", [2, 1], 128, 4),
                                                                  # rows wider than the LayerNorm of one wave takes
                                                                  ("f32", 18, 61, "A", None, 576, 9), ("bf16", 18, 61, "A", None, 640, 20),
                                                                  # a follower's value product of 610 padded rows and 427 without
                                                                  # padding: on both sides of gemm_lds_variant's line for k >= 1024
                                                                  ("bf16", 10, 61, "A", [2, 1], 1024, 32)])
def test_ragged_encoder_equals_the_padded_one(dtype, batch, max_src, share, enc_pi, d, H):
    """Lengths 0 .. max_src.  The rows of a product or a LayerNorm do not depend on each other, so leaving out the
    padding changes no bit (debug = 1 keeps the padded route); a few sentences are checked against the oracle."""
    cfg = _cfg(n_enc=3 if enc_pi else 2, n_dec=2, d=d, H=H, dtype=dtype, batch=batch, src_len=(1, max_src), steps=3, self_pi=[2],
               encdec_pi=[2])
    w = wl.make_weights(cfg, seed=9, sharp=4.0)
    src, lens = wl.make_source(cfg, 9)
    lens[0], lens[-1], lens[batch // 2] = 0, max_src, 1
    rng = np.random.default_rng(9)
    for b in range(batch):
        src[b] = wl.PAD_ID
        src[b, :lens[b]] = rng.integers(3, cfg["V"], lens[b])
    kw = dict(enc_pi=enc_pi) if enc_pi else {}
    got = []
    for debug in (0, 1):
        gpu = hz.make_gpu(cfg, w, share=share, debug=debug, **kw)
        # what an earlier batch without padding left behind has no part in it
        gpu.encode(torch.from_numpy(src % 50 + 3).cuda(), torch.full((batch,), max_src, dtype=torch.int32, device="cuda"))
        got.append(hz.gpu_free_run(gpu, src, lens, 1, cfg["steps"], keep_logits=True)["logits"])
        gpu.close()
    for t in range(cfg["steps"]):
        assert np.isfinite(got[0][t]).all()
        assert np.array_equal(got[0][t], got[1][t]), t
    gpu = hz.make_gpu(cfg, w, share=share, **kw)
    ls = hz.Lockstep(gpu, hz.make_oracle(cfg, w, share=share, **kw), src, lens, 1, subset=np.array([0, 1, batch // 2, batch - 1]))
    for _ in range(cfg["steps"]):
        ls.step(logit_tol=_tol(cfg))
    assert max(ls.log["logit_err"]) <= _tol(cfg)
    gpu.close()


def test_state_of_a_context_holds_no_encoder_scratch():
    """What the matrix-core kernels add to a bf16 context is the fragment-ordered memory of each enc-dec head (debug = 2
    keeps neither it nor the encoder's copy); what caching saves is not given back in partials."""
    cfg = _cfg(n_enc=1, n_dec=2, d=128, H=2, F=512, dtype="bf16", batch=40, src_len=(64, 64), self_pi=[2], encdec_pi=[1, 1])
    w = wl.make_weights(cfg, seed=2)
    size = {}
    for debug in (0, 2):
        gpu = hz.make_gpu(cfg, w, debug=debug)
        size[debug] = gpu.device_bytes(1)
        gpu.close()
    packed = 40 * 2 * (64 // 32) * 8192                     # sentences, heads, blocks of 32 positions
    assert size[0] - size[2] == 2 * packed
    cfg = _cfg(d=512, H=8, F=64, batch=64, src_len=(4, 4), steps=64, n_dec=1, self_pi=[1], encdec_pi=[1])
    gpu = hz.make_gpu(cfg, wl.make_weights(cfg, seed=2), use_cache=0)
    rows = 64 * 64
    # x, q k v, attention output, hidden rows (2 d at least), two partials, and less than a quarter of that for the rest
    # (scores: heads x (positions + source) per row)
    assert gpu.device_bytes(1) <= 1.25 * rows * 512 * 4 * (1 + 3 + 1 + 2 + 2 + 1) + rows * 8 * (64 + 4) * 4
    gpu.close()


@pytest.mark.parametrize("batch,max_src,lens,enc_pi", [(9, 140, (0, 1, 31, 32, 33, 63, 65, 129, 140), None),   # five key blocks: the loop
                                                       (16, 32, None, None),                       # one block, all sentences full
                                                       (9, 70, (70, 64, 33, 32, 1, 0, 69, 70, 5), [2, 1])])   # weights emitted
def test_bf16_encoder_attention_on_matrix_cores(batch, max_src, lens, enc_pi):
    cfg = _cfg(n_enc=3 if enc_pi else 2, n_dec=2, d=128, H=2, dtype="bf16", batch=batch, beam=2, src_len=(max_src, max_src), steps=3,
               self_pi=[2], encdec_pi=[2])
    w = wl.make_weights(cfg, seed=13, sharp=4.0)
    src, n = wl.make_source(cfg, 13)
    if lens is not None:
        n[:] = lens
        src[np.arange(max_src)[None, :] >= n[:, None]] = wl.PAD_ID
    kw = dict(enc_pi=enc_pi) if enc_pi else {}
    gpu = hz.make_gpu(cfg, w, **kw)
    ls = hz.Lockstep(gpu, hz.make_oracle(cfg, w, **kw), src, n, 2)
    for _ in range(cfg["steps"]):
        ls.step(logit_tol=BF16_TOL)
    assert max(ls.log["logit_err"]) <= BF16_TOL, max(ls.log["logit_err"])
    gpu.close()


@pytest.mark.parametrize("beam,k", [(8, 8), (9, 8), (12, 12), (17, 17), (20, 20), (32, 32), (32, 3), (5, 32), (25, 17)])
def test_wide_beam_step_orders_ties_by_index(beam, k):
    """Every row of a sentence holds the same coarse scores, so a row's words tie with each other and with the other
    rows': the picks are decided by (higher score, then lower beam * vocab + word), through the per-row stage and the
    per-sentence merge by one wave (up to 64 candidates) and by four."""
    _check_picks(2004, beam, k)


# The per-row threshold of more than 16 picks: fewer words than picks need lanes (124 of 128), groups of one lane's words,
# of several, of several registers (4100 on).  Rows of random scores, of nothing but ties, and in order of their scores
# (falling and rising), whose best words are neighbours.
@pytest.mark.parametrize("V", [36, 124, 128, 132, 1000, 2048, 4092, 4100, 8004])
@pytest.mark.parametrize("beam,k", [(17, 17), (20, 20), (32, 32), (3, 32)])
def test_wide_beam_thresholds(V, beam, k):
    _check_picks(V, beam, k)


def _check_picks(V, beam, k):
    batch = 5
    cfg = _cfg(batch=batch, beam=beam, V=V, n_dec=1, self_pi=[1], encdec_pi=[1])
    gpu = hz.make_gpu(cfg, wl.make_weights(cfg, seed=3))
    src, lens = wl.make_source(cfg, 3)
    gpu.encode(torch.from_numpy(src).cuda(), torch.from_numpy(lens).cuda())
    rng = np.random.default_rng(7)
    rows = np.round(rng.normal(size=(batch, V)) * 2) / 2
    rows[1] = 0.0                                    # nothing but ties
    rows[3], rows[4] = np.arange(V) / 64, -np.arange(V) / 64
    logits = torch.from_numpy(np.repeat(rows, beam, axis=0).astype(np.float32)).cuda()
    cum = torch.zeros(batch * beam, device="cuda")
    cum[2 * beam + beam // 2] = -np.inf              # a dead hypothesis
    o_tok, o_par = (torch.full((batch, k), -5, dtype=torch.int32, device="cuda") for _ in range(2))
    o_sc = torch.zeros((batch, k), device="cuda")
    gpu.topk(logits, cum, k, o_tok, o_par, o_sc)
    torch.cuda.synchronize()
    for b in range(batch):
        value = np.repeat(rows[b][None], beam, axis=0)
        if b == 2:
            value[beam // 2] = -np.inf
        flat = np.lexsort((np.arange(beam * V), -value.reshape(-1)))[:k]
        assert np.array_equal(o_tok[b].cpu().numpy(), flat % V), b
        assert np.array_equal(o_par[b].cpu().numpy(), b * beam + flat // V), b
    gpu.close()


@pytest.mark.parametrize("beam,steps,dtype", [(20, 70, "f32"), (32, 70, "f32"), (12, 129, "bf16"), (17, 66, "f32")])
def test_wide_beam_tail_permutes_long_histories(beam, steps, dtype):
    """san_decode_n with more than 64 past positions (the tail permutes 64 columns of the ancestry table at a time, the last
    pass ragged) against the three separate calls: the same words and parents at every step, the same scores."""
    V, batch = 212, 2
    cfg = _cfg(dtype=dtype, batch=batch, beam=beam, V=V, steps=steps, n_dec=2, self_pi=[1, 1], encdec_pi=[1, 1])
    w = wl.make_weights(cfg, seed=12, sharp=4.0)
    w["w_out"] = w["w_out"] * np.float32(8.0)
    if dtype == "bf16":
        w["w_out"] = wl.round_to_bf16(w["w_out"])
    src, lens = wl.make_source(cfg, 12)
    gpu = hz.make_gpu(cfg, w)
    ref = hz.gpu_free_run(gpu, src, lens, beam, steps)
    gpu.encode(torch.from_numpy(src).cuda(), torch.from_numpy(lens).cuda())
    rows = batch * beam
    cum = torch.full((rows,), -np.inf, device="cuda")
    cum[::beam] = 0.0
    tok, par = (torch.zeros((steps, rows), dtype=torch.int32, device="cuda") for _ in range(2))
    gpu.decode_n(steps, torch.full((rows,), wl.BOS_ID, dtype=torch.int32, device="cuda"), cum, tok, par,
                 torch.empty((rows, V), device="cuda"), keep_logits=True)
    assert np.array_equal(tok.cpu().numpy(), np.stack(ref["tokens"]))
    assert np.array_equal(par.cpu().numpy(), np.stack(ref["parents"]))
    assert np.array_equal(cum.cpu().numpy(), ref["scores"][-1].reshape(-1))
    moved = np.stack(ref["parents"])[64:] != np.arange(rows)
    assert moved.any()                                       # the permutation has something to do past 64 columns
    gpu.close()


# Small fp32 models, one workgroup per sentence: both widths, every feed-forward width and head width, beams on both sides
# of its row blocks and of its wave-per-part search, vocabularies that leave waves and lanes without words, histories too
# long for sixteen lanes a head, empty sources, both kinds of enc-dec sharing.
_SMALL = {
    "greedy": dict(batch=3),
    "words_fewer_than_waves": dict(V=68, batch=2, beam=2),
    "d64_heads16_beam8": dict(F=64, beam=8, batch=2),
    "d64_heads64_beam3": dict(H=1, F=256, beam=3, batch=2, share="S", encdec_pi=[3]),
    "d64_f512_beam5": dict(H=2, F=512, beam=5, batch=2, self_pi=[1, 2], V=2004),
    "d128_heads16_beam4": dict(d=128, H=8, F=128, beam=4, batch=3, src_len=(1, 40)),
    "d128_heads128_beam2": dict(d=128, H=1, F=512, beam=2, share="S"),
    "d128_heads32_beam6": dict(d=128, H=4, F=64, beam=6, self_pi=[3], encdec_pi=[1, 1, 1]),
    "many_sentences": dict(batch=260, n_dec=2, self_pi=[2], encdec_pi=[2], V=260, src_len=(0, 3)),
    "long_history": dict(beam=4, steps=262, V=260, F=64),
}


@pytest.mark.parametrize("loop", [None, "cands"])
@pytest.mark.parametrize("case", sorted(_SMALL))
def test_small_models_match_oracle(case, loop):
    cfg = _cfg(**_SMALL[case])
    share = cfg.pop("share", "A")
    assert rules.lib().small_model(cfg["d"], cfg["F"], cfg["V"], cfg["n_dec"], cfg["beam"], cfg["batch"])
    ls = _lockstep(cfg, share, loop)
    if loop is None:
        assert max(ls.log["logit_err"]) <= F32_TOL, max(ls.log["logit_err"])
        assert ls.gpu.last_launch_count == 1
    ls.gpu.close()


# Scores that overflow to -inf at every position give a zero context, as in the general attention kernels (debug = 2).
@pytest.mark.parametrize("beam", [1, 4])
@pytest.mark.parametrize("where", ["self", "ctx"])
def test_small_models_zero_context_where_no_score_is_finite(where, beam):
    cfg = _cfg(batch=2, beam=beam)
    w = wl.make_weights(cfg, seed=7)
    w[f"dec0.{where}.bq"] = np.full_like(w[f"dec0.{where}.bq"], 1e25)
    w[f"dec0.{where}.bk"] = np.full_like(w[f"dec0.{where}.bk"], -1e25)
    src, lens = wl.make_source(cfg, 7)
    got = []
    for debug in (0, 2):
        gpu = hz.make_gpu(cfg, w, debug=debug)
        gpu.encode(torch.from_numpy(src).cuda(), torch.from_numpy(lens).cuda())
        logits = torch.empty(2 * beam, cfg["V"], device="cuda")
        for word in (wl.BOS_ID, 5, 9):
            gpu.decode_step(torch.full((2 * beam,), word, dtype=torch.int32, device="cuda"), logits)
        assert (gpu.last_launch_count == 1) == (debug == 0)
        got.append(logits.cpu().numpy())
        gpu.close()
    assert np.isfinite(got[1]).all()
    assert hz.rel_err_rows(got[0], got[1].astype(np.float64)).max() <= F32_TOL


# Several steps inside one launch, with and without end symbols and the graph flag, then single steps on the state they leave,
# against the launches (debug = 2) on the same weights.  The seed's searches have no near ties: scores differ by
# the roundings of 32-bit sums (2e-5 of sums of up to 40 log-probabilities).  (21 steps: no sentence leaves the batch; see
# test_small_models_drop_finished_sentences.)
@pytest.mark.parametrize("eos,compact,beam,graph", [(-1, False, 4, True), (wl.EOS_ID, False, 4, False), (wl.EOS_ID, True, 4, True), (-1, False, 1, False)])
def test_small_models_loop_equals_the_launches(eos, compact, beam, graph):
    cfg = _cfg(batch=6, beam=beam, steps=44, V=260, src_len=(2, 9))
    assert rules.lib().small_model(cfg["d"], cfg["F"], cfg["V"], cfg["n_dec"], beam, cfg["batch"])
    w = wl.make_weights(cfg, seed=5, sharp=4.0)
    w["w_out"] = w["w_out"] * np.float32(20.0)
    if eos >= 0:
        w["w_out"][eos] *= np.float32(2.0)     # some sentences end early
    src, lens = wl.make_source(cfg, 5)
    rows, out = cfg["batch"] * beam, []
    with torch.cuda.stream(torch.cuda.Stream()):
        for debug in (0, 2):
            gpu = hz.make_gpu(cfg, w, eos_id=eos, debug=debug)
            gpu.encode(torch.from_numpy(src).cuda(), torch.from_numpy(lens).cuda())
            tok = torch.full((rows,), wl.BOS_ID, dtype=torch.int32, device="cuda")
            cum = torch.full((cfg["batch"], beam), -float("inf"), device="cuda")
            cum[:, 0] = 0.0
            cum = cum.reshape(-1).contiguous()
            toks = torch.zeros(40, rows, dtype=torch.int32, device="cuda")
            pars = torch.zeros_like(toks)
            logits = torch.empty(rows, cfg["V"], device="cuda")
            gpu.decode_n(21, tok, cum, toks, pars, logits, use_graph=graph, compact=compact)
            step, active = gpu.step, gpu.active()
            more = []
            if len(active) == cfg["batch"] and step == 21:
                t2, c2 = toks[20].clone(), cum.clone()
                gpu.decode_n(3, t2, c2, toks[21:], pars[21:], logits)
                gpu.decode_step(toks[23].clone(), logits)
                more = [c2.cpu().numpy(), logits.cpu().numpy()]
            out.append((step, list(active), toks.cpu().numpy(), pars.cpu().numpy(), cum.cpu().numpy(), *more))
            gpu.close()
    a, b = out
    assert a[0] == b[0] and a[1] == b[1] and len(a) == len(b)
    assert np.array_equal(a[2], b[2]) and np.array_equal(a[3], b[3])
    for x, y in zip(a[4:], b[4:]):
        fin = np.isfinite(y)
        assert np.array_equal(np.isfinite(x), fin) and np.abs(x[fin] - y[fin]).max() <= 2e-5 * np.abs(y[fin]).max()


# Sentences that leave the batch between two launches of several steps (row map, sentence index, caches wider than the batch,
# the loop's words and scores moved up), once and twice (seed 23), down to one sentence, against the oracle's search on the
# full batch.
@pytest.mark.parametrize("beam,eos_scale,seed,left", [(4, 1.6, 10, 6), (2, 2.5, 34, 1), (2, 2.5, 23, 2), (1, 2.0, 2, 3), (3, 2.0, 3, 2)])
def test_small_models_drop_finished_sentences(beam, eos_scale, seed, left):
    batch, T = 8, 40
    cfg = _cfg(batch=batch, beam=beam, V=132, steps=T, src_len=(2, 9))
    rows = batch * beam
    assert rules.lib().small_model(cfg["d"], cfg["F"], cfg["V"], cfg["n_dec"], beam, batch)
    w = wl.make_weights(cfg, seed=seed, sharp=4.0)
    w["w_out"] = w["w_out"] * np.float32(8.0)
    w["w_out"][wl.EOS_ID] *= np.float32(eos_scale)
    src, lens = wl.make_source(cfg, seed)
    ref = hz.make_oracle(cfg, w, eos_id=wl.EOS_ID).search(src, lens, T, beam)
    assert ref["margin"] > 2e-4 and hz.smallest_score_gap(ref, batch, beam) > 1e-4   # no near ties
    done = np.stack([(ref["tokens"][t].reshape(batch, beam) == wl.EOS_ID).all(axis=1) for t in range(T)])
    steps, active = _compaction_schedule(done, T)
    assert len(active) == left < batch
    with torch.cuda.stream(torch.cuda.Stream()):
        gpu = hz.make_gpu(cfg, w, eos_id=wl.EOS_ID, steps=T + 4)
        gpu.encode(torch.from_numpy(src).cuda(), torch.from_numpy(lens).cuda())
        logits = torch.empty((rows, cfg["V"]), device="cuda")
        for graph in (False, True):
            gpu.rewind()
            assert gpu.batch == batch
            toks, pars = (torch.full((T, rows), -7, dtype=torch.int32, device="cuda") for _ in range(2))
            cum = torch.full((batch, beam), -np.inf, device="cuda")
            cum[:, 0] = 0.0
            cum = cum.reshape(-1).contiguous()
            gpu.decode_n(T, torch.full((rows,), wl.BOS_ID, dtype=torch.int32, device="cuda"), cum, toks, pars, logits, use_graph=graph, compact=True)
            assert gpu.last_launch_count == 1 and gpu.step == steps and gpu.active().tolist() == active.tolist()
            got = [x.cpu().numpy() for x in (toks, pars, cum)]
            for t in range(steps):
                assert np.array_equal(got[0][t], ref["tokens"][t].reshape(-1)) and np.array_equal(got[1][t], ref["parents"][t].reshape(-1)), t
            assert (got[0][steps:] == -7).all() and (got[1][steps:] == -7).all()
            np.testing.assert_allclose(got[2], ref["scores"][steps - 1].reshape(-1), rtol=0, atol=1e-3)
        gpu.close()


# The same by san_compact between single steps and between calls of the loop.
@pytest.mark.parametrize("share,loop", [("A", None), ("S", None), ("A", "cands"), ("S", "cands")])
def test_small_models_go_on_after_compaction(share, loop):
    cfg = _cfg(batch=7, beam=3, V=260, steps=16, src_len=(0, 9), encdec_pi=[3])
    assert rules.lib().small_model(cfg["d"], cfg["F"], cfg["V"], cfg["n_dec"], 3, 7)
    w = wl.make_weights(cfg, seed=9, sharp=4.0)
    w["w_out"] = w["w_out"] * np.float32(8.0)
    src, lens = wl.make_source(cfg, 9)
    gpu = hz.make_gpu(cfg, w, share=share, max_batch=9)
    ls = hz.Lockstep(gpu, hz.make_oracle(cfg, w, share=share), src, lens, 3, subset=[2, 5], loop=loop)
    for t in range(14):
        if t == 5:
            hz.lockstep_compact(ls, [0, 2, 3, 5, 6])
        if t == 9:
            hz.lockstep_compact(ls, [1, 3])
            assert gpu.active().tolist() == [2, 5]
        ls.step(logit_tol=F32_TOL)
        assert gpu.last_launch_count == 1
    assert loop or max(ls.log["logit_err"]) <= F32_TOL, max(ls.log["logit_err"])
    gpu.close()


# Scores of all words and rows do not fit the LDS of a workgroup beside a long history: single steps run in one launch, the
# loop's search by the launches, on one state.
def test_small_models_whose_search_does_not_fit_the_lds():
    cfg = _cfg(batch=2, beam=8, F=64, V=4000, steps=12)
    assert rules.lib().small_model(64, 64, 4000, 3, 8, 2)
    w = wl.make_weights(cfg, seed=31, sharp=4.0)
    w["w_out"] = w["w_out"] * np.float32(8.0)
    src, lens = wl.make_source(cfg, 31)
    gpu = hz.make_gpu(cfg, w, steps=600)
    ls = hz.Lockstep(gpu, hz.make_oracle(cfg, w, max_len=600), src, lens, 8)
    for t in range(12):
        ls.loop = "cands" if t % 3 == 2 else None
        ls.step(logit_tol=F32_TOL)
        assert (gpu.last_launch_count == 1) == (ls.loop is None)
    assert max(ls.log["logit_err"]) <= F32_TOL, max(ls.log["logit_err"])
    gpu.close()


def test_small_models_count_the_launches_of_the_last_step():
    cfg = _cfg(batch=2, steps=12)
    w = wl.make_weights(cfg, seed=5)
    src, lens = wl.make_source(cfg, 5)
    gpu = hz.make_gpu(cfg, w)
    gpu.encode(torch.from_numpy(src).cuda(), torch.from_numpy(lens).cuda())
    tok, toks, pars = torch.full((2,), wl.BOS_ID, dtype=torch.int32, device="cuda"), *torch.zeros(2, 4, 2, dtype=torch.int32, device="cuda")
    logits = torch.empty(2, cfg["V"], device="cuda")
    for _ in range(2):
        gpu.decode_n(4, tok, torch.zeros(2, device="cuda"), toks, pars, logits)
        assert gpu.last_launch_count == 1
    gpu.decode_step(tok, logits)
    assert gpu.last_launch_count == 1
    gpu.profile(True)                                        # the general route
    gpu.decode_step(tok, logits)
    assert gpu.last_launch_count > 10
    gpu.close()


# The rule counts the positions that are read: a decode goes from one launch a step to the launches of the general route.
@pytest.mark.parametrize("loop", [None, "cands"])
@pytest.mark.parametrize("beam,H,src", [(8, 4, 420), (4, 1, 612)])
def test_small_models_hand_over_to_the_launches(beam, H, src, loop):
    cfg = _cfg(batch=3, beam=beam, H=H, F=64, V=260, src_len=(src // 2, src), steps=12)
    here = [rules.lib().small_model_at(64, 64, 260, 3, beam, 3, H, 5 * (t + 1) + 4 * src) for t in range(12)]
    assert here == [1] * 8 + [0] * 4
    w = wl.make_weights(cfg, seed=31, sharp=4.0)
    w["w_out"] = w["w_out"] * np.float32(8.0)
    src_ids, lens = wl.make_source(cfg, 31)
    gpu = hz.make_gpu(cfg, w)
    ls = hz.Lockstep(gpu, hz.make_oracle(cfg, w), src_ids, lens, beam, loop=loop)
    for one in here:
        ls.step(logit_tol=F32_TOL)
        assert loop or (gpu.last_launch_count == 1) == one
    assert loop or max(ls.log["logit_err"]) <= F32_TOL, max(ls.log["logit_err"])
    gpu.close()


# Sentences whose scores so far are -inf, or so large that they swallow a word's: all words of a row tie, and the words that
# count are the row's best ones, in the order of their numbers, as from the launches (debug = 2).
@pytest.mark.parametrize("dead", [-np.inf, -1e9, 1e9])
@pytest.mark.parametrize("beam,V", [(1, 1004), (2, 1004), (3, 260), (4, 1004), (5, 260), (8, 1004)])
def test_small_models_take_the_best_words_of_dead_rows(beam, V, dead):
    cfg = _cfg(batch=4, beam=beam, V=V)
    assert rules.lib().small_model(cfg["d"], cfg["F"], V, cfg["n_dec"], beam, cfg["batch"])
    w = wl.make_weights(cfg, seed=6, sharp=4.0)
    w["w_out"] = w["w_out"] * np.float32(20.0)
    src, lens = wl.make_source(cfg, 6)
    rows, got = cfg["batch"] * beam, []
    for debug in (0, 2):
        gpu = hz.make_gpu(cfg, w, debug=debug)
        gpu.encode(torch.from_numpy(src).cuda(), torch.from_numpy(lens).cuda())
        tok = torch.full((rows,), wl.BOS_ID, dtype=torch.int32, device="cuda")
        cum = torch.full((cfg["batch"], beam), dead, device="cuda")
        cum[0, 0] = cum[1, beam - 1] = 0.0     # two sentences with a live row, in one of them behind its dead rows
        cum = cum.reshape(-1).contiguous()
        toks = torch.zeros(3, rows, dtype=torch.int32, device="cuda")
        pars = torch.zeros_like(toks)
        gpu.decode_n(3, tok, cum, toks, pars, torch.empty(rows, V, device="cuda"))
        got.append([x.cpu().numpy() for x in (toks, pars)])
        gpu.close()
    assert np.array_equal(got[0][1], got[1][1]) and np.array_equal(got[0][0], got[1][0])


# The score so far leaves a word's score 2^-16 where the words' own differ by 4e-6: a row's best words are found before the
# scores are added, in whichever waves' parts of the vocabulary they lie, as in the launches (debug = 2).
@pytest.mark.parametrize("beam", [1, 2, 3, 4, 5])
def test_small_models_take_the_best_words_under_large_scores(beam):
    V, d, batch = 1004, 64, 16
    cfg = _cfg(batch=batch, beam=beam, V=V)
    assert rules.lib().small_model(d, cfg["F"], V, cfg["n_dec"], beam, batch)
    w = wl.make_weights(cfg, seed=4)
    last = f"dec{cfg['n_dec'] - 1}.ln3."
    w[last + "g"], w[last + "b"] = np.zeros(d, np.float32), np.full(d, 0.125, np.float32)
    w["w_out"] = np.full((V, d), 0.125, np.float32)               # logits of 1, exactly
    best = np.array([991, 740, 519, 401, 300])[:beam]             # the parts of other waves have words of lower numbers
    w["w_out"][best, 0] += 3.2e-5                                 # and of 1 + 4e-6
    src, lens = wl.make_source(cfg, 4)
    got = []
    for debug in (0, 2):
        gpu = hz.make_gpu(cfg, w, debug=debug)
        gpu.encode(torch.from_numpy(src).cuda(), torch.from_numpy(lens).cuda())
        cum = torch.full((batch, beam), -np.inf, device="cuda")
        cum[:, 0] = -255.0 + 7.3 * torch.arange(batch, device="cuda")   # ends at -145
        cum = cum.reshape(-1).contiguous()
        toks, pars = torch.zeros(2, 1, batch * beam, dtype=torch.int32, device="cuda")
        gpu.decode_n(1, torch.full((batch * beam,), wl.BOS_ID, dtype=torch.int32, device="cuda"), cum, toks, pars,
                     torch.empty(batch * beam, V, device="cuda"))
        assert (gpu.last_launch_count == 1) == (debug == 0)
        got.append(toks.cpu().numpy().reshape(batch, beam))
        gpu.close()
    assert np.array_equal(got[0], got[1])
    assert np.array_equal(np.sort(got[0], axis=1), np.tile(np.sort(best), (batch, 1)))


# bf16 products with their operands straight to LDS, every tile of them: (row counts, widths) whose products take it, rows and
# columns that do not fill the last tile, q/k/v segments, fp32 partials split or not, ragged encoders, candidates, vocabularies
# that end inside a tile.  Checked: a few sentences (a product's rows do not depend on each other), the last ones among them.
_LDS = {   # case: (variant, (M, N, K, kind, k split, ragged) of the product meant, configuration)
    "64x64": (1, (300, 512, 512, 0, 1, 0), dict(batch=300, d=512, H=8, F=512, src_len=(1, 2))),
    "64x64_four_stages": (2, (301, 3072, 1024, 0, 1, 0), dict(batch=301, d=1024, H=16, F=1088, src_len=(1, 2))),
    "128x64_split": (7, (301, 1024, 4096, 2, 4, 0), dict(batch=301, d=1024, H=16, F=4096, src_len=(1, 2))),
    "128x128_ragged": (3, (2440, 2048, 512, 0, 1, 1), dict(batch=40, d=512, H=8, F=2048, src_len=(1, 61))),
    "192x128_ragged": (4, (15250, 512, 512, 2, 1, 1), dict(batch=250, d=512, H=8, F=192, src_len=(1, 61), steps=1)),
    "256x256": (5, (9150, 2048, 512, 0, 1, 1), dict(batch=150, d=512, H=8, F=2048, src_len=(1, 61), steps=1)),
    "320x256": (6, (7930, 3072, 1024, 0, 1, 1), dict(batch=130, d=1024, H=16, F=128, src_len=(1, 61), steps=1)),
    "128x128_logits": (4, (185, 32004, 512, 1, 1, 0), dict(batch=185, d=512, H=8, V=32004, src_len=(1, 2))),
    "128x128_candidates": (3, (68, 32004, 512, 3, 1, 0), dict(batch=17, beam=4, d=512, H=8, V=32004)),
    "192x128_candidates": (4, (300, 32004, 512, 3, 1, 0), dict(batch=75, beam=4, d=512, H=8, V=32004, src_len=(1, 2))),
    "256x256_candidates": (5, (500, 32004, 512, 3, 1, 0), dict(batch=125, beam=4, d=512, H=8, V=32004, src_len=(1, 2))),
}


@pytest.mark.parametrize("case", sorted(_LDS))
def test_bf16_products_straight_to_lds_match_oracle(case):
    variant, product, kw = _LDS[case]
    assert rules.lib().lds_variant(*product) == variant
    cfg = _cfg(dtype="bf16", n_enc=1, n_dec=2, self_pi=[1, 1], encdec_pi=[2], steps=2, **{k: v for k, v in kw.items() if k != "steps"})
    cfg["steps"] = kw.get("steps", 2)
    w = wl.make_weights(cfg, seed=31, sharp=4.0)
    w["w_out"] = wl.round_to_bf16(w["w_out"] * np.float32(8.0))
    src, lens = wl.make_source(cfg, 31)
    n = cfg["batch"]
    gpu = hz.make_gpu(cfg, w)
    ls = hz.Lockstep(gpu, hz.make_oracle(cfg, w), src, lens, cfg["beam"], subset=np.unique([0, n // 3, n - 2, n - 1]),
                     loop="cands" if product[3] == 3 else None)
    for _ in range(cfg["steps"]):
        ls.step(logit_tol=BF16_TOL)
    if product[3] != 3:
        assert max(ls.log["logit_err"]) <= BF16_TOL, max(ls.log["logit_err"])
    gpu.close()


# The 64 x 64 tiles add up as gemm_kernel's groups of waves do: a row's logits in a batch of 300 (straight to LDS) and in a
# smaller one (gemm_kernel) of as many groups are the same bits.  Groups of 128 values of k, and of 64.
@pytest.mark.parametrize("d,V,few,variant,groups", [(512, 764, 16, 1, 4), (512, 2004, 256, 1, 2), (448, 1004, 256, 2, 2), (576, 764, 16, 2, 4),
                                                    (768, 764, 16, 2, 4), (1024, 2004, 256, 2, 2), (1088, 2004, 256, 2, 2)])
def test_bf16_products_straight_to_lds_add_up_like_gemm_kernel(d, V, few, variant, groups):
    L = rules.lib()
    assert L.lds_variant(300, V, d, 1, 1, 0) == variant and L.lds_variant(few, V, d, 1, 1, 0) == 0 and L.skinny(1, few, V, d, 1, 1) == 0
    assert L.k_groups(300, V, d, 1, 0) == L.k_groups(few, V, d, 1, 0) == groups
    rng = np.random.default_rng(5)
    row, w_out = (wl.round_to_bf16(x.astype(np.float32)) for x in (rng.normal(size=d), rng.normal(size=(V, d))))
    got = [_logits_of(_cfg(dtype="bf16", batch=n, d=d, H=d // 64, F=64, V=V, n_dec=1, self_pi=[1], encdec_pi=[1], src_len=(1, 2)), row, w_out, 0)
           for n in (few, 300)]
    assert np.array_equal(got[1], np.broadcast_to(got[0][0], got[1].shape)) and np.array_equal(got[0], got[1][:few])


# The logits may lie on any 4-byte boundary.
@pytest.mark.parametrize("rows", [40, 300])
def test_bf16_logits_on_a_4_byte_boundary(rows):
    cfg = _cfg(dtype="bf16", batch=rows, d=512, H=8, F=192, V=16004, src_len=(1, 2))
    w = wl.make_weights(cfg, seed=3)
    src, lens = wl.make_source(cfg, 3)
    gpu = hz.make_gpu(cfg, w)
    buf = torch.zeros(2, rows * cfg["V"] + 8, device="cuda")
    tok = torch.full((rows,), wl.BOS_ID, dtype=torch.int32, device="cuda")
    for i, off in enumerate((0, 1)):
        gpu.encode(torch.from_numpy(src).cuda(), torch.from_numpy(lens).cuda())
        gpu.decode_step(tok, buf[i, off:off + rows * cfg["V"]].view(rows, cfg["V"]))
    a, b = buf[0, :rows * cfg["V"]].cpu().numpy(), buf[1, 1:1 + rows * cfg["V"]].cpu().numpy()
    assert buf[1, 0] == 0 and (buf[1, 1 + rows * cfg["V"]:] == 0).all()
    assert np.abs(a - b).max() <= 1e-5 * np.abs(a).max()
    gpu.close()


# fp32 products with k dealt to the waves, every tile of them: rows and columns that do not fill the last tile, q/k/v
# segments, fp32 partials, one piece of 16 k-values per wave and many, ragged encoders (rows of 128 columns above).
_KWAVES = {   # case: (variant, (M, N, K, k split) of the product meant, configuration)
    "32x32_eight_waves": (1, (41, 2048, 512, 1), dict(batch=41, d=512, H=8, F=2048)),
    "32x32_one_piece": (1, (33, 576, 128, 1), dict(batch=33, d=192, H=3, F=128, V=576)),
    "64x32": (2, (185, 1536, 512, 1), dict(batch=185, d=512, H=8, F=512, src_len=(1, 2))),
    "64x64": (3, (185, 3072, 1024, 1), dict(batch=185, d=1024, H=16, F=64, src_len=(1, 2))),
    "32x32_four_waves": (4, (45, 192, 64, 1), dict(batch=45, d=64, H=4, F=192, beam=1, V=2004, n_dec=5, self_pi=[5], encdec_pi=[5])),
    "32x32_split": (4, (65, 512, 512, 8), dict(batch=13, beam=5, d=512, H=8, F=64)),
}


@pytest.mark.parametrize("case", sorted(_KWAVES))
def test_fp32_products_dealt_to_waves_match_oracle(case):
    variant, product, kw = _KWAVES[case]
    assert rules.lib().kwaves_variant(*product) == variant and rules.lib().split_wm(*product[:3], product[3], product[3]) == 0
    if product[3] > 1:
        assert rules.lib().pick_ksplit(*product[:3], 0) == product[3]
    ls = _lockstep(_cfg(steps=2, **kw))
    assert max(ls.log["logit_err"]) <= F32_TOL, max(ls.log["logit_err"])
    ls.gpu.close()


# The same in fp32.
def test_fp32_logits_on_a_4_byte_boundary():
    rows = 40
    cfg = _cfg(batch=rows, d=512, H=8, F=64)
    assert rules.lib().kwaves_variant(rows, cfg["V"], 512, 1) > 0
    w = wl.make_weights(cfg, seed=3)
    src, lens = wl.make_source(cfg, 3)
    gpu = hz.make_gpu(cfg, w)
    buf = torch.zeros(2, rows * cfg["V"] + 8, device="cuda")
    tok = torch.full((rows,), wl.BOS_ID, dtype=torch.int32, device="cuda")
    for i in (0, 1):
        gpu.encode(torch.from_numpy(src).cuda(), torch.from_numpy(lens).cuda())
        gpu.decode_step(tok, buf[i, i:i + rows * cfg["V"]].view(rows, cfg["V"]))
    a, b = buf[0, :rows * cfg["V"]].cpu().numpy(), buf[1, 1:1 + rows * cfg["V"]].cpu().numpy()
    assert buf[1, 0] == 0 and (buf[1, 1 + rows * cfg["V"]:] == 0).all()
    assert np.abs(a - b).max() <= 1e-5 * np.abs(a).max()
    gpu.close()


# Where the logits lie changes no bit of them, and no neighbour: output layers of every kernel, last column tiles with 4 live
# columns.
@pytest.mark.parametrize("dtype,rows,V", [("f32", 4, 1004), ("f32", 40, 1004), ("f32", 185, 25604), ("bf16", 40, 1004), ("bf16", 300, 1004),
                                          ("bf16", 256, 25604)])
def test_logits_do_not_depend_on_where_they_lie(dtype, rows, V):
    cfg = _cfg(dtype=dtype, batch=rows, d=512, H=8, F=64, V=V, src_len=(1, 2))
    w = wl.make_weights(cfg, seed=3)
    src, lens = wl.make_source(cfg, 3)
    gpu = hz.make_gpu(cfg, w)
    buf = torch.zeros(4, rows * V + 4, device="cuda")
    tok = torch.full((rows,), wl.BOS_ID, dtype=torch.int32, device="cuda")
    for i in range(4):
        gpu.encode(torch.from_numpy(src).cuda(), torch.from_numpy(lens).cuda())
        gpu.decode_step(tok, buf[i, i:i + rows * V].view(rows, V))
    got = buf.cpu().numpy()
    assert got[0, :rows * V].any()
    for i in range(4):
        assert np.array_equal(got[i, i:i + rows * V], got[0, :rows * V]), i
        assert not got[i, :i].any() and not got[i, i + rows * V:].any()
    gpu.close()


@pytest.mark.parametrize("operands", ["normal", "spread", "relu", "one_live", "below_half_step", "signed_half_step"])
def test_products_dealt_to_waves_are_no_further_from_64_bits(operands):
    """As test_split_products_are_no_further_from_64_bits."""
    V, d, batch = 1004, 512, 40
    assert rules.lib().kwaves_variant(batch, V, d, 1) == 1
    rng = np.random.default_rng(11)
    row, w_out = rng.normal(size=d), 0.02 * rng.normal(size=(V, d))
    step = np.nextafter(np.float32(1.00390625), np.float32(0))
    if operands == "spread":
        row, w_out = row * np.exp(rng.uniform(-8, 8, d)), w_out * np.exp(rng.uniform(-8, 8, (V, d)))
    elif operands == "relu":
        row = np.maximum(row, 0)
    elif operands == "one_live":
        row[np.arange(d) != 77] = 0
    elif operands == "below_half_step":
        row, w_out = np.full(d, step), np.full((V, d), step)
    elif operands == "signed_half_step":
        row, w_out = step * np.sign(row), step * np.sign(w_out)
    row, w_out = row.astype(np.float32), w_out.astype(np.float32)
    cfg = _cfg(batch=batch, d=d, H=8, F=64, V=V, n_dec=1, self_pi=[1], encdec_pi=[1])
    exact = w_out.astype(np.float64) @ row.astype(np.float64)
    err = []
    for debug in (0, 2):
        got = _logits_of(cfg, row, w_out, debug)
        assert np.array_equal(got, np.broadcast_to(got[0], got.shape))
        err.append(np.linalg.norm(got[0] - exact) / np.linalg.norm(exact))
    # 1 % for the roundings of the last additions; a sum per wave, joined in seven
    assert err[0] <= 1.01 * err[1], err
    assert err[0] <= 4 * np.sqrt(d / 16 + 8) * 2.0 ** -25, err
