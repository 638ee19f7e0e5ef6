"""GPU parity of ps_predict_load (fp32 models) against the fp64 oracle, through the C ABI."""
import dataclasses
import os

import numpy as np
import pytest

from oracle import predictor as op
from paper_2504_03702_amd import binding as ps
from paper_2504_03702_amd import workloads as wl
from tests.gpu_util import TOL_FP32, rel_err, run_predict

pytestmark = pytest.mark.gpu
TINY = wl.MODELS["tiny"]


def make(tmp_models, name, cfg=TINY, **kw):
    path = os.path.join(tmp_models, name)
    wl.write_model(path, cfg, wl.make_weights(cfg, seed=0, **kw))
    return ps.ps_model_load(path, 0), op.load_model(path)


def check_tokens(got_f, got_t, ref_t, d_max, tol_tokens=1):
    # the rounding decision is taken in the kernel's precision (fp32) on the kernel's own value
    assert np.array_equal(got_t, np.clip(np.rint(got_f.astype(np.float32)), 0, d_max).astype(np.int32))
    assert np.max(np.abs(got_t - ref_t)) <= tol_tokens


@pytest.mark.parametrize("seed,n_req", [(0, 16), (1, 1), (2, 7), (3, 300)])
def test_tiny_config(tmp_models, seed, n_req):
    print(f"predict fp32 tiny seed={seed} n_req={n_req}", flush=True)
    model, ref = make(tmp_models, "tiny_gpu.bin", ln_jitter=0.1 if seed else 0.0, bias_std=0.05 if seed else 0.0)
    batch = wl.make_prompts("tiny", seed, n_req=n_req)
    got_f, got_t, flags, _ = run_predict(model, batch)
    ref_f, ref_t = op.predict_load(ref, batch.token_ids, batch.offsets)
    assert flags == 0
    assert rel_err(got_f, ref_f).max() < TOL_FP32
    check_tokens(got_f, got_t, ref_t, TINY.d_max)
    assert n_req == 1 or np.ptp(ref_f) > 1.0


def test_padded_layout_equals_packed(tmp_models):
    model, ref = make(tmp_models, "tiny_gpu.bin")
    packed = wl.make_prompts("tiny", 5, n_req=9)
    padded = wl.pad_prompts(packed.valid_lengths(), packed.token_ids, pad_id=77)
    a_f, a_t, fa, _ = run_predict(model, packed)
    b_f, b_t, fb, _ = run_predict(model, padded)
    assert fa == 0 and fb == 0
    assert np.array_equal(a_f, b_f) and np.array_equal(a_t, b_t)       # same rows, same arithmetic
    ref_f, _ = op.predict_load(ref, padded.token_ids, padded.offsets, padded.lengths)
    assert rel_err(b_f, ref_f).max() < TOL_FP32


def test_learnable_prompts_and_odd_shapes(tmp_models):
    # M = 4 learnable prompt rows; 3 heads of size 20; widths that are no multiple of a tile
    cfg = wl.ModelConfig(layers=3, hidden=60, heads=3, ffn=100, vocab=500, max_pos=80, n_soft=4,
                         head_hidden=33, dtype=wl.DTYPE_FP32)
    model, ref = make(tmp_models, "odd_soft.bin", cfg=cfg, ln_jitter=0.1, bias_std=0.05)
    rng = np.random.default_rng(7)
    lengths = np.array([1, 76, 2, 33, 64, 5], np.int32)
    batch = wl.pack_prompts(lengths, rng.integers(0, cfg.vocab, int(lengths.sum())).astype(np.int32))
    got_f, got_t, flags, _ = run_predict(model, batch)
    ref_f, ref_t = op.predict_load(ref, batch.token_ids, batch.offsets)
    assert flags == 0
    assert rel_err(got_f, ref_f).max() < TOL_FP32
    check_tokens(got_f, got_t, ref_t, cfg.d_max)


def test_batch_order_invariance(tmp_models):
    model, _ = make(tmp_models, "tiny_gpu.bin")
    b = wl.make_prompts("tiny", 6, n_req=8)
    lengths = b.valid_lengths()
    chunks = [b.token_ids[b.offsets[r]:b.offsets[r + 1]] for r in range(8)]
    perm = np.array([5, 2, 7, 0, 3, 6, 1, 4])
    pb = wl.pack_prompts(lengths[perm], np.concatenate([chunks[r] for r in perm]))
    a_f, _, _, _ = run_predict(model, b)
    p_f, _, _, _ = run_predict(model, pb)
    assert np.array_equal(p_f, a_f[perm])


def test_faulty_requests_are_isolated(tmp_models):
    model, ref = make(tmp_models, "tiny_gpu.bin")
    b = wl.make_prompts("tiny", 8, n_req=6)
    good_f, good_t, _, _ = run_predict(model, b)
    ids = b.token_ids.copy()
    ids[b.offsets[2] + 3] = TINY.vocab            # request 2: token id out of range
    ids[b.offsets[4]] = -1                        # request 4: negative id
    bad = dataclasses.replace(b, token_ids=ids)
    f, t, flags, first = run_predict(model, bad)
    assert flags == ps.PS_ST_BAD_TOKEN and first == 2
    assert np.isnan(f[[2, 4]]).all() and (t[[2, 4]] == -1).all()
    keep = [0, 1, 3, 5]
    assert np.array_equal(f[keep], good_f[keep]) and np.array_equal(t[keep], good_t[keep])
    with pytest.raises(op.OracleError):
        op.predict_load(ref, ids, b.offsets)
    # lengths: zero, longer than the span, longer than the position table
    padded = wl.pad_prompts(b.valid_lengths(), b.token_ids)
    lens = padded.lengths.copy()
    lens[1] = 0
    lens[3] = int(np.diff(padded.offsets)[3]) + 1
    f, t, flags, first = run_predict(model, dataclasses.replace(padded, lengths=lens))
    assert flags == ps.PS_ST_BAD_LENGTH and first == 1
    assert np.isnan(f[[1, 3]]).all() and (t[[1, 3]] == -1).all()
    assert np.array_equal(f[[0, 2, 4, 5]], good_f[[0, 2, 4, 5]])
    long_ids = np.zeros(TINY.max_pos + 1, np.int32)
    f, t, flags, _ = run_predict(model, wl.pack_prompts(np.array([TINY.max_pos + 1]), long_ids))
    assert flags == ps.PS_ST_BAD_LENGTH and np.isnan(f[0]) and t[0] == -1


def test_wrong_offsets_are_rejected_on_the_device(tmp_models):
    """Offsets are device data: spans that leave the token array, run backwards or overlap so that
    together they ask for more rows than the workspace was sized for are flagged, their requests get
    NaN / -1, and nothing is read or written out of bounds.  All buffers have the sizes the call states."""
    model, _ = make(tmp_models, "tiny_gpu.bin")
    b = wl.make_prompts("tiny", 8, n_req=6)
    good_f, good_t, _, _ = run_predict(model, b)
    n_tok = int(b.offsets[-1])
    # request 1 starts before the array, request 4 ends after it
    offs = b.offsets.copy()
    offs[1] = -3
    f, t, flags, first = run_predict(model, dataclasses.replace(b, offsets=offs))
    assert flags == ps.PS_ST_BAD_LENGTH and first == 0        # span 0 ends at -3 < its start
    assert np.isnan(f[[0, 1]]).all() and (t[[0, 1]] == -1).all()
    assert np.array_equal(f[2:], good_f[2:])
    offs = b.offsets.copy()
    offs[5] = n_tok + 40                                       # request 4 runs past the end, request 5 starts there
    f, t, flags, first = run_predict(model, dataclasses.replace(b, offsets=offs))
    assert flags == ps.PS_ST_BAD_LENGTH and first == 4
    assert np.isnan(f[[4, 5]]).all() and np.array_equal(f[:4], good_f[:4])
    # offsets 0, span, 0, span, ...: every even request claims the same valid span [0, span), every odd one runs
    # backwards.  Each even request is valid on its own; together they need several times the rows the host
    # planned for from the size of the token array
    import torch
    span = min(TINY.max_pos, n_tok)
    n_req = 40
    offs = np.tile(np.array([0, span], np.int32), n_req)[: n_req + 1].copy()
    dev = "cuda:0"
    ids = torch.from_numpy(b.token_ids).to(dev)
    pf = torch.full((n_req,), 5.0, dtype=torch.float32, device=dev)
    pt = torch.full((n_req,), -7, dtype=torch.int32, device=dev)
    ws = ps.alloc_workspace(ps.ps_workspace_bytes(model, n_tok, n_req), dev)
    st = ps.new_status(dev)
    ps.ps_predict_load(model, ids, torch.from_numpy(offs).to(dev), None, pf, pt, ws, st)
    flags, first = ps.ps_status_read(st)
    f, t = pf.cpu().numpy(), pt.cpu().numpy()
    assert flags == ps.PS_ST_BAD_LENGTH and first == 1
    assert np.isnan(f[1::2]).all() and (t[1::2] == -1).all()
    even = f[0::2]
    n_ok = int(np.sum(~np.isnan(even)))
    assert 1 <= n_ok < even.size and not np.isnan(even[:n_ok]).any() and np.isnan(even[n_ok:]).all()
    assert np.all(even[:n_ok] == even[0])                      # the same prompt every time
    assert (t[0::2][n_ok:] == -1).all()


def test_host_side_argument_errors(tmp_models):
    import torch
    model, _ = make(tmp_models, "tiny_gpu.bin")
    b = wl.make_prompts("tiny", 0, n_req=4)
    dev = "cuda:0"
    ids = torch.from_numpy(b.token_ids).to(dev)
    offs = torch.from_numpy(b.offsets).to(dev)
    pf = torch.empty(4, dtype=torch.float32, device=dev)
    pt = torch.empty(4, dtype=torch.int32, device=dev)
    with pytest.raises(ps.PsError) as e:
        ps.ps_predict_load(model, ids, offs, None, pf, pt, ps.alloc_workspace(256, dev))
    assert e.value.code == -5
    assert ps.ps_workspace_bytes(model, -1, 4) == 0
    info = model.info
    assert (info.layers, info.hidden, info.heads, info.ffn, info.vocab, info.dtype) == (2, 128, 2, 512, 8192, 0)


@pytest.mark.parametrize("hidden,heads,ffn,n", [(8, 1, 8, 3), (24, 2, 40, 5), (96, 3, 32, 40), (32, 4, 264, 600), (65, 5, 33, 20), (66, 3, 70, 300), (33, 3, 36, 7),
                                                (5, 1, 3, 9)])
def test_matrix_tiles_at_their_edges(tmp_models, hidden, heads, ffn, n):
    """Contractions of fewer groups of eight than wavefronts, columns that do not fill a tile of 32, rows enough for the
    64-row tiles."""
    cfg = wl.ModelConfig(layers=2, hidden=hidden, heads=heads, ffn=ffn, vocab=300, max_pos=70, head_hidden=17, dtype=wl.DTYPE_FP32)
    print(f"predict fp32 hidden={hidden} ffn={ffn} n={n}", flush=True)
    model, ref = make(tmp_models, f"edges_{hidden}.bin", cfg=cfg, ln_jitter=0.1, bias_std=0.05)
    rng = np.random.default_rng(hidden)
    lengths = rng.integers(1, 65, n).astype(np.int32)
    batch = wl.pack_prompts(lengths, rng.integers(0, cfg.vocab, int(lengths.sum())).astype(np.int32))
    got_f, got_t, flags, _ = run_predict(model, batch)
    ref_f, ref_t = op.predict_load(ref, batch.token_ids, batch.offsets)
    assert flags == 0
    assert rel_err(got_f, ref_f).max() < TOL_FP32
    check_tokens(got_f, got_t, ref_t, cfg.d_max)


@pytest.mark.parametrize("hidden,heads", [(33, 1), (70, 2), (111, 3), (130, 2), (198, 3), (64, 2)])
@pytest.mark.parametrize("n", [2, 150])
def test_head_sizes_off_the_attention_loads(tmp_models, hidden, heads, n):
    """Head sizes above 32 that are no multiple of 4 (keys are read 16 bytes a load, of which all but one row of a head
    then start off a 16-byte boundary) and one that is, with one row and with four rows a wavefront."""
    cfg = wl.ModelConfig(layers=2, hidden=hidden, heads=heads, ffn=48, vocab=300, max_pos=133, head_hidden=17, dtype=wl.DTYPE_FP32)
    print(f"predict fp32 head size {hidden // heads} n={n}", flush=True)
    model, ref = make(tmp_models, f"heads_{hidden}.bin", cfg=cfg, ln_jitter=0.1, bias_std=0.05)
    rng = np.random.default_rng(hidden + n)
    lengths = rng.integers(1, 134, n).astype(np.int32)
    lengths[-1] = 133
    batch = wl.pack_prompts(lengths, rng.integers(0, cfg.vocab, int(lengths.sum())).astype(np.int32))
    got_f, got_t, flags, _ = run_predict(model, batch)
    ref_f, ref_t = op.predict_load(ref, batch.token_ids, batch.offsets)
    assert flags == 0
    assert rel_err(got_f, ref_f).max() < TOL_FP32
    check_tokens(got_f, got_t, ref_t, cfg.d_max)


@pytest.mark.parametrize("hidden,heads", [(8, 2), (64, 1), (128, 2), (136, 2), (200, 2), (124, 1)])
@pytest.mark.parametrize("n", [2, 25, 70])
def test_heads_of_whole_groups(tmp_models, hidden, heads, n):
    """Head sizes that are multiples of 4, below, at and above 64 features, the last too large for keys and values through LDS;
    requests of one tile, of exactly 64 and 128 positions and of three tiles.  With two heads the calls of 2, 25 and
    70 requests take the forms with one and two rows a wavefront through LDS and the one without, with one head of 64 the first
    two only (see attention_form)."""
    cfg = wl.ModelConfig(layers=2, hidden=hidden, heads=heads, ffn=48, vocab=300, max_pos=133, head_hidden=17, dtype=wl.DTYPE_FP32)
    print(f"predict fp32 whole groups {hidden // heads} n={n}", flush=True)
    model, ref = make(tmp_models, f"groups_{hidden}_{heads}.bin", cfg=cfg, ln_jitter=0.1, bias_std=0.05)
    rng = np.random.default_rng(hidden + n)
    lengths = rng.integers(1, 134, n).astype(np.int32)
    lengths[:2] = 133, 64
    lengths[2:6] = np.array([128, 65, 129, 1], np.int32)[:max(n - 2, 0)]
    form = attention_form(hidden // heads, heads, cfg.max_pos, int(lengths.sum()), n)
    assert form == (0 if hidden == 124 else {2: 1, 25: 2, 70: 0}[n] if heads == 2 else {2: 1, 25: 1, 70: 2}[n])
    batch = wl.pack_prompts(lengths, rng.integers(0, cfg.vocab, int(lengths.sum())).astype(np.int32))
    got_f, got_t, flags, _ = run_predict(model, batch)
    ref_f, ref_t = op.predict_load(ref, batch.token_ids, batch.offsets)
    assert flags == 0
    assert rel_err(got_f, ref_f).max() < TOL_FP32
    check_tokens(got_f, got_t, ref_t, cfg.d_max)


def attention_form(d, heads, max_pos, tokens, n):
    """The form that the encoder's rule takes: 1 or 2 rows a wavefront with keys and values through LDS, 0 without LDS."""
    row_heads = -(-(tokens + 7 * n + 64) // 256) * 256 * heads
    lds = lambda rows: 4 * (64 * (2 * d + 4) + 4 * rows * (d + -(-max_pos // 4) * 4))
    rows = 2 if row_heads >= 3072 else 1
    if d % 4 or lds(2) > 65536 or row_heads >= 8192 or (d >= 64 and row_heads // (4 * rows) > 256 * (160 * 1024 // lds(rows))):
        return 0
    return rows


@pytest.mark.parametrize("hidden,heads,max_pos", [(8, 2, 133), (96, 2, 133), (64, 1, 133), (128, 2, 133), (136, 2, 133),
                                                  (100, 1, 133), (64, 1, 640)])
def test_attention_forms_bit_equal(tmp_models, hidden, heads, max_pos):
    """The same requests by themselves, among so many that two rows go to a wavefront (more than 64, so that a row's request is
    searched for) and among so many that nothing goes through LDS: the sums are in one order, so the bits are the same."""
    d = hidden // heads
    cfg = wl.ModelConfig(layers=2, hidden=hidden, heads=heads, ffn=48, vocab=300, max_pos=max_pos, head_hidden=17, dtype=wl.DTYPE_FP32)
    print(f"predict fp32 attention forms {d} features, {max_pos} positions", flush=True)
    model, ref = make(tmp_models, f"forms_{hidden}_{heads}_{max_pos}.bin", cfg=cfg, ln_jitter=0.1, bias_std=0.05)
    rng = np.random.default_rng(hidden + max_pos)
    lengths = np.full(3000, 21, np.int32)
    lengths[:6] = max_pos, 64, 128, 65, 129, 1
    lengths[6:40] = rng.integers(1, 20, 34)
    ids = rng.integers(0, cfg.vocab, int(lengths.sum())).astype(np.int32)
    got, forms = [], []
    for n in ((40, 120, 1200) if heads == 1 else (6, 70, 1200)):
        tokens = int(lengths[:n].sum())
        forms.append(attention_form(d, heads, max_pos, tokens, n))
        f, _, flags, _ = run_predict(model, wl.pack_prompts(lengths[:n], ids[:tokens]))
        assert flags == 0
        got.append(f)
    assert forms == [1, 2, 0]
    assert np.array_equal(got[0], got[2][:len(got[0])]) and np.array_equal(got[1], got[2][:len(got[1])])
    ref_f, _ = op.predict_load(ref, ids[:int(lengths[:40].sum())], np.concatenate([[0], np.cumsum(lengths[:40])]))
    assert rel_err(got[1][:40], ref_f).max() < TOL_FP32


def test_more_feed_forward_units_than_a_grid_has_tiles(tmp_models):
    """2097152 + 100 feed-forward units: more tiles of 32 columns than one launch may have in a dimension."""
    cfg = wl.ModelConfig(layers=1, hidden=2, heads=1, ffn=2097152 + 100, vocab=10, max_pos=8, head_hidden=3, dtype=wl.DTYPE_FP32)
    model, ref = make(tmp_models, "wide.bin", cfg=cfg, ln_jitter=0.1, bias_std=0.05)
    batch = wl.pack_prompts(np.array([3, 1], np.int32), np.array([1, 9, 4, 7], np.int32))
    got_f, got_t, flags, _ = run_predict(model, batch)
    ref_f, ref_t = op.predict_load(ref, batch.token_ids, batch.offsets)
    assert flags == 0
    assert rel_err(got_f, ref_f).max() < TOL_FP32
    check_tokens(got_f, got_t, ref_t, cfg.d_max)


@pytest.mark.parametrize("hidden,heads,ffn", [(32, 1, 32), (96, 3, 160), (128, 2, 512), (224, 7, 96), (256, 4, 1024),
                                              (256, 4, 100), (288, 4, 64)])
def test_maps_that_take_the_layer_norms(tmp_models, hidden, heads, ffn):
    """Narrow models in calls of few rows, where the maps make the LayerNorms of their operands and residuals themselves, on
    both sides of that rule (rows, widths): against the oracle, and the same requests in calls of other sizes to the bit."""
    cfg = wl.ModelConfig(layers=2, hidden=hidden, heads=heads, ffn=ffn, vocab=500, max_pos=80, n_soft=0, head_hidden=48,
                         dtype=wl.DTYPE_FP32)
    model, ref = make(tmp_models, f"norms{hidden}_{ffn}.bin", cfg=cfg, ln_jitter=0.1, bias_std=0.05)
    rng = np.random.default_rng(hidden + ffn)
    lengths = rng.integers(1, 81, 150).astype(np.int32)
    batch = wl.pack_prompts(lengths, rng.integers(0, cfg.vocab, int(lengths.sum())).astype(np.int32))
    got_f, got_t, flags, _ = run_predict(model, batch)
    ref_f, ref_t = op.predict_load(ref, batch.token_ids, batch.offsets)
    assert flags == 0 and rel_err(got_f, ref_f).max() < TOL_FP32
    check_tokens(got_f, got_t, ref_t, cfg.d_max)
    for n in (1, 3, 30):
        part = wl.pack_prompts(lengths[:n], batch.token_ids[: int(batch.offsets[n])])
        f, _, flags, _ = run_predict(model, part)
        assert flags == 0 and np.array_equal(f, got_f[:n]), n
