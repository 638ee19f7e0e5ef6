"""Calls of few requests or few rows: 64 x 64 tiles with the per-request maps in the same launches.  Their
accumulation order is that of the large tiles, so the same requests in a layout with many padding slots (which
takes the large tiles) must give the same bits; the fp64 oracle bounds both."""
import dataclasses

import numpy as np
import pytest

from paper_2504_03702_amd import workloads as wl
from tests.gpu_util import run_predict
from tests.test_gpu_predictor_bf16 import SMALL, check, chunks_bit_equal, make

pytestmark = pytest.mark.gpu

WIDE = wl.ModelConfig(layers=3, hidden=768, heads=12, ffn=1024, vocab=1000, max_pos=640, dtype=wl.DTYPE_BF16)


def padded_to(batch, slots):
    """The packed batch with every request padded to `slots` token slots."""
    lengths = batch.valid_lengths()
    ids = np.full((batch.n_req, slots), 3, np.int32)
    for r in range(batch.n_req):
        ids[r, :lengths[r]] = batch.token_ids[batch.offsets[r]:batch.offsets[r + 1]]
    offsets = (np.arange(batch.n_req + 1) * slots).astype(np.int32)
    return wl.PromptBatch(ids.reshape(-1), offsets, lengths.astype(np.int32))


@pytest.mark.parametrize("cfg", [SMALL, WIDE], ids=["hidden256", "hidden768"])
@pytest.mark.parametrize("lengths", [
    [1], [56], [57], [63, 64, 65], [300, 5, 128],       # one tile, tile edges, several row tiles
    [9] * 15, [70] * 16, [70] * 17, [3] * 200,           # the request counts at which the per-request maps change
], ids=lambda v: f"{len(v)}x{v[0]}")
def test_few_rows_equal_many(tmp_models, cfg, lengths):
    print(f"predict small call hidden={cfg.hidden} lengths={lengths[:4]} n={len(lengths)}", flush=True)
    model, ref = make(tmp_models, f"small_calls_{cfg.hidden}.bin", cfg, ln_jitter=0.1, bias_std=0.05)
    lengths = np.array(lengths, np.int32)
    ids = np.random.default_rng(7).integers(0, cfg.vocab, int(lengths.sum())).astype(np.int32)
    batch = wl.pack_prompts(lengths, ids)
    got = check(model, ref, batch)
    far, _, flags, _ = run_predict(model, padded_to(batch, max(640, 8192 // len(lengths))))
    assert flags == 0 and np.array_equal(got, far)


def test_faulty_request_leaves_the_others(tmp_models):
    """A request too long for the model and one with a token outside the vocabulary, in a call of five."""
    model, _ = make(tmp_models, "small_calls_256.bin", SMALL, ln_jitter=0.1, bias_std=0.05)
    lengths = np.array([20, 700, 64, 33, 90], np.int32)
    ids = np.random.default_rng(9).integers(0, SMALL.vocab, int(lengths.sum())).astype(np.int32)
    good = np.array([0, 2, 4])
    batch = wl.pack_prompts(lengths, ids)
    clean = wl.pack_prompts(lengths[good], np.concatenate([ids[batch.offsets[r]:batch.offsets[r + 1]] for r in good]))
    batch.token_ids[batch.offsets[3] + 5] = SMALL.vocab
    got, tokens, flags, bad = run_predict(model, batch)
    want, _, _, _ = run_predict(model, clean)
    assert flags != 0 and bad == 1
    assert np.isnan(got[[1, 3]]).all() and (tokens[[1, 3]] == -1).all()
    assert np.array_equal(got[good], want)


@pytest.mark.parametrize("head_hidden", [1, 63, 64, 65, 129, 2048, 2100])
def test_head_rounds(tmp_models, head_hidden):
    """Hidden units of the head around its rounds of 64 and beyond the 32 rounds that are kept apart: a request's value
    must not depend on how many workgroups share it (one at 256 requests, several below 129)."""
    print(f"predict head_hidden={head_hidden}", flush=True)
    cfg = dataclasses.replace(SMALL, layers=1, head_hidden=head_hidden)
    model, ref = make(tmp_models, f"head_{head_hidden}.bin", cfg, ln_jitter=0.1, bias_std=0.05)
    lengths = np.random.default_rng(3).integers(1, 20, 256).astype(np.int32)
    ids = np.random.default_rng(4).integers(0, cfg.vocab, int(lengths.sum())).astype(np.int32)
    batch = wl.pack_prompts(lengths, ids)
    got = check(model, ref, batch)
    few = wl.pack_prompts(lengths[:17], ids[:batch.offsets[17]])
    assert np.array_equal(check(model, ref, few), got[:17])


@pytest.mark.parametrize("n_req", [1024, 1025, 1281, 2100])
def test_many_requests_take_large_tiles(tmp_models, n_req):
    """4096 feed-forward units: above 1024 requests the per-request map goes to the large kernel's 128 x 128 tiles.  The
    requests' bits must be those of calls of 500, and the oracle bounds them."""
    print(f"predict many requests n={n_req}", flush=True)
    cfg = dataclasses.replace(SMALL, ffn=4096)
    model, ref = make(tmp_models, "many_requests.bin", cfg, ln_jitter=0.1, bias_std=0.05)
    rng = np.random.default_rng(n_req)
    lengths = rng.integers(1, 6, n_req).astype(np.int32)
    batch = wl.pack_prompts(lengths, rng.integers(0, cfg.vocab, int(lengths.sum())).astype(np.int32))
    check(model, ref, batch)
    got, tokens, flags, _ = run_predict(model, batch)
    assert flags == 0
    chunks_bit_equal(model, batch, got, tokens, chunk=500)
