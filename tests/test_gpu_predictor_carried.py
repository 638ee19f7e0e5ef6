"""Calls whose large maps carry the per-request ones: rows that the two write stand at every place of a tile, requests without
rows are nobody's, and the bits are those of calls that take other launches."""
import numpy as np
import pytest

from paper_2504_03702_amd import binding as ps
from paper_2504_03702_amd import workloads as wl
from tests.gpu_util import run_predict
from tests.test_gpu_predictor_bf16 import SMALL, check, make
from tests.test_gpu_predictor_small_calls import WIDE, padded_to

pytestmark = pytest.mark.gpu


def batch_of(lengths, vocab, seed=3):
    lengths = np.array(lengths, np.int32)
    ids = np.random.default_rng(seed).integers(0, vocab, int(lengths.sum())).astype(np.int32)
    return wl.pack_prompts(lengths, ids)


@pytest.mark.parametrize("cfg", [SMALL, WIDE], ids=["hidden256", "hidden768"])
@pytest.mark.parametrize("lengths", [
    [1] * 17, [8] * 32, [64] * 33, [8, 56, 64, 120, 128, 224, 256] * 5, [3] * 65 + [600], [250] * 40, [600] * 90,
], ids=lambda v: f"{len(v)}x{v[0]}")
def test_many_requests(tmp_models, cfg, lengths):
    print(f"predict carried hidden={cfg.hidden} n={len(lengths)}", flush=True)
    model, ref = make(tmp_models, f"carried_{cfg.hidden}.bin", cfg, ln_jitter=0.1, bias_std=0.05)
    longest = cfg.max_pos
    lengths = [min(n, longest) for n in lengths]
    batch = batch_of(lengths, cfg.vocab)
    few = batch if len(lengths) < 60 else None
    got = check(model, ref, few) if few is not None else run_predict(model, batch)[0]
    # the same requests ahead of 1100 others: launches of their own for the per-request maps
    rest = batch_of(lengths + [2] * 1100, cfg.vocab)
    rest.token_ids[: batch.token_ids.size] = batch.token_ids
    far, _, flags, _ = run_predict(model, rest)
    assert flags == 0 and np.array_equal(got, far[: len(lengths)])


@pytest.mark.parametrize("cfg", [SMALL, WIDE], ids=["hidden256", "hidden768"])
@pytest.mark.parametrize("n,slots", [(1, 640), (5, 640), (7, 600), (9, 640), (16, 640), (16, 300), (13, 288)])
def test_few_requests_of_many_rows(tmp_models, cfg, n, slots):
    print(f"predict carried few hidden={cfg.hidden} n={n} slots={slots}", flush=True)
    model, ref = make(tmp_models, f"carried_{cfg.hidden}.bin", cfg, ln_jitter=0.1, bias_std=0.05)
    rng = np.random.default_rng(n + slots)
    longest = min(slots, cfg.max_pos)
    lengths = rng.integers(1, longest + 1, n)
    lengths[0] = longest
    batch = batch_of(lengths, cfg.vocab, seed=n)
    got = check(model, ref, batch)
    far, _, flags, _ = run_predict(model, padded_to(batch, max(slots, longest)))
    assert flags == 0 and np.array_equal(got, far)
    wide, _, flags, _ = run_predict(model, padded_to(batch, 24000 // n))      # rows for any route
    assert flags == 0 and np.array_equal(got, wide)


def test_few_requests_of_the_widest_model(tmp_models):
    """Hidden 2048, whose lines between small and large tiles lie lower: 1280 packed rows (small), 1792, and eight padded requests
    in 512 slots (large) give each request the same bits."""
    cfg = wl.ModelConfig(layers=2, hidden=2048, heads=32, ffn=2048, vocab=500, max_pos=640, dtype=wl.DTYPE_BF16)
    print("predict carried few hidden=2048", flush=True)
    model, _ = make(tmp_models, "carried_2048.bin", cfg, ln_jitter=0.1, bias_std=0.05)
    lengths = [130, 1, 64, 257, 200, 8, 127, 300]
    batch = batch_of(lengths, cfg.vocab)
    got, _, flags, _ = run_predict(model, batch)
    assert flags == 0 and np.isfinite(got).all()
    more = batch_of(lengths + [250] * 2, cfg.vocab)
    more.token_ids[: batch.token_ids.size] = batch.token_ids
    for other in (more, padded_to(batch, 512)):
        far, _, flags, _ = run_predict(model, other)
        assert flags == 0 and np.array_equal(got, far[: len(lengths)])


def test_requests_without_rows(tmp_models):
    """Faulty requests among carried ones: a token outside the vocabulary (its rows are there), one that is too long (none)."""
    model, _ = make(tmp_models, f"carried_{WIDE.hidden}.bin", WIDE, ln_jitter=0.1, bias_std=0.05)
    lengths = np.array([64, 8, 129, 700, 1, 64, 256] * 6, np.int32)
    ids = np.random.default_rng(5).integers(0, WIDE.vocab, int(lengths.sum())).astype(np.int32)
    batch = wl.pack_prompts(lengths, ids)
    ids = batch.token_ids
    ids[batch.offsets[9]] = WIDE.vocab
    got, tokens, flags, _ = run_predict(model, batch)
    bad = (lengths > WIDE.max_pos) | (np.arange(lengths.size) == 9)
    assert flags == ps.PS_ST_BAD_TOKEN | ps.PS_ST_BAD_LENGTH and np.isnan(got[bad]).all() and (tokens[bad] == -1).all()
    keep = np.flatnonzero(~bad)
    part = wl.pack_prompts(lengths[keep], np.concatenate([ids[batch.offsets[r]:batch.offsets[r + 1]] for r in keep]))
    want, _, flags, _ = run_predict(model, part)
    assert flags == 0 and np.array_equal(got[keep], want)
