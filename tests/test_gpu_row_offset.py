"""float32 decoders whose residual rows have a common offset: the products behind a LayerNorm take the row's mean off in front of the
multiplication, and a residual update rounds once at the size of the row (csrc/gemm_decode.hip).  Teacher-forced logits
against the oracle in float64, relative 2-norm."""
import numpy as np
import pytest

from paper_2503_05931_amd import workloads as W

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


def relative_error(oracle, wl, steps):
    from tests import gpu_util as G
    B = wl.cfg.batch
    toks = np.random.default_rng(B).integers(0, wl.cfg.vocab, size=(B, steps)).astype(np.int32)
    rows = sorted({r for r in (0, 1, 15, 16, 31, 32, 63, 64, 127, 128, B // 2, B - 1) if r < B})
    sub = wl.subset(rows)
    ref = oracle.Model(wl.cfg, wl.weights).decode_forced(sub.enc, sub.enc_lens, toks[rows])
    dec = G.make_decoder(wl)
    got, _ = G.forced_logits_gpu(dec, wl, toks, rows)
    dec.close()
    return float(np.linalg.norm(got - ref) / np.linalg.norm(ref))


def workload(batch, d_model, norm_type=0, n_layers=1, **kw):
    cfg = W.DecoderConfig(name="offset", n_layers=n_layers, d_model=d_model, n_heads=d_model // 64, head_dim=64, d_ffn=256, vocab=192,
                          dtype="fp32", batch=batch, prompt_len=1, max_new=4, norm_type=norm_type, **kw)
    return W.custom(cfg, [1 + (5 * i) % 9 for i in range(batch)], 100 + batch, random_ln=True)


# A bias moves the rows by `shift` standard deviations of the embeddings, inside the layer (b_o; b_ff2 brings them back) or at its end.
# The bound: without a shift all sums together err by 4 (d_model 256) to 7 (1024) units; with it a row's elements are stored, and
# its mean is, within `shift` units of an embedding's spread each, 0.3 to 0.6 of that on average, once to three times on the way; the rows
# that the last product reads are spread 3 (256) to 10 (1024) times as wide.  Of a product over rows with the offset
# still in them, the sums err by as much as the offset again: 300 spreads, 256 columns 4.8e-6 to 7.0e-6, this 1.8e-6 to 2.7e-6.
@pytest.mark.parametrize("d_model,per_shift", [(256, 0.2), (1024, 0.08)])
@pytest.mark.parametrize("batch", [3, 40, 130])  # tiles of 16, 32 and 64 rows
@pytest.mark.parametrize("where,shift,norm_type", [("inside", 300, 0), ("end", 300, 0), ("end", 30, 0), ("end", 1, 0), ("inside", 300, 1)])
def test_updates_that_move_the_mean(oracle, d_model, per_shift, batch, where, shift, norm_type):
    wl = workload(batch, d_model, norm_type)
    w, l = wl.weights, wl.weights["layers"][0]
    by = np.float32(shift * np.std(wl.cfg.emb_scale * w["tok_emb"]))
    if where == "inside":
        l["b_o"] = l["b_o"] + by
        l["b_ff2"] = l["b_ff2"] - by
    else:
        l["b_ff2"] = l["b_ff2"] + by
    err = relative_error(oracle, wl, 3)
    print(f"d {d_model} batch {batch} {where} {shift}: {err:.2e} = {err / U:.1f} units")
    assert err <= U * (8 + per_shift * shift)


# Rows of integers around 2^23, where float32 has integers only; every FFN adds a half of an integer by its product and the other half by
# its bias.  Added to the row one after the other the halves are lost, which is up to 2e-2 of the logits; added up first
# the row is exact.  The vocabulary rows have sum 0, so that the rounding of the row's mean does not count.  That of its 16 tiles' means
# does: 0.35 on average, of means that are 64 / 4 apart, is 2 * 16 * 16 * 0.35 * sqrt(16) of a sum of squares of 256 * 64^2 or
# 3.4e-4 of its root; three times that.
@pytest.mark.parametrize("batch", [3, 40, 130])
def test_a_residual_update_rounds_once(oracle, batch):
    rng = np.random.default_rng(batch)
    wl = workload(batch, 256, n_layers=2, emb_scale=1.0)
    w = wl.weights
    w["tok_emb"] = rng.integers(-110, 111, size=w["tok_emb"].shape).astype(np.float32)
    w["pos_emb"] = np.full_like(w["pos_emb"], 2.0 ** 23 + 1000)
    w["w_out"] = w["w_out"] - w["w_out"].mean(1, keepdims=True)
    w["lnf_g"] = np.ones_like(w["lnf_g"])
    for l in w["layers"]:
        for k in ("w_o", "b_o", "w_co", "b_co", "w_ff1", "w_ff2"):
            l[k] = np.zeros_like(l[k])
        l["b_ff1"] = np.ones_like(l["b_ff1"])
        half = 0.5 * rng.choice([-3, -1, 1, 3], size=wl.cfg.d_model).astype(np.float32)
        l["w_ff2"][:, 7] = half
        l["b_ff2"] = half
    err = relative_error(oracle, wl, 2)
    print(f"batch {batch}: {err:.2e}")
    assert err <= 1e-3
