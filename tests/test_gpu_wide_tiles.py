"""Products of bfloat16 decoders on eight wavefronts (csrc/gemm_decode.hip, eight_wavefronts): every tile that has them, with whole and
ragged last row tiles, in one round of workgroups and, 64 x 64, in several; and the row counts at which 128 x 128 tiles take over
and give way again.  Teacher-forced logits of sampled sequences, at the tiles' edges among them, against the oracle."""
import numpy as np
import pytest

from paper_2503_05931_amd import workloads as W

pytestmark = pytest.mark.gpu


# rows: 81 and 128 (32 x 64, FFN2 on 32 x 16), 130 and 256 (64 x 64, its pair launch 64 x 32), 330 and 512 (1024 columns on 32 x 64 or
# 64 x 32), 701 (64 x 64 there), 1000 (128 x 128 for 4096 columns, 64 x 64 and 32 x 64 for the others), 1409 (two rounds of 128 x 128,
# streamed instead); norm_type 1: the statistics' other form
@pytest.mark.parametrize("batch,norm_type", [(81, 0), (128, 1), (130, 0), (256, 0), (330, 0), (512, 1), (701, 0), (1000, 0), (1409, 0)])
def test_wide_tiles(oracle, batch, norm_type):
    import torch
    from tests import gpu_util as G
    assert torch.cuda.is_available()
    cfg = W.DecoderConfig(name="wide", n_layers=2, d_model=1024, n_heads=8, head_dim=128, d_ffn=4096, vocab=1024, dtype="bf16",
                          batch=batch, prompt_len=1, max_new=3, norm_type=norm_type)
    wl = W.custom(cfg, [1 + (5 * i) % 9 for i in range(batch)], batch, random_ln=True)
    toks = np.random.default_rng(batch).integers(0, cfg.vocab, size=(batch, 2)).astype(np.int32)
    edges = [0, 15, 16, 31, 32, 63, 64, 79, 80, 127, 128, 191, 192, 255, 256, 320, 511, 512, 700, batch // 2, batch - 2, batch - 1]
    rows = sorted({r for r in edges if r < batch})
    sub = wl.subset(rows)
    ref = oracle.Model(wl.cfg, wl.weights).decode_forced(sub.enc, sub.enc_lens, toks[rows])
    dec = G.make_decoder(wl)
    glog, gids = G.forced_logits_gpu(dec, wl, toks, rows)
    err, _ = G.check_forced(ref, glog, gids, G.TOL["bf16"])
    print(f"batch {batch}: max |dlogit| = {err:.2e}")
    dec.close()
