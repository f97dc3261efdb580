"""The decoder step at the sizes where its kernels change over: every K that the
streaming products unroll or loop over, the row counts at which their tile
changes, and key counts around what one round of a workgroup's wavefronts
takes.  Teacher-forced logits against the oracle, with the tolerances of the
other parity tests."""
import numpy as np
import pytest

from paper_2503_05931_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch


def run(oracle, tol, dtype, d_model, head_dim, enc_lens, d_ffn, steps, seed, **kw):
    from tests import gpu_util as G
    cfg = W.DecoderConfig(name="shapes", n_layers=2, d_model=d_model, n_heads=d_model // head_dim, head_dim=head_dim,
                          d_ffn=d_ffn, vocab=192, dtype=dtype, batch=len(enc_lens), prompt_len=1, max_new=steps + 1, **kw)
    wl = W.custom(cfg, enc_lens, seed, random_ln=True)
    toks = np.random.default_rng(seed).integers(0, cfg.vocab, size=(len(enc_lens), steps)).astype(np.int32)
    ref = oracle.Model(cfg, wl.weights).decode_forced(wl.enc, wl.enc_lens, toks)
    dec = G.make_decoder(wl)
    glog, gids = G.forced_logits_gpu(dec, wl, toks)
    err, _ = G.check_forced(ref, glog, gids, G.TOL[tol])
    print(f"{tol} d={d_model} ffn={d_ffn} batch={len(enc_lens)}: max |dlogit| = {err:.2e}")
    dec.close()


# K = d_model: 256 .. 768 loop or, where they have fewer blocks than the ring, are fetched whole; 1024 unrolled; K = d_ffn:
# 4096 unrolled, the others loop with a full ring, without one and with remainders.  Rows: one tile of 16, then 32, 64 and
# 128 rows and one more; 300 rows for short K on the larger tiles; 130 to 900 rows of float32, where every tile is taken, in
# one round of workgroups and in several.
@pytest.mark.parametrize("dtype,d_model,head_dim,d_ffn,batch", [
    ("bf16", 256, 64, 256, 1), ("bf16", 512, 128, 1280, 16), ("bf16", 768, 64, 2304, 17), ("bf16", 1024, 128, 4096, 33),
    ("bf16", 1024, 128, 4352, 65), ("bf16", 1024, 64, 2048, 129), ("bf16", 1024, 128, 4096, 257),
    ("fp32", 256, 64, 768, 17), ("fp32", 512, 128, 2048, 33), ("fp32", 1024, 128, 4096, 65), ("fp32", 768, 64, 1280, 130),
    ("fp32", 1024, 128, 4096, 17), ("fp32", 1024, 64, 4096, 32),
    ("bf16", 256, 64, 256, 300), ("bf16", 512, 64, 768, 300), ("fp32", 256, 64, 256, 300), ("fp32", 512, 128, 512, 300),
    ("fp32", 1024, 128, 4096, 130), ("fp32", 1024, 128, 4096, 300), ("fp32", 1024, 64, 4096, 528), ("fp32", 1024, 128, 4096, 656),
    ("fp32", 768, 64, 3072, 300), ("fp32", 1024, 128, 4352, 900),
])
def test_product_shapes(torch_cuda, oracle, dtype, d_model, head_dim, d_ffn, batch):
    run(oracle, dtype, dtype, d_model, head_dim, [1 + (5 * i) % 9 for i in range(batch)], d_ffn, 2, batch + d_ffn)


# Cross-attention of one or two sequences, and of a few long ones among short ones: those of more than 192 keys are cut, into 4 to 8
# pieces of 64 keys (80 of 513), on 8 wavefronts, or on 4 where no item has more than 64 keys (batch 1) or 8 are not all resident.
@pytest.mark.parametrize("dtype,kv_fp8", [("bf16", 0), ("bf16", 1), ("fp32", 0)])
@pytest.mark.parametrize("batch", [1, 2, 64, 65, 256, 257])
def test_attention_splits(torch_cuda, oracle, dtype, kv_fp8, batch):
    lens = ([256, 513, 257, 255, 512, 1, 16, 17] + [1 + (7 * i) % 33 for i in range(batch)])[:batch]
    if batch == 1:
        lens = [257]
    run(oracle, "bf16+fp8kv" if kv_fp8 else dtype, dtype, 256, 64, lens, 256, 2, 7 + batch, kv_fp8=kv_fp8)


# Self-attention with a long history: batch 32 (128 workgroups, sequences whole) has up to three blocks to each of 8 wavefronts;
# small batches are cut, the last length just past a whole number of chunks.
@pytest.mark.parametrize("dtype,kv_fp8,batch,steps", [
    ("bf16", 0, 32, 300), ("bf16", 1, 32, 300), ("fp32", 0, 32, 300), ("bf16", 0, 3, 513), ("bf16", 1, 2, 300), ("fp32", 0, 2, 300),
])
def test_self_attention_history(torch_cuda, oracle, dtype, kv_fp8, batch, steps):
    lens = [1 + (7 * i) % 33 for i in range(batch)]
    run(oracle, "bf16+fp8kv" if kv_fp8 else dtype, dtype, 256, 64, lens, 256, steps, steps + batch, kv_fp8=kv_fp8)


# Cross-attention of whole sequences of every number of blocks that a wavefront's loop tells apart (none, one, two, odd, even), on 4
# wavefronts (256 sequences of up to 340 keys) and on 8 (bfloat16: 160 to 339 keys on average long, and 32 of like length, one
# workgroup a CU; float32: 100 uneven ones); then sequences of several times the mean's keys among short ones, which are cut into 2
# to 8 pieces, the last one key long (136: where float32 has more than 512 workgroups).
@pytest.mark.parametrize("dtype,kv_fp8", [("bf16", 0), ("bf16", 1), ("fp32", 0)])
@pytest.mark.parametrize("batch,lens", [
    (256, lambda i: 1 + (37 * i) % 340), (256, lambda i: 160 + (37 * i) % 180), (32, lambda i: 380 + (37 * i) % 121), (100, lambda i: 1 + (37 * i) % 340),
    (40, lambda i: [192, 193, 321, 449, 512, 600, 1500][i // 5 % 7] if i % 5 == 0 else 1 + 7 * i % 60),
    (136, lambda i: 200 + 19 * i if i % 9 == 0 else 1 + 7 * i % 60),
])
def test_cross_attention_blocks_and_pieces(torch_cuda, oracle, dtype, kv_fp8, batch, lens):
    run(oracle, "bf16+fp8kv" if kv_fp8 else dtype, dtype, 256, 64, [lens(i) for i in range(batch)], 256, 1, 3 + batch,
        kv_fp8=kv_fp8)


@pytest.mark.parametrize("lens", [[300, 40, 9, 520], [5 + 3 * i for i in range(37)]])
def test_finished_sequences_leave_the_work_list_and_come_back(torch_cuda, oracle, lens):
    """Sequences that end are struck off the cross-attention work list (with few sequences several items each); the same
    batch decoded again has them back."""
    from tests import gpu_util as G
    torch, n, N = torch_cuda, len(lens), 12
    cfg = W.DecoderConfig(name="ends", n_layers=2, d_model=256, n_heads=4, head_dim=64, d_ffn=256, vocab=192, dtype="fp32",
                          batch=n, prompt_len=2, max_new=N, eos_id=2, pad_id=7)
    wl = W.custom(cfg, lens, 31, random_ln=True)
    target = np.array([1 + (5 * i) % N for i in range(n)], np.int32)
    m = oracle.Model(cfg, wl.weights)
    ref_t, ref_l, ref_lg = m.greedy_decode(wl.enc, wl.enc_lens, wl.prompt, N, max_new_per_seq=target, want_logits=True)
    dec = G.make_decoder(wl)
    dec.aed_cross_kv_precompute(dec.to_device(wl.enc), wl.enc_lens)
    near = G.first_near_tie(ref_lg, G.TOL["fp32"])
    for _ in range(2):
        toks, got = dec.aed_greedy_decode(torch.from_numpy(wl.prompt).to(dec.device), N, max_new_per_seq=target)
        toks, got = toks.cpu().numpy(), got.cpu().numpy()
        for b in range(n):
            k = min(int(near[b]), int(ref_l[b]))
            assert (toks[b, :k] == ref_t[b, :k]).all()
            if near[b] >= ref_l[b]:
                assert got[b] == ref_l[b] and (toks[b, got[b]:] == 7).all()
    dec.close()


def test_prompt_fed_by_steps_before_a_single_token(torch_cuda, oracle):
    """A prompt that goes through whole steps (no prefill rows), then one token: no sequence may be off the work list
    (of more than 64 items) before that token, so its logits are the oracle's."""
    from tests import gpu_util as G
    torch, B = torch_cuda, 100
    cfg = W.DecoderConfig(name="one", n_layers=2, d_model=256, n_heads=4, head_dim=64, d_ffn=256, vocab=192, dtype="fp32",
                          batch=B, prompt_len=3, max_new=1)
    wl = W.custom(cfg, [1 + (7 * i) % 33 for i in range(B)], 41, random_ln=True)
    ref = oracle.Model(cfg, wl.weights).decode_forced(wl.enc, wl.enc_lens, wl.prompt)
    dec = G.make_decoder(wl)
    dec.aed_cross_kv_precompute(dec.to_device(wl.enc), wl.enc_lens)
    _, lens = dec.aed_greedy_decode(torch.from_numpy(wl.prompt).to(dec.device), 1)
    assert (lens.cpu().numpy() == 1).all()
    assert np.abs(dec.aed_read_logits() - ref[:, -1]).max() <= G.TOL["fp32"]
    dec.close()
