"""GPU tests of the library's state handling: several decoders alive at once on one device (each on its own stream,
their steps interleaved), and handles created and destroyed many times (nothing the library owns may pile up)."""
import numpy as np
import pytest

from paper_2503_05931_amd import workloads as W

pytestmark = pytest.mark.gpu


def _unit(dtype, d_model, n_heads, head_dim, enc_lens, seed, **kw):
    cfg = W.DecoderConfig(name="unit", n_layers=2, d_model=d_model, n_heads=n_heads, head_dim=head_dim, d_ffn=512,
                          vocab=256, dtype=dtype, batch=len(enc_lens), prompt_len=4, max_new=24, **kw)
    return W.custom(cfg, enc_lens, seed, random_ln=True)


def test_two_decoders_interleaved_on_one_device(oracle):
    """A bf16 decoder whose long sequences are cut into merged chunks and an fp32 decoder of another shape take
    turns, step by step, on their own streams; every logit of both is compared with the oracle, as if each had
    run alone."""
    import torch
    from tests import gpu_util as G
    wl_a = _unit("bf16", 256, 4, 64, [300, 7, 150], seed=5)
    wl_b = _unit("fp32", 512, 4, 128, [9, 33, 1, 64, 17], seed=6)
    S = 20
    tok_a = np.random.default_rng(1).integers(0, 256, size=(3, S)).astype(np.int32)
    tok_b = np.random.default_rng(2).integers(0, 256, size=(5, S)).astype(np.int32)
    ref_a = oracle.Model(wl_a.cfg, wl_a.weights).decode_forced(wl_a.enc, wl_a.enc_lens, tok_a)
    ref_b = oracle.Model(wl_b.cfg, wl_b.weights).decode_forced(wl_b.enc, wl_b.enc_lens, tok_b)
    dec_a, dec_b = G.make_decoder(wl_a), G.make_decoder(wl_b)
    dec_a.aed_cross_kv_precompute(dec_a.to_device(wl_a.enc), wl_a.enc_lens)
    dec_b.aed_cross_kv_precompute(dec_b.to_device(wl_b.enc), wl_b.enc_lens)
    dev_a = torch.from_numpy(np.ascontiguousarray(tok_a.T)).to(dec_a.device)
    dev_b = torch.from_numpy(np.ascontiguousarray(tok_b.T)).to(dec_b.device)
    log_a, ids_a, log_b, ids_b = [], [], [], []
    for s in range(S):  # no synchronisation between the two: their launches overlap on the device
        out, lg = dec_a.aed_decode_step(dev_a[s].contiguous())
        log_a.append(lg); ids_a.append(out)
        out, lg = dec_b.aed_decode_step(dev_b[s].contiguous())
        log_b.append(lg); ids_b.append(out)
    torch.cuda.synchronize()
    G.check_forced(ref_a, torch.stack(log_a, 1).cpu().numpy().astype(np.float64), torch.stack(ids_a, 1).cpu().numpy(),
                   G.TOL["bf16"])
    G.check_forced(ref_b, torch.stack(log_b, 1).cpu().numpy().astype(np.float64), torch.stack(ids_b, 1).cpu().numpy(),
                   G.TOL["fp32"])
    # and a greedy decode on one while the other has a step batch open
    dec_b.aed_cross_kv_precompute(dec_b.to_device(wl_b.enc), wl_b.enc_lens)
    ref_t, ref_l, ref_logits = oracle.Model(wl_b.cfg, wl_b.weights).greedy_decode(wl_b.enc, wl_b.enc_lens, wl_b.prompt, 12,
                                                                               want_logits=True)
    toks, lens = dec_b.aed_greedy_decode(torch.from_numpy(wl_b.prompt).to(dec_b.device), 12)
    out, lg = dec_a.aed_decode_step(dev_a[0].contiguous())   # dec_a's batch is still at position S: one more step
    toks = toks.cpu().numpy()
    first = G.first_near_tie(ref_logits, G.TOL["fp32"])
    for b in range(5):
        assert (toks[b, :first[b]] == ref_t[b, :first[b]]).all()
    dec_a.close()
    dec_b.close()


@pytest.mark.parametrize("dtype,prefill_rows", [("bf16", 48), ("fp32", 0)])
def test_batches_of_many_shapes_in_turn(oracle, dtype, prefill_rows):
    """More shapes than a decoder keeps graphs of, and the first ones again, greedy and by steps: every batch comes out
    as on a decoder that has seen nothing else, bit for bit, and the first as the oracle has it."""
    import torch
    from tests import gpu_util as G
    shapes = [[20], [300, 7], [5, 6, 7], [400], [9, 200, 33, 1], [64] * 5, [20], [21], [300, 7], [7, 300], [260]]
    wl = _unit(dtype, 256, 4, 64, [400] * 5, seed=12)
    kw = dict(max_batch=5, max_total=2000, prefill_rows=prefill_rows)
    rng = np.random.default_rng(4)
    enc = {i: W.draw_enc_states(wl.cfg, rng, np.array(s, np.int32)) for i, s in enumerate(shapes)}

    def decode(dec, i):
        lens = np.array(shapes[i], np.int32)
        prompt = torch.from_numpy(wl.prompt[:len(lens)].copy()).to(dec.device)
        dev = dec.to_device(enc[i])
        dec.aed_cross_kv_precompute(dev, lens)
        toks, _ = dec.aed_greedy_decode(prompt, 7)
        out = [toks.cpu().numpy(), dec.aed_read_logits()]
        dec.aed_cross_kv_precompute(dev, lens)
        for t in range(2):
            ids, lg = dec.aed_decode_step(prompt[:, t].contiguous())
            out += [ids.cpu().numpy(), lg.cpu().numpy()]
        return out

    shared = G.make_decoder(wl, **kw)
    for i, lens in enumerate(shapes):
        got = decode(shared, i)
        alone = G.make_decoder(wl, **kw)
        for a, b in zip(got, decode(alone, i)):
            assert np.array_equal(a, b), f"batch {i} of {lens}"
        alone.close()
        if i == 0:
            ref = oracle.Model(wl.cfg, wl.weights).decode_forced(enc[0], np.array(lens, np.int32), wl.prompt[:1, :2].copy())
            assert np.abs(np.stack([got[3], got[5]], 1) - ref).max() <= G.TOL[dtype]
    shared.close()


def test_create_destroy_many_times_leaves_nothing_behind():
    """40 handles created, used (one batch, a few greedy tokens: graphs, events and pinned memory come into being) and
    destroyed: the device's free memory afterwards is what it was after the first few (torch's own caches warm up
    during those)."""
    import torch
    from tests import gpu_util as G
    wl = _unit("bf16", 256, 4, 64, [20, 5], seed=9)
    prompt = None
    free_after = []
    for i in range(40):
        dec = G.make_decoder(wl, poison=False)
        if prompt is None:
            prompt = torch.from_numpy(wl.prompt).to(dec.device)
            enc = dec.to_device(wl.enc)
        dec.aed_cross_kv_precompute(enc, wl.enc_lens)
        toks, lens = dec.aed_greedy_decode(prompt, 6)
        assert int(lens.sum().item()) == 12
        dec.close()
        del dec, toks, lens
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        free_after.append(torch.cuda.mem_get_info()[0])
    # allow the allocator's granularity, not a per-handle loss: 35 more handles may not cost 32 MiB
    assert free_after[4] - free_after[-1] < (32 << 20), f"free memory fell from {free_after[4]} to {free_after[-1]}"


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_a_steps_results_go_where_they_are_asked_for(dtype):
    """aed_decode_step with either output missing, and logits to an address that is no multiple of 16: the same values as to
    tensors of their own, and nothing beside them is written."""
    import ctypes as C
    import torch
    from tests import gpu_util as G
    wl = _unit(dtype, 256, 4, 64, [9, 33, 1, 64, 17], seed=8)
    B, V, S = 5, wl.cfg.vocab, 18  # past a page's end
    toks = torch.from_numpy(np.random.default_rng(3).integers(0, V, size=(S, B)).astype(np.int32)).cuda()
    dec = G.make_decoder(wl)
    dec.aed_cross_kv_precompute(dec.to_device(wl.enc), wl.enc_lens)
    want = [dec.aed_decode_step(toks[s]) for s in range(S)]
    dec.aed_cross_kv_precompute(dec.to_device(wl.enc), wl.enc_lens)
    for s in range(S):
        ids = torch.full((B + 2,), -5, dtype=torch.int32, device="cuda")
        logits = torch.full((B * V + 8,), -7.0, dtype=torch.float32, device="cuda")
        off = s % 4 if s % 3 else 0  # 0, 4, 8 and 12 bytes past a multiple of 16
        torch.cuda.synchronize()
        st = dec.lib.aed_decode_step(dec.handle, C.c_void_p(toks[s].data_ptr()), C.c_void_p(ids[1:].data_ptr()) if s % 5 else None,
                                     C.c_void_p(logits[off:].data_ptr()) if s % 7 else None)
        assert st == 0
        torch.cuda.synchronize()
        assert (ids[[0, -1]] == -5).all() and (ids[1:-1] == (want[s][0] if s % 5 else -5)).all()
        assert (logits[:off] == -7).all() and (logits[off + B * V:] == -7).all()
        got = logits[off:off + B * V].view(B, V)
        assert (got == (want[s][1] if s % 7 else -7)).all()
    dec.close()
