"""GPU parity of the request queue (slot refill): every request that goes
through aed_greedy_decode_queue must come out as the oracle decodes it on its
own -- greedy decoding of a sequence does not depend on what shares its batch.
Token ids and lengths are compared exactly for every request whose oracle
logits have no near-tie (top-1/top-2 margin <= 2 * tolerance) before its end."""
import numpy as np
import pytest

from paper_2503_05931_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch


def queue_workload(dtype, n_req, seed, max_new, d_model=256, n_heads=4, head_dim=64, max_enc=130, eos_id=-1, pad_id=0,
                   min_enc=1, kv_fp8=0, long_every=1):
    rng = np.random.default_rng(seed)
    enc_lens = rng.integers(min_enc, max_enc + 1, size=n_req)
    if long_every > 1:
        enc_lens[np.arange(n_req) % long_every != 0] //= 10
        enc_lens = np.maximum(enc_lens, 1)
    enc_lens[rng.integers(0, n_req)] = max_enc          # the longest length occurs
    cfg = W.DecoderConfig(name="queue", n_layers=2, d_model=d_model, n_heads=n_heads, head_dim=head_dim, d_ffn=512,
                          vocab=256, dtype=dtype, batch=n_req, prompt_len=3, max_new=max_new, eos_id=eos_id,
                          pad_id=pad_id, kv_fp8=kv_fp8)
    return W.custom(cfg, enc_lens, seed, random_ln=True)


def pick_eos(oracle, dtype, n_req, seed, max_new, **kw):
    """An id that some requests emit on their own a few steps in, so natural and forced ends both occur."""
    wl0 = queue_workload(dtype, n_req, seed, max_new, **kw)
    free, _ = oracle.Model(wl0.cfg, wl0.weights).greedy_decode(wl0.enc, wl0.enc_lens, wl0.prompt, max_new)
    ids, counts = np.unique(free[:, 2:10], return_counts=True)
    return int(ids[counts.argmax()])


def run_queue_case(torch, oracle, dtype, n_req, slots, seed, max_new, frames_cap=None, **kw):
    from tests import gpu_util as G
    tol = G.TOL["bf16+fp8kv" if kw.get("kv_fp8") else dtype]
    eos = pick_eos(oracle, dtype, n_req, seed, max_new, **kw)
    wl = queue_workload(dtype, n_req, seed, max_new, eos_id=eos, pad_id=5, **kw)
    rng = np.random.default_rng(seed + 1)
    target = rng.integers(1, max_new + 8, size=n_req).astype(np.int32)  # some above max_new: no forced end
    m = oracle.Model(wl.cfg, wl.weights)
    ref_t, ref_l, ref_logits = m.greedy_decode(wl.enc, wl.enc_lens, wl.prompt, max_new, max_new_per_seq=target,
                                               want_logits=True)
    order = np.argsort(-wl.enc_lens)[:slots]
    cap = frames_cap or int(wl.enc_lens[order].sum())
    dec = G.make_decoder(wl, max_batch=slots, max_total=cap)
    toks, lens, steps = dec.aed_greedy_decode_queue(dec.to_device(wl.enc), wl.enc_lens,
                                                    torch.from_numpy(wl.prompt).to(dec.device), max_new,
                                                    max_new_per_req=target)
    toks, lens = toks.cpu().numpy(), lens.cpu().numpy()
    first = G.first_near_tie(ref_logits, tol)
    fixed = 0
    for r in range(n_req):
        assert 1 <= lens[r] <= min(max_new, int(target[r]))
        assert (toks[r, lens[r]:] == 5).all(), "pad_id after the end"
        if first[r] >= ref_l[r]:
            fixed += 1
            assert lens[r] == ref_l[r], f"request {r}: length {lens[r]} != {ref_l[r]}"
            assert (toks[r] == ref_t[r]).all(), f"request {r}: tokens differ"
        else:
            assert (toks[r, :first[r]] == ref_t[r, :first[r]]).all(), f"request {r}: tokens differ before the near-tie"
    # slot refill must beat running the requests as fixed batches of `slots` in queue order
    fixed_batches = sum((wl.cfg.prompt_len - 1) + int(ref_l[i:i + slots].max()) for i in range(0, n_req, slots))
    print(f"queue {dtype}: {n_req} requests / {slots} slots, {fixed}/{n_req} without near-tie, "
          f"{steps} steps (fixed batches: {fixed_batches})")
    if dtype == "fp32":  # at the bf16 tolerance near-ties are common; the prefix check above still binds
        assert fixed >= n_req * 3 // 4
    dec.close()
    return steps, fixed_batches


def test_queue_fp32_more_requests_than_slots(torch_cuda, oracle):
    steps, fixed_batches = run_queue_case(torch_cuda, oracle, "fp32", n_req=37, slots=8, seed=5, max_new=24)
    assert steps <= fixed_batches + 8 * 5  # polling granularity: at most 8 steps per fixed batch of slack


def test_queue_frames_scarce(torch_cuda, oracle):
    # the frame axis holds little more than the longest request: the queue stalls on frames, not on slots,
    # and parked slots are re-used once frames come back
    run_queue_case(torch_cuda, oracle, "fp32", n_req=21, slots=6, seed=9, max_new=16, frames_cap=200)


def test_queue_bf16(torch_cuda, oracle):
    run_queue_case(torch_cuda, oracle, "bf16", n_req=50, slots=16, seed=13, max_new=20, d_model=512, n_heads=4,
                   head_dim=128, max_enc=300)


def test_queue_of_long_requests_among_short_ones(torch_cuda, oracle):
    # one request in six has ten times the others' frames and is cut into several work items; the others pad the list
    run_queue_case(torch_cuda, oracle, "fp32", n_req=30, slots=5, seed=37, max_new=10, max_enc=700, long_every=6)


def test_queue_large_refill_through_the_frame_map(torch_cuda, oracle):
    # the first refill brings in more than 5 120 frames at d_model 1024, so the cross K/V of the new requests go
    # through the 256 x 256 direct-to-LDS kernel and its frame map
    run_queue_case(torch_cuda, oracle, "bf16", n_req=36, slots=26, seed=29, max_new=8, d_model=1024, n_heads=8,
                   head_dim=128, max_enc=300, min_enc=200)


def test_queue_large_refill_with_fp8_caches(torch_cuda, oracle):
    # the same refill size with 8-bit caches: the 256 x 256 kernel writes E4M3 codes through the frame map
    run_queue_case(torch_cuda, oracle, "bf16", n_req=36, slots=26, seed=31, max_new=8, d_model=1024, n_heads=8,
                   head_dim=128, max_enc=300, min_enc=200, kv_fp8=1)


def test_queue_fewer_requests_than_slots_and_errors(torch_cuda, oracle):
    from tests import gpu_util as G
    from paper_2503_05931_amd import binding
    torch = torch_cuda
    run_queue_case(torch, oracle, "fp32", n_req=3, slots=8, seed=17, max_new=12, frames_cap=512)
    run_queue_case(torch, oracle, "fp32", n_req=1, slots=4, seed=19, max_new=12, frames_cap=256)
    # errors are found on the host and leave the decoder usable
    wl = queue_workload("fp32", 4, 23, 12)              # eos_id = -1
    dec = G.make_decoder(wl, max_batch=2, max_total=300)
    prm = torch.from_numpy(wl.prompt).to(dec.device)
    with pytest.raises(binding.AedError) as e:
        dec.aed_greedy_decode_queue(dec.to_device(wl.enc), wl.enc_lens, prm, 12)
    assert e.value.status == binding.AED_EINVAL
    dec.close()
    eos = 11
    wl = queue_workload("fp32", 4, 23, 12, eos_id=eos)
    dec = G.make_decoder(wl, max_batch=2, max_total=100)   # the longest request has 130 frames
    prm = torch.from_numpy(wl.prompt).to(dec.device)
    with pytest.raises(binding.AedError) as e:
        dec.aed_greedy_decode_queue(dec.to_device(wl.enc), wl.enc_lens, prm, 12)
    assert e.value.status == binding.AED_ECAPACITY
    with pytest.raises(binding.AedError) as e:
        dec.aed_greedy_decode_queue(dec.to_device(wl.enc), wl.enc_lens, prm, wl.cfg.max_dec_len)
    assert e.value.status == binding.AED_ECAPACITY
    dec.close()
    dec = G.make_decoder(wl, max_batch=2, max_total=300, kv_pages=1)
    prm = torch.from_numpy(wl.prompt).to(dec.device)
    with pytest.raises(binding.AedError) as e:
        dec.aed_greedy_decode_queue(dec.to_device(wl.enc), wl.enc_lens, prm, 12)
    assert e.value.status == binding.AED_ECAPACITY
    # and the decoder still runs a queue after the refused calls (pool of 2 pages: one per slot)
    dec.close()
    dec = G.make_decoder(wl, max_batch=2, max_total=300, kv_pages=2)
    prm = torch.from_numpy(wl.prompt).to(dec.device)
    with pytest.raises(binding.AedError):
        dec.aed_greedy_decode_queue(dec.to_device(wl.enc), wl.enc_lens, prm, 0)
    toks, lens, steps = dec.aed_greedy_decode_queue(dec.to_device(wl.enc), wl.enc_lens, prm, 12)
    ref_t, ref_l, ref_logits = oracle.Model(wl.cfg, wl.weights).greedy_decode(wl.enc, wl.enc_lens, wl.prompt, 12,
                                                                              want_logits=True)
    first = G.first_near_tie(ref_logits, G.TOL["fp32"])
    for r in range(4):
        if first[r] >= ref_l[r]:
            assert lens.cpu().numpy()[r] == ref_l[r] and (toks.cpu().numpy()[r] == ref_t[r]).all()
    dec.close()
