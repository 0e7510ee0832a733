"""GPU parity: the HIP library (through its C ABI) against the CPU oracle on the
same seeded inputs -- kept / retrieved indices bit-exact, copied bytes exact,
float outputs within 1e-5 (fp32 payload) / 2e-2 (bf16 payload)."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2605_22269_amd import binding as mk
from paper_2605_22269_amd import synth
from mukv_testlib import Pair, gpu_context, np_view, out_err, to_f64

pytestmark = pytest.mark.gpu

W = synth.WORKLOADS


def mk_tol(w):
    return 2e-2 if w.dtype == "bf16" else 1e-5


def questions_for(w, lengths, seed):
    return [synth.random_question(w, n, seed + i) for i, n in enumerate(lengths)]


# ------------------------------------------------------------------ config 1 (exactly) -----
def test_tiny_config_end_to_end():
    w = W["tiny"]
    p = Pair(w, seed=11)
    p.ingest()
    st = p.check_compress()
    qs = questions_for(w, [w.question_tokens], 100)
    for mode in (mk.MUKV_SEMI, mk.MUKV_HIER, mk.MUKV_PARALLEL):
        p.check_retrieve(qs, mode, w.k_seg, w.k_frame, w.lambda_frame)
    print("tiny: refined frames", int(st["refined"].sum()), "min margin", float(st["margin"].min()))
    p.close()


# ---------------------------------------- 7B shape, short stream (several chunks, ragged) ----
def test_7b_shape_short_stream():
    w = W["7b"].scaled(n_frames=21, n_questions=2)   # 8 + 8 + 5 frames; segments 16 + 5
    p = Pair(w, seed=5)
    p.ingest()
    st = p.check_compress()
    p.check_retrieve(questions_for(w, [32, 17], 200), mk.MUKV_SEMI, 2, 8, 0.3)
    print("7b: refined frames", int(st["refined"].sum()), "min margin", float(st["margin"].min()))
    p.close()


def test_7b_shape_retrieval_modes():
    w = W["7b"].scaled(n_frames=40, n_layers=2, n_questions=3)
    p = Pair(w, seed=6)
    p.ingest()
    p.check_compress()
    qs = questions_for(w, [32, 16, 64], 300)
    for mode in (mk.MUKV_SEMI, mk.MUKV_HIER, mk.MUKV_PARALLEL):
        p.check_retrieve(qs, mode, 2, 6, 0.3)
    p.check_retrieve(qs, mk.MUKV_SEMI, 2, 6, 0.0)
    p.check_retrieve(qs, mk.MUKV_SEMI, 2, 6, 0.7, n_global=1)
    # timestamp before the end of the stream, cutting segment 1 (frames 16..31) after frame 20
    p.check_retrieve(qs, mk.MUKV_SEMI, 2, 6, 0.3, n_visible=21)
    p.check_retrieve(qs, mk.MUKV_HIER, 1, 4, 0.3, n_visible=21)
    # more blocks asked for than exist
    p.check_retrieve(qs, mk.MUKV_SEMI, 5, 48, 0.3)
    p.check_retrieve(qs, mk.MUKV_PARALLEL, 5, 48, 0.3, n_visible=3)
    p.close()


@pytest.mark.parametrize("distinct", [1, 3, 40])
def test_retrieval_with_many_equal_scores(distinct):
    # 1300 frames cycling through `distinct` different ones: whole classes of frame and segment
    # scores tie exactly, and the selections must still be the oracle's (lowest index first).
    # One class of 1300 overflows the candidate list of the selection kernel's short route,
    # classes of 433 stay inside it, 40 classes put ties across the cut; k_frame = 300 asks for
    # more candidates than the kernel has threads.
    w = W["tiny"].scaled(n_frames=1300, n_questions=2)
    p = Pair(w, seed=90 + distinct, chunk=100)
    P = w.tokens_per_frame
    k0, v0, q0 = p.stream.next_chunk(distinct)
    for c0 in range(0, 1300, 100):
        fr = (torch.arange(c0, c0 + 100) % distinct)
        tok = (fr[:, None] * P + torch.arange(P)[None, :]).reshape(-1)
        k, v, q = k0[:, :, tok].contiguous(), v0[:, :, tok].contiguous(), q0[:, tok].contiguous()
        p.orc.compress_chunk(np_view(k), np_view(v), q_last=np_view(q))
        p.gpu.compress_chunk(k.cuda(), v.cuda(), q.cuda())
        torch.cuda.synchronize()
    qs = questions_for(w, [16, 9], 600)
    for mode in (mk.MUKV_SEMI, mk.MUKV_HIER, mk.MUKV_PARALLEL):
        p.check_retrieve(qs, mode, 4, 8, 0.3)
    p.check_retrieve(qs, mk.MUKV_SEMI, 40, 300, 0.3)
    p.check_retrieve(qs, mk.MUKV_PARALLEL, 3, 512, 0.3)
    p.close()


def test_retrieval_of_list_lengths_at_the_selection_kernels_edges():
    # lists ranked directly (up to 512), pre-filtered from registers (up to 4096) and from LDS; 900 distinct frames, so that
    # exact ties lie on both sides of every cut
    w = W["tiny"].scaled(n_frames=4200, n_questions=2, n_layers=1, tokens_per_frame=8, keep_ratio=0.25, superpatches_per_frame=2)
    p = Pair(w, seed=97, chunk=300)
    P = w.tokens_per_frame
    k0, v0, q0 = p.stream.next_chunk(900)
    for c0 in range(0, 4200, 300):
        tok = (torch.arange(c0, c0 + 300) % 900)[:, None] * P + torch.arange(P)[None, :]
        k, v, q = (x.index_select(-2, tok.reshape(-1)).contiguous() for x in (k0, v0, q0))
        p.orc.compress_chunk(np_view(k), np_view(v), q_last=np_view(q))
        p.gpu.compress_chunk(k.cuda(), v.cuda(), q.cuda())
        torch.cuda.synchronize()
    qs = questions_for(w, [16, 9], 610)
    for n in (1, 511, 512, 513, 4095, 4096, 4097, 4200):
        p.check_retrieve(qs, mk.MUKV_SEMI, 4, 33, 0.3, n_visible=n)
    p.check_retrieve(qs, mk.MUKV_HIER, 5, 40, 0.3, n_visible=4100)
    p.check_retrieve_patches(qs, mk.MUKV_SEMI, 4, 20, 0.3, n_visible=256)    # lists with entries that have no key
    p.check_retrieve_patches(qs, mk.MUKV_SEMI, 4, 20, 0.3, n_visible=2049)
    p.close()


@pytest.mark.parametrize("k", [1, 8, 64, 255, 257, 700])
def test_plan_of_a_gather_over_stores_by_list_length(k):
    # lanes that share an entry: 64, ..., 2, 1; units named twice, and names of no unit
    w = W["tiny"].scaled(n_frames=300, n_layers=1, tokens_per_frame=4, keep_ratio=0.5, superpatches_per_frame=1)
    p = Pair(w, seed=98, chunk=100)
    p.ingest()
    kap = p.gpu.kappa
    rs = np.random.default_rng(k)
    lists = [rs.integers(-2, 310, k), rs.integers(0, 300, k)]
    idx = [torch.from_numpy(x.astype(np.int32))[None].cuda() for x in lists]
    ko, vo, n = mk.gather_multi([p.gpu, p.gpu], idx, [1, 3], 2 * k * kap)
    taken = sorted({(u // (1, 3)[i], i, int(u)) for i in range(2) for u in lists[i] if 0 <= u < 300})
    rows = [u * kap + r for _, _, u in taken for r in range(kap)]
    k_all, v_all = p.gpu.store_rows(0, 300 * kap)
    torch.cuda.synchronize()
    assert int(n[0]) == len(rows)
    for got, want in ((ko, k_all), (vo, v_all)):
        assert torch.equal(got[0, 0, :, :len(rows)], want[0][:, rows])
        assert not got[0, 0, :, len(rows):].any()
    p.close()


@pytest.mark.parametrize("name,frames", [("7b", 41), ("tiny", 100), ("72b", 21)])
def test_batches_of_sixteen_or_more_questions(name, frames):
    # from 16 questions on, the frame scores come from the fp64 matrix-core kernel: ragged
    # frame and question counts, a timestamp that cuts a segment, every retrieval mode
    w = W[name].scaled(n_frames=frames, n_layers=2, n_questions=37)
    p = Pair(w, seed=95, chunk=8)
    p.ingest()
    p.check_compress()
    for nq in (16, 37):
        qs = questions_for(w, [5 + (7 * i) % 40 for i in range(nq)], 700)
        p.check_retrieve(qs, mk.MUKV_SEMI, 2, 6, 0.3)
        p.check_retrieve(qs, mk.MUKV_HIER, 2, 6, 0.3, n_visible=frames - 3)
        p.check_retrieve(qs, mk.MUKV_PARALLEL, 2, 6, 0.3, n_visible=9)
    p.close()


def test_gather_and_attend_skip_numbers_that_name_no_frame():
    # -1 is the padding of a short retrieval; numbers at or past the frames held are skipped the same way
    w = W["7b"].scaled(n_frames=10, n_layers=2, n_questions=2)
    p = Pair(w, seed=8, chunk=5)
    p.ingest()
    p.check_compress()
    lists = [[7, 10, -1, 3, 4096, -5], [-1, 11, 12, 2**31 - 1, 0, 9]]
    idx = torch.tensor(lists, dtype=torch.int32, device="cuda")
    for order in (mk.MUKV_TEMPORAL, mk.MUKV_AS_GIVEN):
        kg, vg, nt = p.gpu.gather_kv(idx, order=order)
        torch.cuda.synchronize()
        for b in range(2):
            ko, vo, n = p.orc.gather(np.array(lists[b], np.int64), order=orc.TEMPORAL if order == mk.MUKV_TEMPORAL else orc.AS_GIVEN)
            assert int(nt[b]) == n == 2 * p.orc.kappa
            np.testing.assert_array_equal(np_view(kg[b].cpu()), ko)
            np.testing.assert_array_equal(np_view(vg[b].cpu()), vo)
    p.check_attend(1, 2, lists, [3, 2], True, seed=9)
    p.close()


# ------------------------------------------------------ 72B shape, short stream -----------
def test_72b_shape_short_stream():
    w = W["72b"].scaled(n_frames=40, n_layers=3)   # kappa 8 of 64; one full 32-frame segment + 8
    p = Pair(w, seed=7)
    p.ingest()
    p.check_compress()
    qs = questions_for(w, [32], 400)
    for mode in (mk.MUKV_SEMI, mk.MUKV_HIER, mk.MUKV_PARALLEL):
        p.check_retrieve(qs, mode, 2, 8, 0.3)
    p.close()


# ------------------------------------------------------------------------ edge cases ------
@pytest.mark.parametrize("alpha", [0.0, 1.0, 0.5])
@pytest.mark.parametrize("causal", [True, False])
def test_signal_mixes_and_masks(alpha, causal):
    w = W["tiny"].scaled(n_frames=10, alpha=alpha, n_layers=2, n_kv_heads=2)
    p = Pair(w, seed=21, chunk=4, gpu_kw={"causal": causal}, orc_kw={"causal": causal})
    p.ingest()
    p.check_compress()
    p.close()


def test_attention_handed_over_by_the_caller():
    w = W["tiny"].scaled(n_frames=9)
    p = Pair(w, seed=22, chunk=4)
    p.ingest(att_from_oracle=True)
    p.check_compress()
    p.close()


def test_keep_ratio_one_is_identity():
    w = W["tiny"].scaled(n_frames=6, keep_ratio=1.0, n_layers=2)
    p = Pair(w, seed=23, chunk=3)
    p.ingest()
    st = p.check_compress()
    P = w.tokens_per_frame
    assert np.array_equal(st["kept_idx"].cpu().numpy(), np.tile(np.arange(P, dtype=np.int32), (6, 1)))
    p.close()


def test_chunking_invariance_bitwise():
    w = W["7b"].scaled(n_frames=12, n_layers=2)
    ref = None
    for chunk in (12, 8, 5, 1):
        p = Pair(w, seed=24, chunk=chunk)
        p.ingest()
        st = p.check_compress()
        torch.cuda.synchronize()
        cur = {k: st[k].cpu().numpy() for k in ("kept_idx", "rep_frame_k", "rep_seg_k", "rep_seg_v", "rep_patch_v")}
        if ref is not None:
            for k in cur:
                np.testing.assert_array_equal(cur[k], ref[k], err_msg=f"{k} chunk={chunk}")
        ref = ref or cur
        p.close()


def test_exact_ties_resolve_to_lowest_position():
    # all keys zero and alpha = 0: every fused score is 0 -> the first kappa tokens
    w = W["tiny"].scaled(n_frames=2, alpha=0.0)
    g = Pair(w, seed=1, chunk=2).gpu
    L, Hkv, P, D = w.n_layers, w.n_kv_heads, w.tokens_per_frame, w.head_dim
    k = torch.zeros(L, Hkv, 2 * P, D, device="cuda")
    v = torch.randn(L, Hkv, 2 * P, D, device="cuda")
    g.compress_chunk(k, v)
    st = g.state()
    torch.cuda.synchronize()
    assert np.array_equal(st["kept_idx"].cpu().numpy(), np.tile(np.arange(g.kappa, dtype=np.int32), (2, 1)))
    g.close()
    # duplicated tokens, non-causal: the copies tie exactly; oracle and GPU must agree
    w = W["tiny"].scaled(n_frames=3, n_kv_heads=2, n_q_heads=4)
    p = Pair(w, seed=2, chunk=3, gpu_kw={"causal": False}, orc_kw={"causal": False})
    k, v, q = p.stream.next_chunk(3)
    for a, b in ((3, 40), (7, 8), (20, 21), (0, 48)):
        k[:, :, b::P] = k[:, :, a::P]
    kn, vn, qn = np_view(k), np_view(v), np_view(q)
    ro = p.orc.compress_chunk(kn, vn, q_last=qn)
    p.gpu.compress_chunk(k.cuda(), v.cuda(), q.cuda())
    st = p.gpu.state()
    torch.cuda.synchronize()
    assert np.array_equal(st["kept_idx"].cpu().numpy(), ro["kept"])
    p.close()


def test_strided_inputs_hf_layout():
    # per-layer [1, Hkv, T_total, D] prefill tensors: a chunk is a slice along T, so the head
    # stride exceeds n*P*D; layers sit in one big buffer here
    w = W["tiny"].scaled(n_frames=8, n_layers=3, n_kv_heads=2)
    p = Pair(w, seed=31, chunk=4)
    P = w.tokens_per_frame
    k, v, q = p.stream.next_chunk(8)
    big_k, big_v, big_q = k.cuda(), v.cuda(), q.cuda()
    for f0 in (0, 4):
        sl = slice(f0 * P, (f0 + 4) * P)
        p.sig_orc.append(p.orc.compress_chunk(np_view(k[:, :, sl]), np_view(v[:, :, sl]), q_last=np_view(q[:, sl])))
        p.sig_gpu.append(p.gpu.compress_chunk(big_k[:, :, sl], big_v[:, :, sl], big_q[:, sl], want_signals=True))
    p.check_compress()
    p.close()


def test_gather_orders_and_padding():
    w = W["tiny"].scaled(n_frames=16, n_layers=2, n_questions=2)
    p = Pair(w, seed=41)
    p.ingest()
    idx = torch.tensor([[9, 2, -1, 4, 15], [0, -1, -1, -1, -1]], dtype=torch.int32, device="cuda")
    for order, oorder in ((mk.MUKV_TEMPORAL, orc.TEMPORAL), (mk.MUKV_AS_GIVEN, orc.AS_GIVEN)):
        kg, vg, nt = p.gpu.gather_kv(idx, order)
        torch.cuda.synchronize()
        for b in range(2):
            ko, vo, n = p.orc.gather(idx[b].cpu().numpy(), oorder)
            assert int(nt[b]) == n
            np.testing.assert_array_equal(np_view(kg[b]), ko)
            np.testing.assert_array_equal(np_view(vg[b]), vo)
    p.close()


@pytest.mark.parametrize("k_frame", [1, 63, 64, 65, 130])
def test_gather_list_lengths_around_a_wave(k_frame):
    # lists of up to 64 entries are planned inside a wave, longer ones in LDS: same bytes either way, with
    # padding, numbers past the cache and a frame named twice in the list
    w = W["tiny"].scaled(n_frames=80, n_layers=2, n_questions=2)
    p = Pair(w, seed=43, chunk=16)
    p.ingest()
    rng = np.random.default_rng(k_frame)
    lists = np.stack([rng.permutation(80)[:k_frame] if k_frame <= 80 else rng.integers(0, 80, k_frame) for _ in range(2)])
    if k_frame >= 3:
        lists[0, 1] = -1
        lists[1, 0] = 80
        lists[1, k_frame - 1] = lists[1, k_frame - 2]
    idx = torch.tensor(lists, dtype=torch.int32, device="cuda")
    for order, oorder in ((mk.MUKV_TEMPORAL, orc.TEMPORAL), (mk.MUKV_AS_GIVEN, orc.AS_GIVEN)):
        kg, vg, nt = p.gpu.gather_kv(idx, order)
        torch.cuda.synchronize()
        for b in range(2):
            ko, vo, n = p.orc.gather(lists[b].astype(np.int64), oorder)
            assert int(nt[b]) == n
            np.testing.assert_array_equal(np_view(kg[b]), ko)
            np.testing.assert_array_equal(np_view(vg[b]), vo)
    p.close()


def test_determinism_bitwise():
    w = W["7b"].scaled(n_frames=8, n_layers=2)
    outs = []
    for _ in range(2):
        p = Pair(w, seed=51)
        k, v, q = p.stream.next_chunk(8)
        sg = p.gpu.compress_chunk(k.cuda(), v.cuda(), q.cuda(), want_signals=True)
        st = p.gpu.state()
        torch.cuda.synchronize()
        outs.append((sg["fused"].cpu().numpy(), st["kept_idx"].cpu().numpy(), st["rep_seg_k"].cpu().numpy()))
        p.close()
    for a, b in zip(*outs):
        np.testing.assert_array_equal(a, b)


def test_capacity_and_argument_errors_on_device():
    w = W["tiny"].scaled(n_frames=8)
    g = Pair(w, seed=1, chunk=4).gpu
    L, Hkv, P, D = w.n_layers, w.n_kv_heads, w.tokens_per_frame, w.head_dim
    k = torch.zeros(L, Hkv, 5 * P, D, device="cuda")
    q = torch.zeros(w.n_q_heads, 5 * P, D, device="cuda")
    with pytest.raises(mk.MuKVError) as e:
        g.compress_chunk(k, k, q)                       # 5 frames > max_chunk_frames
    assert e.value.status == mk.MUKV_ERR_CAPACITY
    with pytest.raises(mk.MuKVError) as e:
        g.compress_chunk(k[:, :, : 4 * P], k[:, :, : 4 * P])  # alpha > 0 but no attention source
    assert e.value.status == mk.MUKV_ERR_INVALID_ARG
    k4, q4 = k[:, :, : 4 * P].contiguous(), q[:, : 4 * P].contiguous()
    g.compress_chunk(k4, k4, q4)
    g.compress_chunk(k4, k4, q4)
    with pytest.raises(mk.MuKVError) as e:
        g.compress_chunk(k4, k4, q4)                    # cache full
    assert e.value.status == mk.MUKV_ERR_CAPACITY
    assert g.n_frames == 8
    qt = torch.zeros(4, w.n_q_heads, D, device="cuda")
    offs = torch.tensor([0, 2, 4], dtype=torch.int32, device="cuda")
    with pytest.raises(mk.MuKVError) as e:
        g.retrieve(qt, offs, k_seg=1, k_frame=1)        # 2 questions > max_questions
    assert e.value.status == mk.MUKV_ERR_CAPACITY
    with pytest.raises(mk.MuKVError) as e:
        g.retrieve(qt, offs[:2], k_seg=1, k_frame=600)
    assert e.value.status == mk.MUKV_ERR_UNSUPPORTED
    torch.cuda.synchronize()
    g.close()


# ----------------------------------------------------- attention kernels and fp64 re-scoring --
@pytest.mark.parametrize("path", [mk.MUKV_ATT_GENERIC, mk.MUKV_ATT_MFMA])
@pytest.mark.parametrize("causal", [True, False])
def test_attention_paths_bf16(path, causal):
    w = W["7b"].scaled(n_frames=10, n_layers=2)
    p = Pair(w, seed=61, chunk=4, gpu_kw={"att_path": path, "causal": causal}, orc_kw={"causal": causal})
    p.ingest()
    p.check_compress()
    p.close()


@pytest.mark.parametrize("name,frames,kw", [
    # att_tile_kernel: frequency workgroups up to one and a half rounds of its places (13 a frame, 1536 places), and one frame more
    ("tiny", 177, {}), ("tiny", 178, {}),
    ("tiny", 27, {"tokens_per_frame": 196, "keep_ratio": 0.1}), ("tiny", 28, {"tokens_per_frame": 196, "keep_ratio": 0.1}),   # 14, 256
    ("7b", 45, {"n_layers": 1, "tokens_per_frame": 50}),                    # matrix-core attention of few frames, frequency beside it
    ("7b", 46, {"n_layers": 1, "tokens_per_frame": 50}),                    # more than 1280 (frame, head) pairs: two launches
    ("7b", 63, {"n_layers": 1, "tokens_per_frame": 50}),
    ("7b", 64, {"n_layers": 1, "tokens_per_frame": 50}),                    # of many: the indicator on the way
    ("7b", 1, {"n_layers": 1, "tokens_per_frame": 13}),                     # one wave a workgroup
])
def test_both_signals_of_a_chunk_in_one_launch(name, frames, kw):
    w = W[name].scaled(n_frames=frames, **kw)
    p = Pair(w, seed=121, chunk=frames)
    p.ingest()
    p.check_compress()
    p.close()


@pytest.mark.parametrize("dtype,D,hq,hkv,P,frames,causal", [
    ("f32", 128, 4, 2, 256, 3, True), ("f32", 128, 2, 1, 129, 2, False),     # the largest frame; past eight tiles
    ("f32", 64, 4, 1, 128, 130, True),                                       # eight tiles; a workgroup per head
    ("f32", 16, 4, 2, 17, 3, True), ("f32", 32, 2, 2, 16, 3, False),         # one past a tile, a tile
    ("bf16", 64, 14, 2, 241, 2, True), ("bf16", 64, 16, 4, 15, 40, True),    # 16 tiles with one token in the last; less than a tile
    ("bf16", 32, 6, 3, 113, 4, False), ("bf16", 16, 4, 1, 33, 5, True),
    ("bf16", 128, 4, 1, 209, 2, True),                                       # one token more than the 128-feature kernel takes
])
def test_fp32_attention_signal_at_the_edges_of_its_tiles(dtype, D, hq, hkv, P, frames, causal):
    w = W["tiny"].scaled(n_frames=frames, n_layers=1, n_q_heads=hq, n_kv_heads=hkv, head_dim=D, dtype=dtype, tokens_per_frame=P, keep_ratio=0.3)
    p = Pair(w, seed=122, chunk=frames, gpu_kw={"causal": causal}, orc_kw={"causal": causal})
    p.ingest()
    p.check_compress()
    p.close()


@pytest.mark.parametrize("P", [50, 16, 208, 7])
def test_mfma_ragged_token_counts(P):
    w = W["7b"].scaled(n_frames=5, n_layers=1, tokens_per_frame=P, keep_ratio=0.3, n_q_heads=8, n_kv_heads=2)
    p = Pair(w, seed=62 + P, chunk=3, gpu_kw={"att_path": mk.MUKV_ATT_MFMA})
    p.ingest()
    p.check_compress()
    p.close()


def test_mfma_whole_group_per_workgroup():
    # enough frames in one call that a workgroup loops over all heads of its KV group
    w = W["7b"].scaled(n_frames=152, n_layers=1)
    p = Pair(w, seed=63, chunk=152, gpu_kw={"att_path": mk.MUKV_ATT_MFMA})
    p.ingest()
    p.check_compress()
    p.close()


@pytest.mark.parametrize("name", ["tiny", "7b"])
def test_fp64_rescoring_of_every_frame(name):
    w = W[name].scaled(n_frames=6, n_layers=2)
    p = Pair(w, seed=64, chunk=4, gpu_kw={"refine_margin": 10.0})
    p.ingest()
    st = p.check_compress()
    assert int(st["refined"].sum()) == 6
    for so, sg in zip(p.sig_orc, p.sig_gpu):   # fp64 path: only the final float rounding differs
        assert np.abs(sg["fused"].cpu().numpy() - so["fused"]).max() <= 2e-7
    p.close()


def test_no_rescoring_when_disabled():
    w = W["tiny"].scaled(n_frames=6)
    p = Pair(w, seed=65, chunk=6, gpu_kw={"refine_margin": 0.0})
    p.ingest()
    st = p.check_compress()
    assert int(st["refined"].sum()) == 0
    p.close()


# ------------------------------------------------------------------ gathered (batched) chunks --
@pytest.mark.parametrize("name,frames,chunk,batch", [("7b", 21, 4, 3), ("tiny", 30, 4, 32), ("72b", 19, 8, 2)])
def test_batched_chunks_match_oracle(name, frames, chunk, batch):
    w = W[name].scaled(n_frames=frames, n_layers=2, n_questions=2)
    p = Pair(w, seed=71, chunk=chunk, gpu_kw={"batch_chunks": batch})
    p.ingest()
    p.check_compress()
    p.check_retrieve(questions_for(w, [16, 24], 500), mk.MUKV_SEMI, 2, 5, 0.3)
    p.close()


def test_batching_does_not_change_a_bit():
    w = W["7b"].scaled(n_frames=26, n_layers=2)
    ref = None
    for batch in (1, 2, 5):
        p = Pair(w, seed=72, chunk=4, gpu_kw={"batch_chunks": batch})
        p.ingest()
        st = p.check_compress()
        cur = {k: st[k].cpu().numpy() for k in ("kept_idx", "rep_frame_k", "rep_seg_k", "rep_patch_v", "margin")}
        cur["fused"] = torch.cat([sg["fused"] for sg in p.sig_gpu]).cpu().numpy()
        if ref is not None:
            for k in cur:
                np.testing.assert_array_equal(cur[k], ref[k], err_msg=f"{k} batch={batch}")
        ref = ref or cur
        p.close()


def test_batch_is_flushed_when_the_layout_changes():
    # the second chunk comes with other strides (a slice of a larger buffer): the gathered chunk
    # must be launched with its own strides first
    w = W["tiny"].scaled(n_frames=8, n_layers=2, n_kv_heads=2)
    p = Pair(w, seed=73, chunk=4, gpu_kw={"batch_chunks": 4})
    P = w.tokens_per_frame
    k, v, q = p.stream.next_chunk(8)
    kd, vd, qd = k.cuda(), v.cuda(), q.cuda()
    k0, v0, q0 = kd[:, :, : 4 * P].contiguous(), vd[:, :, : 4 * P].contiguous(), qd[:, : 4 * P].contiguous()
    p.sig_orc.append(p.orc.compress_chunk(np_view(k[:, :, : 4 * P]), np_view(v[:, :, : 4 * P]), q_last=np_view(q[:, : 4 * P])))
    p.sig_gpu.append(p.gpu.compress_chunk(k0, v0, q0, want_signals=True))
    p.sig_orc.append(p.orc.compress_chunk(np_view(k[:, :, 4 * P:]), np_view(v[:, :, 4 * P:]), q_last=np_view(q[:, 4 * P:])))
    p.sig_gpu.append(p.gpu.compress_chunk(kd[:, :, 4 * P:], vd[:, :, 4 * P:], qd[:, 4 * P:], want_signals=True))
    p.check_compress()
    p.close()


# ----------------------------------------- copies overlapped with the next batch's scoring ----
@pytest.mark.parametrize("name,frames,chunk,batch,margin", [("7b", 37, 4, 3, -1.0), ("tiny", 50, 4, 4, 10.0),
                                                            ("72b", 19, 8, 1, -1.0), ("tiny", 21, 4, 2, 0.0)])
def test_overlapped_copy_matches_oracle(name, frames, chunk, batch, margin):
    # every input stays alive in Pair.keep_alive, as the overlapped mode asks
    w = W[name].scaled(n_frames=frames, n_layers=2, n_questions=2)
    p = Pair(w, seed=74, chunk=chunk, gpu_kw={"batch_chunks": batch, "overlap_copy": 1, "refine_margin": margin})
    p.ingest()
    p.check_compress()
    p.check_retrieve(questions_for(w, [16, 24], 510), mk.MUKV_SEMI, 2, 5, 0.3)
    p.close()


def test_overlapped_copy_does_not_change_a_bit():
    w = W["7b"].scaled(n_frames=40, n_layers=3)
    ref = None
    for overlap in (0, 1):
        p = Pair(w, seed=75, chunk=4, gpu_kw={"batch_chunks": 2, "overlap_copy": overlap})
        p.ingest()
        st = p.check_compress()
        n = w.n_frames * p.gpu.kappa
        gk, gv = p.gpu.store_rows(0, n)
        cur = {k: st[k].cpu().numpy() for k in ("kept_idx", "rep_frame_k", "rep_seg_k", "rep_seg_v", "rep_patch_v", "margin")}
        cur["store_k"], cur["store_v"] = np_view(gk).copy(), np_view(gv).copy()
        if ref is not None:
            for k in cur:
                np.testing.assert_array_equal(cur[k], ref[k], err_msg=k)
        ref = ref or cur
        p.close()


def test_overlapped_copy_retrieve_without_flush_or_sync():
    # retrieve + gather right behind the last compress call, on the same stream, no host sync
    # in between: the library itself must order them after the copies still in flight
    w = W["7b"].scaled(n_frames=24, n_layers=2, n_questions=1)
    p = Pair(w, seed=76, chunk=8, gpu_kw={"batch_chunks": 1, "overlap_copy": 1})
    ks, vs, qs = [], [], []
    for _ in range(3):
        k, v, q = p.stream.next_chunk(8)
        p.orc.compress_chunk(np_view(k), np_view(v), q_last=np_view(q))
        ks.append(k.cuda()); vs.append(v.cuda()); qs.append(q.cuda())
    torch.cuda.synchronize()
    for k, v, q in zip(ks, vs, qs):
        p.gpu.compress_chunk(k, v, q)
    p.check_retrieve(questions_for(w, [32], 520), mk.MUKV_SEMI, 1, 6, 0.3)
    p.close()


# ------------------------------------------------------------- HIP graph replay, reset --------
@pytest.mark.parametrize("overlap,margin", [(1, 10.0), (1, -1.0), (0, 10.0)])
def test_graph_replay_matches_the_oracle_every_time(overlap, margin):
    # the whole path (gathered chunks, re-scoring chain on the side stream, put-off copy,
    # retrieve, gather) captured once and replayed: every replay, with eager work and host
    # synchronisation between them, must leave the oracle's results
    w = W["7b"].scaled(n_frames=28, n_layers=2, n_questions=1)
    p = Pair(w, seed=97, chunk=4, gpu_kw={"batch_chunks": 3, "overlap_copy": overlap, "refine_margin": margin})
    chunks = []
    for _ in range(7):
        k, v, q = p.stream.next_chunk(4)
        p.orc.compress_chunk(np_view(k), np_view(v), q_last=np_view(q))
        chunks.append((k.cuda(), v.cuda(), q.cuda()))
    qt = synth.random_question(w, 24, 530)
    qd = qt.cuda()
    offs = torch.tensor([0, 24], dtype=torch.int32, device="cuda")
    r_out = {"seg_idx": torch.empty(1, 2, dtype=torch.int32, device="cuda"),
             "seg_score": torch.empty(1, 2, dtype=torch.float32, device="cuda"),
             "frame_idx": torch.empty(1, 6, dtype=torch.int32, device="cuda"),
             "frame_score": torch.empty(1, 6, dtype=torch.float32, device="cuda")}
    shape = (1, w.n_layers, w.n_kv_heads, 6 * p.gpu.kappa, w.head_dim)
    g_out = (torch.empty(shape, dtype=w.torch_dtype, device="cuda"), torch.empty(shape, dtype=w.torch_dtype, device="cuda"),
             torch.empty(1, dtype=torch.int32, device="cuda"))

    gen = torch.Generator().manual_seed(531)   # two new tokens attend to the retrieved rows and five local rows (Eq. 9)
    q_new = torch.randn(1, 2, w.n_q_heads, w.head_dim, generator=gen).to(w.torch_dtype)
    k_loc = torch.randn(5, w.n_kv_heads, w.head_dim, generator=gen).to(w.torch_dtype)
    v_loc = torch.randn(5, w.n_kv_heads, w.head_dim, generator=gen).to(w.torch_dtype)
    q_new_d, k_loc_d, v_loc_d = q_new.cuda(), k_loc.cuda(), v_loc.cuda()
    l_off = torch.tensor([0, 5], dtype=torch.int32, device="cuda")
    a_out = torch.empty_like(q_new_d)

    def step(chs):
        p.gpu.reset()
        for k, v, q in chs:
            p.gpu.compress_chunk(k, v, q)
        p.gpu.retrieve(qd, offs, mode=mk.MUKV_SEMI, k_seg=2, k_frame=6, lambda_frame=0.3, out=r_out)
        p.gpu.gather_kv(r_out["frame_idx"], out=g_out)
        p.gpu.attend(1, q_new_d, r_out["frame_idx"], k_loc_d, v_loc_d, l_off, True, out=a_out)

    junk_stream = synth.SynthStream(w, 197, device="cuda")
    junk = [junk_stream.next_chunk(4) for _ in range(7)]
    step(chunks)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step(chunks)
    torch.cuda.synchronize()
    want = p.orc.retrieve(np_view(qt), orc.RetrieveParams(orc.SEMI, 2, 6, 0.3))
    ko, vo, n_tok = p.orc.gather(want["frame_idx"])
    a_want = p.orc.attend(1, np_view(q_new[0]), want["frame_idx"], np_view(k_loc), np_view(v_loc), True)
    for replay in range(3):
        step(junk)                           # eager work between the replays: another stream through
        for t in r_out.values():             # the same context, so cache and outputs hold other values
            t.fill_(-7)
        g_out[0].zero_()
        a_out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        st = p.gpu.state()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(st["kept_idx"].cpu().numpy(), p.orc.kept, err_msg=f"replay {replay}")
        np.testing.assert_array_equal(st["rep_seg_k"].cpu().numpy(), p.orc.seg_reps(which="k").astype(np.float32))
        np.testing.assert_array_equal(r_out["frame_idx"][0].cpu().numpy(), want["frame_idx"])
        np.testing.assert_array_equal(r_out["seg_idx"][0].cpu().numpy(), want["seg_idx"])
        assert int(g_out[2][0]) == n_tok
        np.testing.assert_array_equal(np_view(g_out[0][0]), ko)
        np.testing.assert_array_equal(np_view(g_out[1][0]), vo)
        assert out_err(to_f64(np_view(a_out[0].cpu())), a_want) <= 2e-2
        if margin > 1.0:
            assert int(st["refined"].sum()) == 28
    p.close()


def test_reset_drops_a_copy_that_was_put_off():
    # a stream is abandoned with its last batch's copy (and re-scoring) still put off; the next
    # stream through the same context must come out as if the context were new
    w = W["7b"].scaled(n_frames=12, n_layers=2)
    p = Pair(w, seed=98, chunk=4, gpu_kw={"batch_chunks": 1, "overlap_copy": 1, "refine_margin": 10.0})
    junk = synth.SynthStream(w, 99, device="cpu")
    for _ in range(2):
        k, v, q = junk.next_chunk(4)
        kd, vd, qd = k.cuda(), v.cuda(), q.cuda()
        p.keep_alive += [kd, vd, qd]
        p.gpu.compress_chunk(kd, vd, qd)
    p.gpu.reset()
    p.ingest()
    st = p.check_compress()
    assert int(st["refined"].sum()) == 12
    p.close()


@pytest.mark.parametrize("how", ["reset", "restore"])
def test_attention_after_the_cache_was_emptied_or_replaced(how):
    # decode steps whose rows workgroups share count arrivals in the context; the first one after a reset or a restore clears the
    # counts, eager or as part of a graph, and short prefills go on beside it
    w = W["7b"].scaled(n_frames=24, n_layers=1, n_questions=1)
    p = Pair(w, seed=99, chunk=8)
    junk = synth.SynthStream(w, 100, device="cpu")
    fi = torch.arange(8, dtype=torch.int32, device="cuda")[None]
    q = torch.randn(1, 1, w.n_q_heads, w.head_dim, device="cuda", generator=torch.Generator("cuda").manual_seed(101)).to(w.torch_dtype)
    if how == "restore":
        p.ingest()
        snap = p.gpu.snapshot()
        p.gpu.reset()
    k, v, x = (t.cuda() for t in junk.next_chunk(8))
    p.gpu.compress_chunk(k, v, x)
    for _ in range(3):
        p.gpu.attend(0, q, fi)
    if how == "restore":
        p.gpu.restore(snap)
    else:
        p.gpu.reset()
        p.ingest()
    fi, out = torch.arange(24, dtype=torch.int32, device="cuda")[None], torch.empty_like(q)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):                                                   # the clearing launch is captured with it
        for _ in range(2):
            p.gpu.attend(0, q, fi, out=out)
    p.check_attend(0, 1, [list(range(24))], [30], causal=True, seed=102)
    p.check_prefill(0, 40, [[1, 5, 9]], [2], True, seed=103)
    want = p.gpu.attend(0, q, fi)
    for i in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want), i
        p.check_attend(0, 1, [list(range(20 + i))], [30], causal=True, seed=104 + i)
        p.check_prefill(0, 40, [[1, 5, 9]], [2], True, seed=107 + i)
    p.close()


# ----------------------------------------------------------- seeded sweep of small shapes ------
def _random_case(i):
    rng = np.random.default_rng(4000 + i)
    hkv = int(rng.choice([1, 2, 4, 8]))
    group = int(rng.choice([1, 2, 7]))
    d = int(rng.choice([16, 32, 64, 128]))
    while hkv * d > 1024:
        hkv //= 2
    dtype = str(rng.choice(["bf16", "f32"]))
    p_tok = int(rng.integers(3, 257)) if i % 3 else int(rng.choice([16, 64, 196, 208, 256]))
    s_pat = int(rng.integers(1, min(p_tok, 6) + 1))
    rho = float(rng.choice([0.1, 0.25, 0.5, 0.9, 1.0]))
    if int(np.floor(rho * p_tok + 1e-9)) < 1:
        rho = 1.0
    w = synth.Workload(f"case{i}", int(rng.integers(1, 4)), hkv * group, hkv, d, dtype, int(rng.integers(3, 30)), p_tok,
                       int(rng.choice([1, 3, 8])), superpatches_per_frame=s_pat, chunk_frames=int(rng.integers(1, 7)),
                       spike_prob=float(rng.choice([0.0, 0.1])), keep_ratio=rho, alpha=float(rng.choice([0.0, 0.3, 0.7, 1.0])),
                       lambda_frame=float(rng.choice([0.0, 0.3, 0.8])), k_seg=int(rng.integers(1, 5)),
                       k_frame=int(rng.integers(1, 9)), question_tokens=int(rng.integers(1, 40)), n_questions=3)
    kw = {"causal": bool(rng.integers(0, 2)), "batch_chunks": int(rng.choice([1, 3])), "overlap_copy": int(rng.integers(0, 2)),
          "refine_margin": float(rng.choice([-1.0, 0.0, 10.0]))}
    if i % 6 == 5:   # the other reading of the transform's axis
        kw["freq_axis"] = mk.MUKV_FREQ_TOKEN
    return w, kw


@pytest.mark.parametrize("i", range(48))
def test_seeded_sweep_of_small_shapes(i):
    # shapes nobody picked by hand: head counts and groups, every head size, odd token counts,
    # super-patch counts, keep ratios, signal mixes, masks, chunkings, launch modes
    w, kw = _random_case(i)
    token_axis = kw.get("freq_axis", mk.MUKV_FREQ_FEATURE) == mk.MUKV_FREQ_TOKEN
    p = Pair(w, seed=5000 + i, chunk=w.chunk_frames, gpu_kw=dict(kw),
             orc_kw={"causal": kw["causal"], "freq_axis": orc.TOKEN_AXIS if token_axis else orc.FEATURE_AXIS})
    p.ingest()
    p.check_compress(raw_signals=not token_axis)   # the token-axis signal grows with P: only its fused form has an absolute bar
    qs = questions_for(w, [w.question_tokens, 1, 7], 800 + i)
    for mode in (mk.MUKV_SEMI, mk.MUKV_HIER, mk.MUKV_PARALLEL):
        p.check_retrieve(qs, mode, w.k_seg, w.k_frame, w.lambda_frame)
    p.check_retrieve(qs, mk.MUKV_SEMI, w.k_seg, w.k_frame, w.lambda_frame, n_visible=max(1, w.n_frames - 2))
    p.check_retrieve_patches(qs, (mk.MUKV_SEMI, mk.MUKV_HIER, mk.MUKV_PARALLEL)[i % 3], w.k_seg, w.k_frame + 3, w.lambda_frame)
    out, _ = p.check_retrieve(qs, mk.MUKV_SEMI, w.k_seg, w.k_frame, w.lambda_frame)
    idx = [[int(x) for x in row] for row in out["frame_idx"].cpu().numpy()]
    p.check_attend(i % w.n_layers, 1 + i % 5, idx, [1 + i % 5 + (3 * i + b) % 9 for b in range(3)], causal=bool(i % 2), seed=i)
    # the prefill of a few frames' worth of new tokens over the same retrieved frames, behind 0..8 older rows
    p.check_prefill((i + 1) % w.n_layers, (1 + i % 3) * w.tokens_per_frame + i % 2, idx, [(5 * i + 3 * b) % 9 for b in range(3)],
                    causal=bool((i // 2) % 2), seed=900 + i)
    p.close()


# -------------------------------------------------------- super-patch level of the search -----
@pytest.mark.parametrize("name,frames,kw", [("tiny", 32, {}), ("7b", 21, {"n_layers": 2}),
                                            ("72b", 19, {"n_layers": 2}),               # kappa 8 of 64: empty super-patches
                                            ("tiny", 40, {"superpatches_per_frame": 7, "keep_ratio": 0.1})])
def test_super_patch_retrieval_and_gather(name, frames, kw):
    w = W[name].scaled(n_frames=frames, n_questions=3, **kw)
    p = Pair(w, seed=120, chunk=8)
    p.ingest()
    p.check_compress()
    qs = questions_for(w, [w.question_tokens, 3, 20], 900)
    for mode in (mk.MUKV_SEMI, mk.MUKV_HIER, mk.MUKV_PARALLEL):
        p.check_retrieve_patches(qs, mode, 2, 9, 0.3)
    p.check_retrieve_patches(qs, mk.MUKV_SEMI, 2, 9, 0.0)
    p.check_retrieve_patches(qs, mk.MUKV_SEMI, 3, 200, 0.5, n_visible=frames - 5)   # more asked for than exist
    p.check_retrieve(qs, mk.MUKV_SEMI, 2, 5, 0.3)                                    # the frame level is untouched
    p.close()


def test_super_patch_level_with_many_questions():
    # 16 and more questions: the fp64 matrix-core scoring over the super-patch table
    w = W["7b"].scaled(n_frames=37, n_layers=2, n_questions=20)
    p = Pair(w, seed=121, chunk=8)
    p.ingest()
    qs = questions_for(w, [4 + (5 * i) % 30 for i in range(20)], 950)
    p.check_retrieve_patches(qs, mk.MUKV_SEMI, 2, 12, 0.3)
    p.check_retrieve_patches(qs, mk.MUKV_HIER, 2, 12, 0.3, n_visible=30)
    p.close()


@pytest.mark.parametrize("name,frames,kw", [("tiny", 32, {}), ("7b", 40, {"n_layers": 2}), ("72b", 70, {"n_layers": 2})])
def test_combined_gather_over_the_three_levels(name, frames, kw):
    w = W[name].scaled(n_frames=frames, n_questions=2, **kw)
    p = Pair(w, seed=130, chunk=8)
    p.ingest()
    S, F = w.superpatches_per_frame, w.frames_per_segment
    # overlapping choices at all levels, invalid entries, one question with almost nothing
    segs = [[1, -1, 0], [-1, -1, 99]]
    frms = [[F + 1, frames - 1, 3, -1], [2, 2, -1, frames + 5]]
    pats = [[S * 3 + 1, S * (frames - 2) + S - 1, S * (F + 1), -1, S * 5 + 0], [S * 2 + 1, -1, S * frames + 3, 7 * S, 7 * S + 1]]
    p.check_gather_union(segs, frms, pats)
    p.check_gather_union(None, frms, None)
    p.check_gather_union(segs, None, None)
    p.check_gather_union(None, None, pats)
    p.check_gather_union(segs, frms, pats, rows_cap=3 * p.gpu.kappa + 1)       # too small: first rows only, full count
    # fed by the searches themselves
    qs = questions_for(w, [w.question_tokens, 5], 970)
    out, _ = p.check_retrieve(qs, mk.MUKV_SEMI, 2, 4, 0.3)
    pout, _ = p.check_retrieve_patches(qs, mk.MUKV_SEMI, 2, 6, 0.3)
    p.check_gather_union(out["seg_idx"].cpu().tolist(), out["frame_idx"].cpu().tolist(), pout["patch_idx"].cpu().tolist())
    p.close()


@pytest.mark.parametrize("scale", [1e-3, 30.0, 300.0])
@pytest.mark.parametrize("name", ["7b", "tiny"])
def test_extreme_input_magnitudes(name, scale):
    # logits far outside the comfortable range: near-uniform and near-one-hot softmax rows
    w = W[name].scaled(n_frames=12, n_layers=2, n_questions=2)
    p = Pair(w, seed=140, chunk=4, gpu_kw={"batch_chunks": 2})
    for _ in range(3):
        k, v, q = p.stream.next_chunk(4)
        k, v, q = (k.float() * scale).to(k.dtype), (v.float() * scale).to(v.dtype), (q.float() * scale).to(q.dtype)
        kd, vd, qd = k.cuda(), v.cuda(), q.cuda()
        p.keep_alive += [kd, vd, qd]
        p.sig_orc.append(p.orc.compress_chunk(np_view(k), np_view(v), q_last=np_view(q)))
        p.sig_gpu.append(p.gpu.compress_chunk(kd, vd, qd, want_signals=True))
    p.check_compress(exact_reps=True, raw_signals=False)   # the fused, normalised scores keep the absolute bar
    qs = [synth.random_question(w, 9, 990) * scale, synth.random_question(w, 20, 991)]
    qs = [x.to(w.torch_dtype) for x in qs]
    p.check_retrieve(qs, mk.MUKV_SEMI, 2, 4, 0.3)
    p.close()


@pytest.mark.parametrize("name,frames,nq", [("7b", 45, 5), ("tiny", 61, 20), ("72b", 40, 17)])
def test_questions_with_their_own_timestamps(name, frames, nq):
    # one call, every question at another time: before the first segment ends, on a segment
    # boundary, inside a segment, at the end, "everything" (-1); fewer than 16 and 16+ questions
    w = W[name].scaled(n_frames=frames, n_layers=2, n_questions=nq)
    p = Pair(w, seed=150, chunk=8)
    p.ingest()
    F = w.frames_per_segment
    base = [3, F, F + 1, 2 * F, frames - 1, frames, -1, 1, 2 * F + F // 2]
    nvs = [base[i % len(base)] if base[i % len(base)] <= frames else frames for i in range(nq)]
    qs = questions_for(w, [4 + (3 * i) % 25 for i in range(nq)], 1000)
    for mode in (mk.MUKV_SEMI, mk.MUKV_HIER, mk.MUKV_PARALLEL):
        p.check_retrieve_at(qs, nvs, "frame", mode, 2, 5)
        p.check_retrieve_at(qs, nvs, "patch", mode, 2, 7)
    p.close()


def test_outputs_stay_inside_their_buffers():
    # every output sits between guard words; the calls may not touch them
    w = W["7b"].scaled(n_frames=24, n_layers=2, n_questions=3)
    p = Pair(w, seed=160, chunk=8)
    p.ingest()
    g = p.gpu
    qs = questions_for(w, [8, 3, 20], 1100)
    offs = torch.tensor([0, 8, 11, 31], dtype=torch.int32, device="cuda")
    qt = torch.cat(qs).cuda().contiguous()
    GUARD = 64

    def guarded(n, dtype):
        buf = torch.full((n + 2 * GUARD,), -77, dtype=dtype, device="cuda")
        return buf, buf[GUARD:GUARD + n]

    def intact(buf):
        assert bool((buf[:GUARD] == -77).all()) and bool((buf[-GUARD:] == -77).all())

    bufs = {}
    out = {}
    for name, n, dt in (("seg_idx", 3 * 2, torch.int32), ("seg_score", 3 * 2, torch.float32),
                        ("frame_idx", 3 * 5, torch.int32), ("frame_score", 3 * 5, torch.float32)):
        bufs[name], view = guarded(n, dt)
        out[name] = view.view(3, -1)
    g.retrieve(qt, offs, mode=mk.MUKV_SEMI, k_seg=2, k_frame=5, out=out)
    pout = {}
    for name, n, dt in (("patch_idx", 3 * 7, torch.int32), ("patch_score", 3 * 7, torch.float32)):
        bufs[name], view = guarded(n, dt)
        pout[name] = view.view(3, -1)
    g.retrieve_patches(qt, offs, mode=mk.MUKV_SEMI, k_seg=2, k_patch=7, out=pout)
    L, Hkv, D, kap = w.n_layers, w.n_kv_heads, w.head_dim, g.kappa

    def kv_out(rows, tag):
        n = 3 * L * Hkv * rows * D
        bufs[tag + "k"], kview = guarded(n, w.torch_dtype)
        bufs[tag + "v"], vview = guarded(n, w.torch_dtype)
        bufs[tag + "n"], nview = guarded(3, torch.int32)
        return kview.view(3, L, Hkv, rows, D), vview.view(3, L, Hkv, rows, D), nview

    g.gather_kv(out["frame_idx"], out=kv_out(5 * kap, "g"))
    g.gather_patches(pout["patch_idx"], out=kv_out(7 * g.patch_cap, "p"))
    g.gather_union(out["seg_idx"], out["frame_idx"], pout["patch_idx"], rows_cap=3 * kap + 5, out=kv_out(3 * kap + 5, "u"))
    torch.cuda.synchronize()
    for b in bufs.values():
        intact(b)
    p.close()


# ------------------------------------------------------------------ snapshot of the cache ------
@pytest.mark.parametrize("name,first,rest,kw", [
    ("7b", 21, 19, {}),                                               # cut inside a segment
    ("tiny", 32, 13, {"batch_chunks": 4, "overlap_copy": 1}),          # cut on a segment boundary, copy put off
    ("72b", 7, 9, {"refine_margin": 10.0}),                            # every frame re-scored in fp64
])
def test_snapshot_resumes_a_stream_in_another_context(name, first, rest, kw):
    # ingest the first part, save, load into a fresh context that held something else, ingest
    # the rest there: tables, retrieval and gathers must equal the oracle's over the whole stream
    w = W[name].scaled(n_frames=first + rest, n_layers=2, n_questions=3)
    p = Pair(w, seed=170, chunk=4, gpu_kw=kw)
    p.ingest(first)
    snap = p.gpu.snapshot()
    assert snap.numel() == mk.mukv_snapshot_size(p.gpu.h)
    other = gpu_context(w, max_frames=first + rest, max_chunk_frames=4, **kw)
    junk = synth.SynthStream(w, 171, device="cpu")
    k, v, q = junk.next_chunk(4)
    held = [k.cuda(), v.cuda(), q.cuda()]
    other.compress_chunk(*held)
    other.restore(snap)
    assert other.n_frames == first
    # the same bytes come back out of the second context
    assert torch.equal(other.snapshot(), snap)
    p.gpu.close()
    p.gpu = other
    p.ingest(rest)
    p.check_compress()
    qs = questions_for(w, [6, 17, 3], 1200)
    p.check_retrieve(qs, mk.MUKV_SEMI, 2, 5, 0.3)
    p.check_retrieve_patches(qs, mk.MUKV_HIER, 2, 6)
    p.close()


def test_snapshot_argument_errors():
    w = W["tiny"].scaled(n_frames=8, n_layers=2)
    p = Pair(w, seed=172, chunk=4)
    p.ingest()
    snap = p.gpu.snapshot()
    small = torch.empty(snap.numel() - 1, dtype=torch.uint8)
    with pytest.raises(mk.MuKVError) as e:
        mk.mukv_snapshot_save(p.gpu.h, small.data_ptr(), small.numel(), None)
    assert e.value.status == mk.MUKV_ERR_CAPACITY
    with pytest.raises(mk.MuKVError) as e:      # truncated
        mk.mukv_snapshot_load(p.gpu.h, snap.data_ptr(), snap.numel() - 1, None)
    assert e.value.status == mk.MUKV_ERR_INVALID_ARG
    bad = snap.clone()
    bad[0] ^= 0xFF
    with pytest.raises(mk.MuKVError) as e:      # not a snapshot
        p.gpu.restore(bad)
    assert e.value.status == mk.MUKV_ERR_INVALID_ARG
    other = gpu_context(w.scaled(n_layers=3), max_frames=8, max_chunk_frames=4)
    with pytest.raises(mk.MuKVError) as e:      # another configuration
        other.restore(snap)
    assert e.value.status == mk.MUKV_ERR_SHAPE
    tight = gpu_context(w, max_frames=4, max_chunk_frames=4)
    with pytest.raises(mk.MuKVError) as e:      # more frames than the context can hold
        tight.restore(snap)
    assert e.value.status == mk.MUKV_ERR_CAPACITY
    # failed loads left the first context as it was
    p.check_compress()
    other.close()
    tight.close()
    p.close()


# ------------------------------------------- attention over the retrieved context (Eq. 9) ------
@pytest.mark.parametrize("name,frames,kw", [("tiny", 20, {}), ("7b", 24, {"n_layers": 2}), ("72b", 16, {"n_layers": 2})])
def test_attention_over_retrieved_and_local_rows(name, frames, kw):
    w = W[name].scaled(n_frames=frames, n_questions=4, **kw)
    p = Pair(w, seed=180, chunk=4)
    p.ingest()
    idx = [[3, frames - 1, -1, 0, 7], [-1, -1, -1, -1, -1], [5, 5, 2, frames + 3, 9], [1, 2, 3, 4, 6]]  # skipped, doubled, out of range
    last = w.n_layers - 1
    p.check_attend(last, 1, idx, [1, 4, 9, 30], causal=True, seed=1)        # decode: one token, ragged local rows
    p.check_attend(0, 3, idx, [3, 5, 3, 17], causal=True, seed=2)           # layer 0, three tokens, causal among them
    p.check_attend(last, 3, idx, [3, 5, 3, 17], causal=False, seed=3)
    p.check_attend(last, 16, idx, [16, 20, 16, 40], causal=True, seed=4)    # the most tokens a call takes
    p.check_attend(last, 2, idx, None, seed=5)                              # no local rows; question 1 sees nothing: zeros
    p.check_attend(last, 5, None, [5, 8, 5, 6], causal=True, seed=6)        # no retrieved rows: plain causal self-attention
    p.check_attend(last, 4, idx, [2, 1, 0, 3], causal=True, seed=7)         # fewer local rows than tokens
    p.close()


def test_attention_over_long_contexts_and_many_questions():
    # 64 questions (a tile's rows unsplit, several blocks per wave) and one question (its rows split over workgroups);
    # many local rows
    w = W["7b"].scaled(n_frames=40, n_layers=2, n_questions=64)
    p = Pair(w, seed=181, chunk=8)
    p.ingest()
    rs = np.random.default_rng(5)
    idx = [[int(x) for x in rs.permutation(40)[:32]] for _ in range(64)]
    assert 32 * p.gpu.kappa > 512
    p.check_attend(1, 2, idx, [int(x) for x in rs.integers(2, 40, 64)], causal=True, seed=8)
    p.check_attend(1, 1, idx[:1], [700], causal=True, seed=9)
    p.check_attend(0, 1, [idx[0][:1]], [3], causal=True, seed=10)
    p.close()


@pytest.mark.parametrize("dtype,D,hq,hkv,n_q,B", [
    ("bf16", 128, 28, 4, 1, 1), ("bf16", 64, 16, 1, 3, 2), ("bf16", 16, 4, 2, 16, 4), ("f32", 128, 8, 8, 2, 3), ("f32", 32, 17, 1, 1, 4),
])
def test_attention_merged_by_the_last_of_a_tiles_workgroups(dtype, D, hq, hkv, n_q, B):
    # three to eight shares (two: the test after this), shares without rows among them; call after call, and replay after replay
    # with other calls between, the counts of arrivals are where they were
    w = W["tiny"].scaled(n_frames=40, n_questions=4, n_layers=1, n_q_heads=hq, n_kv_heads=hkv, head_dim=D, dtype=dtype, tokens_per_frame=49,
                         keep_ratio=0.5)
    p = Pair(w, seed=186, chunk=8)
    p.ingest()
    frames = [int(x) for x in np.random.default_rng(7).permutation(40)]
    for k in (5, 6, 8, 11, 14, 17, 22, 27, 33, 40):
        p.check_attend(0, n_q, [frames[:k]] * B, [n_q + 5 * b for b in range(B)], causal=bool(k % 2), seed=30 + k)
    p.check_attend(0, n_q, [[-1] * 33] * B, [n_q] * B, causal=True, seed=91)
    q = torch.randn(B, n_q, hq, D, device="cuda", generator=torch.Generator("cuda").manual_seed(92)).to(w.torch_dtype)
    fi = torch.tensor([frames] * B, dtype=torch.int32, device="cuda")
    want, out = p.gpu.attend(0, q, fi), torch.empty_like(q)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(3):
            p.gpu.attend(0, q, fi, out=out)
    for i in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want), i
        p.check_attend(0, n_q, [frames[:20 + i]] * B, [n_q] * B, causal=True, seed=93 + i)
    p.close()


@pytest.mark.parametrize("dtype,D,hq,hkv,n_q,B,k", [
    ("bf16", 128, 28, 4, 1, 32, 28),    # 128 tiles, two shares each: as many counts as there are
    ("f32", 128, 8, 8, 2, 16, 9),
    ("bf16", 64, 16, 1, 16, 8, 30),     # 128 tiles of one KV head: sixteen a question
    ("bf16", 16, 4, 2, 1, 33, 40),      # 66 tiles, three shares
])
def test_attention_of_as_many_tiles_as_have_shared_rows(dtype, D, hq, hkv, n_q, B, k):
    w = W["tiny"].scaled(n_frames=40, n_questions=B, n_layers=1, n_q_heads=hq, n_kv_heads=hkv, head_dim=D, dtype=dtype, tokens_per_frame=49,
                         keep_ratio=0.5)
    p = Pair(w, seed=187, chunk=8)
    p.ingest()
    rs = np.random.default_rng(8)
    lists = [[int(x) for x in rs.permutation(40)[:k]] for _ in range(B)]
    for seed in (110, 111):
        p.check_attend(0, n_q, lists, [n_q + b % 5 for b in range(B)], causal=True, seed=seed)
    p.check_prefill(0, 20, [lists[0][:2]], [3], True, seed=112)
    p.check_attend(0, n_q, lists[:1], [n_q], causal=True, seed=113)
    p.close()


@pytest.mark.parametrize("dtype,D,hq,hkv,n_q", [
    ("bf16", 128, 14, 2, 1), ("bf16", 64, 16, 1, 1), ("bf16", 32, 17, 1, 2), ("bf16", 16, 4, 2, 5),     # queries short of,
    ("f32", 128, 28, 4, 1), ("f32", 64, 8, 2, 4), ("f32", 32, 6, 3, 16), ("f32", 16, 4, 1, 3),          # on and past a tile
])
def test_attention_at_the_edges_of_row_blocks_and_shares(dtype, D, hq, hkv, n_q):
    # blocks of 16 or 32 rows dealt to four waves, rows split over workgroups from 9 (fp32, 128 features) to 13 blocks on
    w = W["tiny"].scaled(n_frames=40, n_questions=4, n_layers=1, n_q_heads=hq, n_kv_heads=hkv, head_dim=D, dtype=dtype, tokens_per_frame=49,
                         keep_ratio=0.5)
    p = Pair(w, seed=183, chunk=8)
    p.ingest()
    kap = p.gpu.kappa
    assert kap == 24
    frames = [int(x) for x in np.random.default_rng(6).permutation(40)]
    for k, ends in ((0, (1, 15, 16, 17)), (1, (31, 32, 33, 65)), (5, (127, 128, 129, 161)), (26, (639, 640, 641, 672)), (40, (960, 992, 993, 1023))):
        lists = [frames[:k]] * 4 if k else None
        p.check_attend(0, n_q, lists, [n - k * kap for n in ends], causal=bool(k % 2), seed=20 + k)
    p.check_attend(0, n_q, [frames[:30] + [-1] * 6 + [40], [-1] * 37, [-1] * 36 + [3], frames[:37]], [0, 0, 2, 5], causal=True, seed=90)
    p.check_attend(0, n_q, [frames[:27]], [70], causal=True, seed=91)
    p.close()


def test_attention_follows_the_retrieval_without_a_gather():
    # the indices stay on the device between the two calls; extreme scores (near one-hot rows)
    w = W["7b"].scaled(n_frames=48, n_layers=2, n_questions=3)
    p = Pair(w, seed=182, chunk=8)
    p.ingest()
    qs = questions_for(w, [6, 11, 4], 1300)
    out, res = p.check_retrieve(qs, mk.MUKV_SEMI, 2, 6, 0.3)
    g = torch.Generator().manual_seed(3)
    q = (torch.randn(3, 1, w.n_q_heads, w.head_dim, generator=g) * 6).to(w.torch_dtype)
    got = p.gpu.attend(1, q.cuda(), out["frame_idx"])
    torch.cuda.synchronize()
    for b in range(3):
        want = p.orc.attend(1, np_view(q[b]), res[b]["frame_idx"])
        assert out_err(to_f64(np_view(got[b].cpu())), want) <= 2e-2
    p.close()


def test_attention_argument_errors():
    w = W["tiny"].scaled(n_frames=8, n_layers=2, n_questions=2)
    p = Pair(w, seed=183, chunk=4)
    p.ingest()
    g = p.gpu
    q = torch.zeros(2, 1, w.n_q_heads, w.head_dim, dtype=w.torch_dtype, device="cuda")
    idx = torch.zeros(2, 3, dtype=torch.int32, device="cuda")
    kl = torch.zeros(4, w.n_kv_heads, w.head_dim, dtype=w.torch_dtype, device="cuda")
    lo = torch.tensor([0, 2, 4], dtype=torch.int32, device="cuda")

    def status(fn):
        with pytest.raises(mk.MuKVError) as e:
            fn()
        return e.value.status

    assert status(lambda: g.attend(w.n_layers, q, idx)) == mk.MUKV_ERR_INVALID_ARG          # no such layer
    assert status(lambda: g.attend(0, q, idx, kl, None, lo)) == mk.MUKV_ERR_INVALID_ARG     # local rows given in part
    big = torch.zeros(2, 17, w.n_q_heads, w.head_dim, dtype=w.torch_dtype, device="cuda")
    assert status(lambda: g.attend(0, big, idx)) == mk.MUKV_ERR_UNSUPPORTED                 # more than 16 tokens
    three = torch.zeros(3, 1, w.n_q_heads, w.head_dim, dtype=w.torch_dtype, device="cuda")
    assert status(lambda: g.attend(0, three, None, kl, kl, lo)) == mk.MUKV_ERR_CAPACITY     # more questions than the context holds
    assert status(lambda: mk.mukv_attend(g.h, 0, q.data_ptr(), 1, None, 3, None, None, None, 2, 1, q.data_ptr(),
                                         None)) == mk.MUKV_ERR_INVALID_ARG                   # k_frame without a list
    p.close()


# --------------------------------- the token-axis reading of the frequency indicator (Eq. 2) ------
@pytest.mark.parametrize("name,frames,alpha,kw", [
    ("tiny", 24, 0.7, {}),
    ("tiny", 24, 0.0, {}),                                            # the signal alone: every mirror pair is an exact tie
    ("7b", 21, 0.7, {"batch_chunks": 2, "overlap_copy": 1}),          # P = 196 = 4 * 7 * 7
    ("7b", 12, 0.3, {"refine_margin": 10.0}),                         # every frame through the fp64 pass
    ("72b", 16, 0.5, {"batch_chunks": 4}),
])
def test_frequency_signal_along_the_token_axis(name, frames, alpha, kw):
    w = W[name].scaled(n_frames=frames, n_layers=2, n_questions=2, alpha=alpha)
    gkw = dict(kw, freq_axis=mk.MUKV_FREQ_TOKEN)
    p = Pair(w, seed=190, chunk=4, gpu_kw=gkw, orc_kw={"freq_axis": orc.TOKEN_AXIS})
    p.ingest()
    st = p.check_compress(raw_signals=False)      # the raw signal grows with P: its bar is relative, below
    for so, sg in zip(p.sig_orc, p.sig_gpu):
        got, want = sg["fft"].cpu().numpy(), so["fft"]
        assert np.abs(got - want).max() <= mk_tol(w) * max(1.0, float(np.abs(want).max()))
        np.testing.assert_array_equal(got[:, 1:], got[:, 1:][:, ::-1])      # mirror rows: the same bits
    if kw.get("refine_margin", 0) >= 10.0:
        assert int(st["refined"].sum()) == frames
    qs = questions_for(w, [7, 3], 1400)
    p.check_retrieve(qs, mk.MUKV_SEMI, 2, 4, 0.3)
    p.close()


def test_token_axis_signal_with_odd_token_counts():
    # P odd, P prime, P below one load batch: no row is its own mirror except row 0
    for i, P in enumerate((3, 7, 13, 97, 255)):
        w = synth.Workload(f"tok{P}", 1, 4, 2, 32, "f32" if i % 2 else "bf16", 6, P, 3, superpatches_per_frame=1 + i % 3,
                           keep_ratio=0.5, alpha=0.4, chunk_frames=3,
                           k_seg=1, k_frame=2, question_tokens=5, n_questions=1)
        p = Pair(w, seed=191 + i, chunk=3, gpu_kw={"freq_axis": mk.MUKV_FREQ_TOKEN}, orc_kw={"freq_axis": orc.TOKEN_AXIS})
        p.ingest()
        p.check_compress(raw_signals=False)
        p.close()


# ------------------------------------- a unit of several frames ranked as one (Sec. 3.3) -----
def _unit_workload(dtype, P, S, rho, alpha, units, **kw):
    base = dict(dtype=dtype, tokens_per_frame=P, superpatches_per_frame=S, keep_ratio=rho, alpha=alpha,
                n_frames=units, frames_per_segment=2, n_layers=2, n_kv_heads=2, n_q_heads=4, head_dim=32,
                spike_prob=0.05, k_seg=1, k_frame=2, n_questions=2)
    base.update(kw)
    return W["tiny"].scaled(**base)


@pytest.mark.parametrize("dtype,P,S,rho,alpha,units,chunk", [
    ("bf16", 6 * 49, 6, 0.8, 0.8, 7, 3),     # just above what the per-frame kernels take
    ("f32", 1000, 1, 0.5, 0.5, 4, 4),
    ("bf16", 2049, 7, 0.1, 1.0, 3, 2),       # the last thread's tokens are ragged
    ("f32", 3000, 32, 0.8, 0.0, 3, 1),       # frequency indicator alone
    ("bf16", 8192, 32, 0.8, 0.8, 2, 1),      # the largest unit
    ("bf16", 257, 257, 1.0, 0.5, 3, 3),      # everything kept, every token its own super-patch
])
def test_segment_ranked_as_one_unit(dtype, P, S, rho, alpha, units, chunk):
    w = _unit_workload(dtype, P, S, rho, alpha, units)
    p = Pair(w, seed=300 + P, chunk=chunk, with_q=False)
    p.ingest(att_seed=7000 + P)
    st = p.check_compress()
    print(f"unit of {P} tokens: kappa {p.orc.kappa}, re-scored {int(st['refined'].sum())} of {units}")
    # the cache behaves like any other downstream: retrieval over units, gather, attention
    qs = questions_for(w, [5, 9], 310)
    p.check_retrieve(qs, mk.MUKV_SEMI, 1, 2, 0.3)
    p.check_retrieve_patches(qs, mk.MUKV_PARALLEL, 1, min(3, S * units), 0.3)
    p.check_attend(1, 3, [[0, units - 1], [units - 1, -1]], [4, 0], True, seed=311)
    p.close()


def test_segment_of_the_paper_as_one_unit():
    # 32 frames of 196 tokens, 80 % kept, frames as super-patches, 7B head layout
    w = _unit_workload("bf16", 32 * 196, 32, 0.8, 0.8, 3, n_kv_heads=4, n_q_heads=28, head_dim=128, frames_per_segment=1)
    p = Pair(w, seed=320, chunk=2, with_q=False)
    p.ingest(att_seed=7320)
    st = p.check_compress()
    assert p.orc.kappa == 5017
    p.check_attend(0, 2, [[2, 0]], [3], True, seed=321)
    p.close()


@pytest.mark.parametrize("kw", [{"refine_margin": 10.0}, {"batch_chunks": 2, "overlap_copy": 1},
                                {"batch_chunks": 3, "refine_margin": 10.0, "overlap_copy": 1}])
def test_large_units_with_rescoring_batching_and_overlapped_copy(kw):
    w = _unit_workload("bf16", 700, 4, 0.3, 0.6, 9)
    p = Pair(w, seed=330, chunk=2, with_q=False, gpu_kw=kw)
    p.ingest(att_seed=7330)
    st = p.check_compress()
    if kw.get("refine_margin", 0) > 1:
        assert int(st["refined"].sum()) == 9
    p.close()


@pytest.mark.parametrize("name,kw", [("tiny", {}), ("7b", {"n_layers": 2})])
@pytest.mark.parametrize("margin", [0.0, 10.0])                # ranked in fp32; every frame ranked again in fp64
def test_keep_of_a_frame_with_a_nan_key(name, kw, margin):
    # a NaN key leaves its token a NaN score beside finite ones (the attention signal is handed over): that token
    # ranks first, the others as their scores say, and no other frame notices -- kappa tokens per frame are kept, not
    # one more written over the next frame's
    w = W[name].scaled(n_frames=8, alpha=0.5, **kw)
    p = Pair(w, seed=345, chunk=8, with_q=False, gpu_kw={"refine_margin": margin})
    P = w.tokens_per_frame
    k, v, _ = synth.SynthStream(w, 345, device="cpu", with_q=False).next_chunk(8)
    att = synth.handed_over_attention(8, P, 346)
    p.orc.compress_chunk(np_view(k), np_view(v), att=att.numpy().astype(np.float64))
    f, t = 2, 5
    k[:, :, f * P + t] = float("nan")
    dev = [x.cuda() for x in (k, v, att)]
    sig = p.gpu.compress_chunk(dev[0], dev[1], att_signal=dev[2], want_signals=True)
    p.gpu.flush()
    st = p.gpu.state()
    torch.cuda.synchronize()
    kept, fused = st["kept_idx"].cpu().numpy(), sig["fused"].cpu().numpy()[f]
    assert int(st["refined"].sum()) == (8 if margin else 0)
    assert np.flatnonzero(np.isnan(fused)).tolist() == [t]
    first = np.argsort(-np.where(np.isnan(fused), np.inf, fused), kind="stable")[:p.orc.kappa]
    np.testing.assert_array_equal(kept[f], np.sort(first))
    others = [i for i in range(8) if i != f]
    np.testing.assert_array_equal(kept[others], p.orc.kept[others])
    p.close()


def test_rescoring_beside_a_long_copy_and_before_a_short_one():
    # 26 frames are 274 MB of rows in and out (fp64 chain on the side stream, its rows copied by itself), the 4 of the
    # last chunk 42 MB (everything on the caller's stream, one copy); every frame re-scored
    w = W["72b"].scaled(n_frames=30, n_layers=28, n_q_heads=8, tokens_per_frame=49, keep_ratio=0.95, n_questions=1)
    assert w.n_kv_heads == 8 and w.head_dim == 128 and 4 * 26 * 46 * 28 * 8 * 128 * 2 > 256 * 2**20
    p = Pair(w, seed=340, chunk=26, gpu_kw={"refine_margin": 10.0})
    p.ingest()
    st = p.check_compress()
    assert int(st["refined"].sum()) == 30
    p.close()


def test_large_unit_argument_errors():
    w = _unit_workload("bf16", 512, 2, 0.5, 0.5, 2)
    with pytest.raises(mk.MuKVError) as e:                   # the token-axis indicator is per frame
        gpu_context(w, freq_axis=mk.MUKV_FREQ_TOKEN)
    assert e.value.status == mk.MUKV_ERR_UNSUPPORTED
    with pytest.raises(mk.MuKVError) as e:
        gpu_context(_unit_workload("bf16", 8193, 1, 0.5, 0.5, 2))
    assert e.value.status == mk.MUKV_ERR_UNSUPPORTED
    g = gpu_context(w)
    k, v, q = synth.SynthStream(w, 1).next_chunk(1)
    with pytest.raises(mk.MuKVError) as e:                   # the attention signal has to be handed over
        g.compress_chunk(k.cuda(), v.cuda(), q.cuda())
    assert e.value.status == mk.MUKV_ERR_UNSUPPORTED
    assert g.state()["n_frames"] == 0
    g.close()


# --------------------- prefill of new tokens that also yields Eq. 1 (Sec. 3.2, Sec. 3.3) -----
@pytest.mark.parametrize("name,frames,kw,n_q,old", [
    ("tiny", 12, {}, 49, [0, 5]),                       # fp32 payload, one frame of new tokens
    ("7b", 10, {"n_layers": 2}, 196, [0, 3]),           # bf16, matrix-core scores, G = 7
    ("72b", 12, {"n_layers": 2}, 2 * 64 + 5, [7]),      # G = 8, ragged
    ("tiny", 6, {"head_dim": 16, "dtype": "bf16", "n_kv_heads": 2}, 30, [0, 1, 40]),   # bf16 rows of 16 features
])
def test_prefill_attention_and_received_signal(name, frames, kw, n_q, old):
    w = W[name].scaled(n_frames=frames, n_questions=len(old), **kw)
    p = Pair(w, seed=400, chunk=4)
    p.ingest()
    p.gpu.flush()
    fi = [[(3 * b + 1) % frames, -1, (5 * b + 2) % frames] for b in range(len(old))]
    for causal in (True, False):
        _, _, e_out, e_sig = p.check_prefill(w.n_layers - 1, n_q, fi, old, causal, seed=401)
        print(f"{name} n_q={n_q} causal={causal}: out err {e_out:.2e}, signal err {e_sig:.2e}")
    p.check_prefill(0, n_q, None, old, True, seed=402)   # no past cache at all
    p.close()


def test_prefill_of_a_long_unit_takes_unsplit_tiles():
    # enough 128-query tiles to fill the chip twice over, so that no tile's rows are shared (72B head layout: 8 KV heads x 8)
    w = W["72b"].scaled(n_frames=6, n_layers=1, n_questions=1)
    p = Pair(w, seed=440, chunk=3)
    p.ingest()
    n_q = 1100                                   # 8800 queries per KV head: 69 tiles x 8 heads >= 512 workgroups, ragged
    for causal in (True, False):
        _, _, e_out, e_sig = p.check_prefill(0, n_q, [[4, 0, -1]], [9], causal, seed=441)
        print(f"unsplit tiles, causal={causal}: out err {e_out:.2e}, signal err {e_sig:.2e}")
    p.close()


@pytest.mark.parametrize("D,hq,hkv,n_q,n_frames,old", [
    (64, 14, 2, 1, 3, [0]),             # one token, fewer rows than one step
    (64, 32, 8, 32, 9, [0, 31, 1]),     # 128 queries per KV head, a tile exactly; three questions (24 (question, head) pairs)
    (64, 10, 5, 65, 40, [3]),           # pairs that divide neither 8 nor are divided by it; several steps, shared rows
    (128, 28, 4, 18, 12, [0, 64]),      # 126 queries: two short of a tile
    (128, 28, 4, 19, 40, [200]),        # five past it; more steps than one set of row tables
    (128, 16, 2, 129, 2, [0]),          # one key past a key tile
    (128, 8, 8, 257, 0, [0]),           # one head per group, no past
])
def test_prefill_matrix_tile_edges(D, hq, hkv, n_q, n_frames, old):
    w = W["7b"].scaled(n_frames=max(n_frames, 4), n_layers=1, head_dim=D, n_q_heads=hq, n_kv_heads=hkv, n_questions=len(old))
    p = Pair(w, seed=450, chunk=4)
    p.ingest()
    fi = [[(7 * b + i) % n_frames for i in range(n_frames)] for b in range(len(old))] if n_frames else None
    for causal in (True, False):
        p.check_prefill(0, n_q, fi, old, causal, seed=451)
    p.close()


@pytest.mark.parametrize("D,hq,hkv,n_q,n_frames,old", [
    (128, 28, 4, 129, 8, [0]),          # nine steps of rows between two: one of them without rows
    (128, 28, 4, 129, 0, [0]),          # three steps: four waves a tile
    (128, 28, 4, 256, 0, [0]),          # four: two each; the first tile sees one step, so one of the two sees nothing
    (128, 16, 2, 147, 12, [0, 100]),    # tables filled twice, ragged rows
    (128, 64, 8, 512, 1, [1]),          # 256 tiles exactly
    (64, 32, 8, 161, 9, [31]),
    (64, 10, 5, 300, 3, [0, 7]),        # seven steps, ten (question, head) pairs
    (64, 10, 5, 300, 0, [0, 7]),        # five steps of 64 features: four waves a tile
    (128, 28, 4, 512, 0, [0]),          # eight steps, where the two begin
    (128, 64, 8, 528, 1, [1]),          # one tile more per KV head than there are places: the two smallest are a pair
    (64, 64, 8, 890, 0, [0]),           # 56 for 32: all but eight in pairs
    (64, 64, 8, 900, 0, [0]),           # 57: four waves a tile
    (128, 64, 8, 600, 17, [0]),         # 38 for 32 behind more rows than pairs are for: four waves a tile
    (128, 7, 1, 4700, 0, [0]),          # 258 tiles of one KV head
])
def test_prefill_tiles_whose_rows_two_halves_of_a_workgroup_share(D, hq, hkv, n_q, n_frames, old):
    w = W["7b"].scaled(n_frames=max(n_frames, 4), n_layers=1, head_dim=D, n_q_heads=hq, n_kv_heads=hkv, n_questions=len(old))
    p = Pair(w, seed=470, chunk=4)
    p.ingest()
    fi = [[(5 * b + i) % n_frames for i in range(n_frames)] for b in range(len(old))] if n_frames else None
    for causal in (True, False):
        p.check_prefill(0, n_q, fi, old, causal, seed=471)
    p.close()


@pytest.mark.parametrize("D,hq,hkv,n_q,B", [(128, 28, 4, 1, 1), (128, 28, 4, 128, 1), (64, 10, 5, 33, 3), (64, 128, 4, 127, 2), (128, 8, 8, 64, 4)])
def test_prefills_of_few_tokens_call_after_call_and_replay_after_replay(D, hq, hkv, n_q, B):
    # from one term of Eq. 1 a column to 128 of them; replay after replay with other calls between
    w = W["7b"].scaled(n_frames=4, n_layers=1, head_dim=D, n_q_heads=hq, n_kv_heads=hkv, n_questions=4)
    p = Pair(w, seed=480, chunk=4)
    p.ingest()
    for i, causal in enumerate((True, False, True)):
        p.check_prefill(0, n_q, [[(i + b) % 4] for b in range(B)], [3 * b for b in range(B)], causal, seed=481 + i)
    g = torch.Generator("cuda").manual_seed(485)
    q, k, v = (torch.randn(*shape, device="cuda", generator=g).to(w.torch_dtype) for shape in ((B, n_q, hq, D), (B * n_q, hkv, D), (B * n_q, hkv, D)))
    offs = torch.arange(B + 1, dtype=torch.int32, device="cuda") * n_q
    ws = torch.empty(mk.mukv_prefill_workspace_size(p.gpu.h, n_q, 0, B), dtype=torch.uint8, device="cuda")
    want, want_sig = p.gpu.prefill_attend(0, q, None, k, v, offs, workspace=ws)
    out, sig = torch.empty_like(want), torch.empty_like(want_sig)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(2):
            p.gpu.prefill_attend(0, q, None, k, v, offs, out=out, signal=sig, workspace=ws)
    for i in range(3):
        out.zero_(), sig.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want) and torch.equal(sig, want_sig), i
        p.check_prefill(0, n_q, [[b % 4] for b in range(4)], [0] * 4, True, seed=486 + i)
    p.close()


@pytest.mark.parametrize("D,hq,hkv,sizes", [(128, 28, 4, (128, 97)), (64, 32, 8, (33, 1)), (128, 8, 8, (64, 300))])
def test_prefills_that_overlap_each_with_a_workspace_of_its_own(D, hq, hkv, sizes):
    # what such a call writes is the caller's: on two streams at once the calls do not meet, and afterwards nothing is left behind
    w = W["7b"].scaled(n_frames=4, n_layers=1, head_dim=D, n_q_heads=hq, n_kv_heads=hkv, n_questions=1)
    p = Pair(w, seed=490, chunk=4)
    p.ingest()
    g = torch.Generator("cuda").manual_seed(491)
    calls = []
    for n_q in sizes:
        q, k, v = (torch.randn(*shape, device="cuda", generator=g).to(w.torch_dtype) for shape in ((1, n_q, hq, D), (n_q, hkv, D), (n_q, hkv, D)))
        offs = torch.tensor([0, n_q], dtype=torch.int32, device="cuda")
        ws = torch.empty(mk.mukv_prefill_workspace_size(p.gpu.h, n_q, 0, 1), dtype=torch.uint8, device="cuda")
        want = p.gpu.prefill_attend(0, q, None, k, v, offs, workspace=ws)
        outs = [(torch.zeros_like(want[0]), torch.zeros_like(want[1])) for _ in range(50)]
        calls.append((torch.cuda.Stream(), q, k, v, offs, ws, want, outs))
    torch.cuda.synchronize()
    for i in range(50):
        for st, q, k, v, offs, ws, _, outs in calls:
            with torch.cuda.stream(st):
                p.gpu.prefill_attend(0, q, None, k, v, offs, out=outs[i][0], signal=outs[i][1], workspace=ws)
    torch.cuda.synchronize()
    for _, _, _, _, _, _, want, outs in calls:
        for i, (out, sig) in enumerate(outs):
            assert torch.equal(out, want[0]) and torch.equal(sig, want[1]), i
    for n_q in sizes:
        p.check_prefill(0, n_q, [[1, 3]], [2], True, seed=492)
    p.check_attend(0, 1, [[0, 1, 2, 3]], [9], causal=True, seed=493)
    p.close()


@pytest.mark.parametrize("D,hq,hkv,n_q,n_frames,bad", [
    (128, 28, 4, 150, 8, 100),     # tiles in two halves: the first sees 411 rows, its halves walk 512
    (64, 32, 8, 161, 8, 100),
    (128, 28, 4, 1568, 4, 1000),   # this row's tile has a workgroup to itself, the smallest ones are in pairs
    (128, 28, 4, 1568, 4, 200),    # one of a pair's
    (128, 28, 4, 100, 0, 50),      # Eq. 1 summed by the attention itself
    (128, 14, 2, 160, 32, 50),     # the rows of a tile shared by workgroups
    (64, 64, 8, 1100, 0, 120),     # four waves a tile
])
def test_prefill_rows_that_no_query_of_a_tile_sees_do_not_reach_it(D, hq, hkv, n_q, n_frames, bad):
    w = W["7b"].scaled(n_frames=max(n_frames, 4), n_layers=1, head_dim=D, n_q_heads=hq, n_kv_heads=hkv, n_questions=1)
    p = Pair(w, seed=500, chunk=4)
    p.ingest()
    g = torch.Generator("cuda").manual_seed(501)
    q, k, v = (torch.randn(*shape, device="cuda", generator=g).to(w.torch_dtype) for shape in ((1, n_q, hq, D), (n_q, hkv, D), (n_q, hkv, D)))
    offs = torch.tensor([0, n_q], dtype=torch.int32, device="cuda")
    fi = torch.arange(n_frames, dtype=torch.int32, device="cuda")[None] if n_frames else None
    want, want_sig = p.gpu.prefill_attend(0, q, fi, k, v, offs)
    v[bad] = float("nan")
    out, sig = p.gpu.prefill_attend(0, q, fi, k, v, offs)
    G = hq // hkv
    at = torch.arange(n_q * G)                                                  # (token, head of the KV group)
    last = ((at // 128 * 128 + 127).clamp(max=n_q * G - 1) // G).view(n_q, G)   # last token of its tile
    apart = (last < bad).repeat(1, hkv).cuda()                                  # [n_q][hq]: the whole tile is before the row
    assert apart.any() and not apart.all()
    assert torch.equal(out[0][apart], want[0][apart])
    assert torch.isnan(out[0][bad:].float()).all()                              # who sees it gets it
    assert torch.equal(sig, want_sig)                                           # (weights do not depend on values)
    p.close()


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f32", 128), ("bf16", 64)])
def test_scores_of_any_finite_size(dtype, D):
    # scores of 1e12: every softmax is a choice of one row (two largest within the 1e-6 of a sum in fp32: none here), and
    # no weight may overflow on the rounding of the maximum
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    P, n, H = 49, 3, 4
    g = torch.Generator().manual_seed(461)
    k, v, q = ((torch.randn(*s, generator=g) * m).to(t) for s, m in
               (((1, H, n * P, D), 1e6), ((1, H, n * P, D), 1.0), ((H, n * P, D), 1e6)))
    ctx = mk.MuKV(n_layers=1, n_q_heads=H, n_kv_heads=H, head_dim=D, tokens_per_frame=P, frames_per_segment=8,
                  superpatches_per_frame=4, dtype=t, keep_ratio=0.25, max_frames=4, max_chunk_frames=4, max_questions=1)
    att = ctx.compress_chunk(k.cuda(), v.cuda(), q.cuda(), want_signals=True)["att"]
    ctx.flush()
    torch.cuda.synchronize()
    sc = torch.einsum("hfid,hfjd->hfij", q.double().view(H, n, P, D), k[0].double().view(H, n, P, D)) / D ** 0.5
    sc = sc.masked_fill(torch.triu(torch.ones(P, P, dtype=torch.bool), 1), -1e300).softmax(-1)
    assert (att.cpu().double() - sc.mean((0, 2))).abs().max() <= 1e-6
    qn = q[:, :2].transpose(0, 1).contiguous()[None]                           # [1][2][H][D]
    out = ctx.attend(0, qn.cuda(), None, k[0].transpose(0, 1).contiguous().cuda(), v[0].transpose(0, 1).contiguous().cuda(),
                     torch.tensor([0, n * P], dtype=torch.int32).cuda(), False)
    w = (torch.einsum("hid,hjd->hij", q[:, :2].double(), k[0].double()) / D ** 0.5).softmax(-1)
    want = torch.einsum("hij,hjd->ihd", w, v[0].double())
    assert (out[0].cpu().double() - want).abs().max() <= 1e-5
    ctx.close()


@pytest.mark.parametrize("dtype,D", [("f32", 16), ("f32", 64), ("f32", 128), ("bf16", 16), ("bf16", 32)])
@pytest.mark.parametrize("past", [0, 3])     # frames of 128 rows: rows unsplit, and (fp32) split over workgroups
def test_received_attention_of_scores_of_any_size(dtype, D, past):
    # without a mask the tokens' shares of a query's weights add up to one whatever the size of the scores (a past of scores of
    # zero has no weight beside them)
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    H, n = 3, 70
    ctx = mk.MuKV(n_layers=1, n_q_heads=H, n_kv_heads=H, head_dim=D, tokens_per_frame=128, frames_per_segment=8, alpha=0.0,
                  superpatches_per_frame=4, dtype=t, keep_ratio=1.0, max_frames=4, max_chunk_frames=4, max_questions=1)
    g = torch.Generator().manual_seed(464)
    if past:
        zero = torch.zeros(1, H, past * 128, D, dtype=t).cuda()
        ctx.compress_chunk(zero, zero)
    idx = torch.arange(past, dtype=torch.int32)[None].cuda() if past else None
    q0, k0 = torch.randn(1, n, H, D, generator=g), torch.randn(n, H, D, generator=g)
    k0[..., 0], q0[..., 0] = 4.0, 4.0 * D ** 0.5     # the first feature brings every score 16, the others 1 or so
    v, offs = torch.randn(n, H, D, generator=g).to(t).cuda(), torch.tensor([0, n], dtype=torch.int32).cuda()
    for size in (1e2, 1e4, 1e6, 3e7, 1e12, 1e30):
        q, k = (q0 * size ** 0.5).to(t).cuda(), (k0 * size ** 0.5).to(t).cuda()
        out, sig = ctx.prefill_attend(0, q, idx, k, v, offs, False)
        assert torch.isfinite(out).all()
        # a weight: the exponential within two ulps, its product with 1 / normaliser, sums of 70 and of 210 in fp32
        assert abs(float(sig.double().sum()) - 1.0) <= 1e-6, (size, float(sig.double().sum()))
        one = torch.tensor([0, 1], dtype=torch.int32).cuda()
        _, sig = ctx.prefill_attend(0, q[:, :1].contiguous(), idx, k[:1], v[:1], one, True)
        assert abs(float(sig) - 1.0) <= 5e-7, (size, float(sig))
    ctx.close()


@pytest.mark.parametrize("dtype,D", [("f32", 16), ("f32", 32), ("f32", 64), ("f32", 128), ("bf16", 16)])
def test_scores_finite_once_scaled(dtype, D):
    # q.k is past fp32 (5.4e38 .. 2e39), q.k log2(e) / sqrt(D) is not (2e38): one row, ten times the others, takes all the weight
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    H, n = 2, 40
    ctx = mk.MuKV(n_layers=1, n_q_heads=H, n_kv_heads=H, head_dim=D, tokens_per_frame=16, frames_per_segment=8,
                  superpatches_per_frame=4, dtype=t, keep_ratio=0.25, max_frames=4, max_chunk_frames=4, max_questions=1)
    q = torch.full((1, n, H, D), 2.0 ** 50)
    k = torch.full((n, H, D), 2e37 * D ** 0.5 / 1.4426950408889634 / D / 2.0 ** 50)
    k[7] *= 10
    v = torch.randn(n, H, D, generator=torch.Generator().manual_seed(463)).to(t)
    q, k, v, offs = q.to(t).cuda(), k.to(t).cuda(), v.cuda(), torch.tensor([0, n], dtype=torch.int32).cuda()
    out = ctx.attend(0, q[:, :2].contiguous(), None, k, v, offs, False)
    assert torch.equal(out[0], v[7].expand(2, H, D))
    out, _ = ctx.prefill_attend(0, q, None, k, v, offs, False)
    assert torch.equal(out[0], v[7].expand(n, H, D))
    ctx.close()


@pytest.mark.parametrize("D,hq,hkv,most", [(64, 16, 4, 1.2e-7), (128, 28, 4, 1.23e-7)])
def test_fp32_attention_stays_as_near_to_64_bits(D, hq, hkv, most):
    # 30 rows, 64 questions, mean relative distance: 1.15 / 1.17e-7 (D = 64 / 128, standard error 0.01).  Sums that join evenly
    # give 1.18 / 1.21, a block's 16 rows one after another and exponents rounded at their own size 1.26 / 1.28
    ctx = mk.MuKV(n_layers=1, n_q_heads=hq, n_kv_heads=hkv, head_dim=D, tokens_per_frame=16, frames_per_segment=8,
                  superpatches_per_frame=4, dtype=torch.float32, keep_ratio=0.25, max_frames=4, max_chunk_frames=4, max_questions=64)
    B, n = 64, 30
    g = torch.Generator().manual_seed(467)
    q = torch.randn(B, 1, hq, D, generator=g)
    k, v = torch.randn(B * n, hkv, D, generator=g), torch.randn(B * n, hkv, D, generator=g)
    out = ctx.attend(0, q.cuda(), None, k.cuda(), v.cuda(), (torch.arange(B + 1) * n).to(torch.int32).cuda(), True)
    kd, vd = (x.double().view(B, n, hkv, D).transpose(1, 2) for x in (k, v))
    w = (torch.matmul(q.double().view(B, hkv, hq // hkv, D), kd.transpose(2, 3)) / D ** 0.5).softmax(-1)
    want = torch.matmul(w, vd).view(B, hq * D)
    far = (out.cpu().double().view(B, hq * D) - want).norm(dim=1) / want.norm(dim=1)
    assert far.mean() <= most
    ctx.close()


@pytest.mark.parametrize("dtype,D,hq,hkv,n_q,n_frames,old", [
    ("f32", 128, 28, 4, 1, 2, [0]),           # one token: 7 queries of 16
    ("f32", 128, 28, 4, 65, 2, [0, 7]),       # a new token past 64; shares of a few tiles
    ("f32", 64, 14, 2, 16, 0, [5]),           # a wave's keys exactly
    ("f32", 32, 4, 4, 17, 1, [0, 0, 3]),      # one past it, one head per group: 17 queries
    ("f32", 16, 16, 1, 200, 2, [31]),         # one KV head: many shares
    ("bf16", 32, 64, 8, 150, 2, [0] * 43),    # so many questions (3 * 8 * 43 workgroups) that the queries are not shared
    ("bf16", 16, 14, 2, 63, 3, [1]),          # rows of two pieces
])
def test_prefill_column_sums_edges(dtype, D, hq, hkv, n_q, n_frames, old):
    w = W["7b"].scaled(n_frames=4, n_layers=1, dtype=dtype, head_dim=D, n_q_heads=hq, n_kv_heads=hkv, n_questions=len(old))
    p = Pair(w, seed=457, chunk=4)
    p.ingest()
    fi = [[(b + i) % 4 for i in range(n_frames)] for b in range(len(old))] if n_frames else None
    for causal in (True, False):
        p.check_prefill(0, n_q, fi, old, causal, seed=458)
    p.close()


@pytest.mark.parametrize("D,hq,hkv,n_q,n_frames,old", [
    (128, 28, 4, 31, 0, [0, 40]),       # 32 keys at a time and one less; behind older rows
    (128, 28, 4, 64, 0, [1]),           # the keys of 64 tokens lie across the last two steps of rows
    (128, 16, 2, 65, 1, [200, 0]),      # one more: some keys are no longer staged
    (64, 32, 8, 128, 0, [300]),         # as many as are summed here
    (128, 64, 8, 127, 2, [0, 0, 70, 5]),  # tiles fill the chip: one workgroup walks many rows
    (128, 8, 8, 128, 0, [3]),           # one head per group: a tile has as many tokens as queries
    (64, 14, 2, 2, 0, [0]),
])
def test_prefill_of_few_tokens_sums_attention_in_the_tile(D, hq, hkv, n_q, n_frames, old):
    w = W["7b"].scaled(n_frames=4, n_layers=1, head_dim=D, n_q_heads=hq, n_kv_heads=hkv, n_questions=len(old))
    p = Pair(w, seed=455, chunk=4)
    p.ingest()
    fi = [[(b + i) % 4 for i in range(n_frames)] for b in range(len(old))] if n_frames else None
    for causal in (True, False):
        p.check_prefill(0, n_q, fi, old, causal, seed=456)
    p.close()


@pytest.mark.parametrize("name,kw,n_q,n_frames", [
    ("7b", {}, 40, 0),                        # matrix-core prefill, rows of a tile in one workgroup
    ("7b", {}, 40, 12),                       # shared by several, merged
    ("7b", {}, 150, 0),                       # four waves a tile, Eq. 1 in a launch of its own
    ("7b", {}, 150, 12),                      # two halves of a workgroup that join: the key in the first one's rows
    ("7b", {}, 150, 11),                      # in the second one's
    ("7b", {"head_dim": 64}, 40, 0),
    ("7b", {"head_dim": 64}, 40, 12),
    ("7b", {"head_dim": 64}, 150, 12),
    ("7b", {"head_dim": 64}, 150, 11),
    ("7b", {"head_dim": 32}, 40, 5),          # scores on the matrix cores, merged
    ("tiny", {}, 40, 5),                      # fp32
    ("7b", {}, 3, 12),                        # decode
    ("tiny", {}, 3, 1),
])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_attention_non_finite_scores_reach_the_output(name, kw, n_q, n_frames, bad):
    # one new token's key holds a non-finite feature: a query that sees a NaN or +inf score has no softmax and gives
    # NaN (never the zeros of a query that sees nothing), a score of -inf is a weight of zero, and the tokens before
    # that key -- which the mask hides from them -- are as they would be without it.  The oracle does the same in fp64.
    w = W[name].scaled(n_frames=12, n_layers=1, n_questions=1, **kw)
    p = Pair(w, seed=460, chunk=4)
    p.ingest()
    gen = torch.Generator().manual_seed(461)
    q = torch.randn(1, n_q, w.n_q_heads, w.head_dim, generator=gen).to(w.torch_dtype)
    kl, vl = (torch.randn(n_q, w.n_kv_heads, w.head_dim, generator=gen).to(w.torch_dtype) for _ in range(2))
    j = n_q // 2
    kl[j] = 0
    kl[j, :, 0] = bad
    frames = [(5 * i) % 12 for i in range(n_frames)]
    fi = torch.tensor([frames], dtype=torch.int32, device="cuda") if frames else None
    offs = torch.tensor([0, n_q], dtype=torch.int32, device="cuda")
    with np.errstate(invalid="ignore"):
        want, want_sig = p.orc.prefill_attend(0, np_view(q[0]), frames, np_view(kl), np_view(vl), True)
    assert np.isnan(want[j:]).any() and np.isfinite(want[:j]).all() and np.isnan(want_sig[j])
    calls = [p.gpu.prefill_attend(0, q.cuda(), fi, kl.cuda(), vl.cuda(), offs, True)]
    if n_q <= 16:
        calls.append((p.gpu.attend(0, q.cuda(), fi, kl.cuda(), vl.cuda(), offs, True), None))
    torch.cuda.synchronize()
    for out, sig in calls:
        got = to_f64(np_view(out[0].cpu()))
        np.testing.assert_array_equal(np.isnan(got), np.isnan(want))
        fine = ~np.isnan(want)
        assert out_err(got[fine], want[fine]) <= mk_tol(w)
        assert sig is None or np.isnan(sig[0].cpu().numpy()[np.isnan(want_sig)]).all()
    p.close()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("n_q", [5, 40, 150, 450])      # (450: two halves of a workgroup, most of them without a row)
def test_prefill_rows_of_no_question_stay_out(D, n_q):
    # the last step of rows is part empty, one entry of the frame list names no frame, and there are no rows besides the
    # retrieved ones: what stands in for a row that is not there must not be a frame the question did not retrieve --
    # zero times its NaN is NaN.  Frame 0 has NaN values.
    w = W["7b"].scaled(n_frames=8, n_layers=1, head_dim=D, n_questions=1, tokens_per_frame=50)
    p = Pair(w, seed=465, chunk=4)
    k, v, q = synth.SynthStream(w, 465, device="cpu").next_chunk(8)
    v[:, :, :w.tokens_per_frame] = float("nan")
    for c in range(2):
        kc, vc, qc = (x[:, c * 200:(c + 1) * 200] if x.dim() == 3 else x[:, :, c * 200:(c + 1) * 200] for x in (k, v, q))
        p.orc.compress_chunk(np_view(kc.contiguous()), np_view(vc.contiguous()), q_last=np_view(qc.contiguous()))
        dev = [x.contiguous().cuda() for x in (kc, vc, qc)]
        p.keep_alive += dev
        p.gpu.compress_chunk(*dev)
    assert (3 * p.orc.kappa) % 64
    gen = torch.Generator().manual_seed(466)
    q_new = torch.randn(1, n_q, w.n_q_heads, D, generator=gen).to(w.torch_dtype)
    row = torch.zeros(1, w.n_kv_heads, D, dtype=w.torch_dtype, device="cuda")       # (not one of the question's: it has none)
    fi = torch.tensor([[-1, 5, 1]], dtype=torch.int32, device="cuda")
    out, sig = p.gpu.prefill_attend(0, q_new.cuda(), fi, row, row, torch.tensor([0, 0], dtype=torch.int32, device="cuda"), True)
    torch.cuda.synchronize()
    assert out_err(to_f64(np_view(out[0].cpu())), p.orc.attend(0, np_view(q_new[0]), [5, 1])) <= mk_tol(w)
    assert not sig.any()
    p.close()


def test_prefill_signal_feeds_the_compression():
    # one stream, chunk by chunk: prefill of the chunk's tokens over frames already in the cache -> its
    # signal, handed to mukv_compress_chunk.  The oracle is given the same float32 signal, so the keep
    # must agree bit for bit; the signal itself is checked against the oracle's within 1e-5.
    w = W["7b"].scaled(n_frames=12, n_layers=2)
    P, chunk = w.tokens_per_frame, 2
    p = Pair(w, seed=410, chunk=chunk)
    ls = w.n_layers - 1
    for c0 in range(0, w.n_frames, chunk):
        k, v, q = p.stream.next_chunk(chunk)
        past = [[f for f in (c0 - 1, c0 - 4) if f >= 0] + [-1] * 2][0][:2]
        ql = q.transpose(0, 1).contiguous()                       # [n][Hq][D]
        kl, vl = k[ls].transpose(0, 1).contiguous(), v[ls].transpose(0, 1).contiguous()
        offs = torch.tensor([0, chunk * P], dtype=torch.int32).cuda()
        fi = torch.tensor([past], dtype=torch.int32).cuda()
        _, sig = p.gpu.prefill_attend(ls, ql[None].cuda(), fi, kl.cuda(), vl.cuda(), offs, True)
        torch.cuda.synchronize()
        _, want = p.orc.prefill_attend(ls, np_view(ql), past, np_view(kl), np_view(vl), True)
        assert np.abs(sig[0].cpu().numpy() - want).max() <= 1e-5
        att = sig.reshape(chunk, P).contiguous()
        kd, vd = k.cuda(), v.cuda()
        p.keep_alive += [kd, vd, att]
        p.sig_orc.append(p.orc.compress_chunk(np_view(k), np_view(v), att=att.cpu().numpy().astype(np.float64)))
        p.sig_gpu.append(p.gpu.compress_chunk(kd, vd, att_signal=att, want_signals=True))
    p.check_compress()
    p.close()


def test_prefill_argument_errors():
    w = W["tiny"].scaled(n_frames=4)
    p = Pair(w, seed=420, chunk=4)
    p.ingest()
    g = p.gpu
    q = torch.zeros(1, 8, w.n_q_heads, w.head_dim, device="cuda")
    kl = torch.zeros(8, w.n_kv_heads, w.head_dim, device="cuda")
    offs = torch.tensor([0, 8], dtype=torch.int32, device="cuda")
    need = mk.mukv_prefill_workspace_size(g.h, 8, 0, 1)
    assert need > 0
    small = torch.empty(need - 4, dtype=torch.uint8, device="cuda")
    out, sig = torch.empty_like(q), torch.empty(1, 8, device="cuda")
    with pytest.raises(mk.MuKVError) as e:
        mk.mukv_prefill_attend(g.h, 0, q.data_ptr(), 8, None, 0, kl.data_ptr(), kl.data_ptr(), offs.data_ptr(), 1, 1,
                               out.data_ptr(), sig.data_ptr(), small.data_ptr(), small.numel(), None)
    assert e.value.status == mk.MUKV_ERR_CAPACITY
    with pytest.raises(mk.MuKVError) as e:      # the new tokens are local rows: they cannot be left out
        mk.mukv_prefill_attend(g.h, 0, q.data_ptr(), 8, None, 0, None, None, None, 1, 1, out.data_ptr(), sig.data_ptr(),
                               small.data_ptr(), need, None)
    assert e.value.status == mk.MUKV_ERR_INVALID_ARG
    with pytest.raises(mk.MuKVError) as e:
        mk.mukv_prefill_workspace_size(g.h, 8193, 0, 1)
    assert e.value.status == mk.MUKV_ERR_UNSUPPORTED
    p.close()


def test_large_units_snapshot_and_graph_replay_with_prefill():
    # units of 600 tokens: snapshot / restore in the middle of the stream; then the whole step -- reset, chunks with
    # the signal handed over (batched, copy put off, every unit re-scored), retrieval, prefill attention over
    # the retrieved units -- captured once and replayed with other work in between
    w = _unit_workload("bf16", 600, 3, 0.4, 0.7, 8, head_dim=128, n_kv_heads=2, n_q_heads=4)
    kw = {"batch_chunks": 2, "overlap_copy": 1, "refine_margin": 10.0}
    p = Pair(w, seed=340, chunk=2, with_q=False, gpu_kw=kw)
    p.ingest(4, att_seed=7340)
    snap = p.gpu.snapshot()
    other = gpu_context(w, max_frames=8, max_chunk_frames=2, **kw)
    other.restore(snap)
    assert torch.equal(other.snapshot(), snap)
    p.gpu.close()
    p.gpu = other
    p.ingest(4, att_seed=7340)
    p.check_compress()

    P = w.tokens_per_frame
    chunks = []
    st2 = synth.SynthStream(w, 340, device="cpu", with_q=False)      # the same stream again, for the captured step
    for c in range(4):
        k, v, _ = st2.next_chunk(2)
        att = synth.handed_over_attention(2, P, 7340 + 2 * c)
        chunks.append((k.cuda(), v.cuda(), att.cuda()))
    qt = synth.random_question(w, 9, 345)
    qd, offs = qt.cuda(), torch.tensor([0, 9], dtype=torch.int32, device="cuda")
    r_out = {"seg_idx": torch.empty(1, 1, dtype=torch.int32, device="cuda"), "seg_score": torch.empty(1, 1, device="cuda"),
             "frame_idx": torch.empty(1, 2, dtype=torch.int32, device="cuda"), "frame_score": torch.empty(1, 2, device="cuda")}
    gen = torch.Generator().manual_seed(346)
    n_q = 70
    q_new = torch.randn(1, n_q, w.n_q_heads, w.head_dim, generator=gen).to(w.torch_dtype)
    k_loc = torch.randn(n_q + 3, w.n_kv_heads, w.head_dim, generator=gen).to(w.torch_dtype)
    v_loc = torch.randn(n_q + 3, w.n_kv_heads, w.head_dim, generator=gen).to(w.torch_dtype)
    q_d, k_d, v_d = q_new.cuda(), k_loc.cuda(), v_loc.cuda()
    l_off = torch.tensor([0, n_q + 3], dtype=torch.int32, device="cuda")
    ws = torch.empty(mk.mukv_prefill_workspace_size(p.gpu.h, n_q, 2, 1), dtype=torch.uint8, device="cuda")
    o_out, s_out = torch.empty_like(q_d), torch.empty(1, n_q, device="cuda")

    def step():
        p.gpu.reset()
        for k, v, att in chunks:
            p.gpu.compress_chunk(k, v, None, att_signal=att)
        p.gpu.retrieve(qd, offs, mode=mk.MUKV_SEMI, k_seg=1, k_frame=2, lambda_frame=0.3, out=r_out)
        p.gpu.prefill_attend(1, q_d, r_out["frame_idx"], k_d, v_d, l_off, True, out=o_out, signal=s_out, workspace=ws)

    step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    torch.cuda.synchronize()
    want = p.orc.retrieve(np_view(qt), orc.RetrieveParams(orc.SEMI, 1, 2, 0.3))
    o_want, s_want = p.orc.prefill_attend(1, np_view(q_new[0]), want["frame_idx"], np_view(k_loc), np_view(v_loc), True)
    for replay in range(3):
        p.gpu.reset()                                 # eager work between the replays: as many frames (the frame
        for c in (3, 1, 0, 2):                        # count lives on the host), other contents
            p.gpu.compress_chunk(*chunks[c][:2], None, att_signal=chunks[(c + 1) % 4][2])
        p.gpu.flush()
        o_out.zero_()
        s_out.fill_(-1)
        r_out["frame_idx"].fill_(-7)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        st = p.gpu.state()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(st["kept_idx"].cpu().numpy(), p.orc.kept, err_msg=f"replay {replay}")
        assert int(st["refined"].sum()) == 8
        np.testing.assert_array_equal(r_out["frame_idx"][0].cpu().numpy(), want["frame_idx"])
        assert out_err(to_f64(np_view(o_out[0].cpu())), o_want) <= 2e-2
        assert np.abs(s_out[0].cpu().numpy() - s_want).max() <= 1e-6
    p.close()


@pytest.mark.parametrize("name,kw,n_q,n_loc", [("7b", {"n_layers": 2}, 20, 12), ("tiny", {}, 20, 12),
                                               ("7b", {"n_layers": 2}, 40, 12), ("72b", {"n_layers": 2}, 40, 12),
                                               ("7b", {"n_layers": 2}, 150, 3)])
def test_prefill_with_fewer_local_rows_than_new_tokens(name, kw, n_q, n_loc):
    # n_q query tokens but only n_loc local rows: the first n_q - n_loc tokens have no row of their own -- they
    # see the retrieved rows only (the oracle's attention without local rows) and receive no attention.  With
    # 28 such tokens in the 40-token cases, and 147 of 150, whole 128-query tiles of the matrix-core kernel (18 or 16
    # tokens) hold nothing but tokens without a row, which must still see every retrieved row.
    w = W[name].scaled(n_frames=8, **kw)
    p = Pair(w, seed=430, chunk=4)
    p.ingest()
    gen = torch.Generator().manual_seed(431)
    q = torch.randn(1, n_q, w.n_q_heads, w.head_dim, generator=gen).to(w.torch_dtype)
    kl = torch.randn(n_loc, w.n_kv_heads, w.head_dim, generator=gen).to(w.torch_dtype)
    vl = torch.randn(n_loc, w.n_kv_heads, w.head_dim, generator=gen).to(w.torch_dtype)
    fi = torch.tensor([[5, 1]], dtype=torch.int32, device="cuda")
    out, sig = p.gpu.prefill_attend(0, q.cuda(), fi, kl.cuda(), vl.cuda(), torch.tensor([0, n_loc], dtype=torch.int32).cuda(), True)
    torch.cuda.synchronize()
    sig = sig[0].cpu().numpy()
    n0 = n_q - n_loc
    assert np.all(sig[:n0] == 0.0) and np.all(sig[n0:] > 0.0)
    got = to_f64(np_view(out[0].cpu()))
    want = p.orc.attend(0, np_view(q[0, :n0]), [5, 1])
    assert out_err(got[:n0], want) <= mk_tol(w)
    # the last n_loc tokens are an ordinary prefill of n_loc tokens
    want_l, sig_l = p.orc.prefill_attend(0, np_view(q[0, n0:]), [5, 1], np_view(kl), np_view(vl), True)
    assert out_err(got[n0:], want_l) <= mk_tol(w)
    assert np.abs(sig[n0:] * n_q / n_loc - sig_l).max() <= 1e-6      # the mean runs over the n_q query rows of the call
    p.close()


@pytest.mark.parametrize("margin", [-1.0, 0.0])      # the keep in fp64, in fp32
@pytest.mark.parametrize("P,rho", [(257, 0.5), (300, 1.0), (1025, 0.003), (4096, 0.7)])
def test_keep_of_a_unit_with_few_distinct_scores(P, rho, margin):
    # the digit search ends with every bit looked at, at once where all keys are equal, or at the one key left
    att = torch.zeros(6, P)
    att[1, 7::11] = 1.0                                   # two values, the cut inside one of them
    att[2] = torch.arange(P).remainder(3) / 8.0
    att[3, P // 2] = 1.0                                  # one token above all others
    att[4] = torch.linspace(0.5, 1.0, P)                  # all different
    att[5] = 0.25 + torch.arange(P).remainder(5) * 2.0 ** -23   # neighbours in the last bit
    w = _unit_workload("bf16", P, 4, rho, 1.0, 6)
    p = Pair(w, seed=330, chunk=3, with_q=False, gpu_kw={"refine_margin": margin})
    for u in (0, 3):
        k, v, _ = p.stream.next_chunk(3)
        p.orc.compress_chunk(np_view(k), np_view(v), att=att[u:u + 3].numpy().astype(np.float64))
        p.gpu.compress_chunk(k.cuda(), v.cuda(), att_signal=att[u:u + 3].contiguous().cuda())
        torch.cuda.synchronize()
    p.check_compress()
    p.close()


@pytest.mark.parametrize("i", range(16))
def test_seeded_sweep_of_large_units(i):
    # units of 257..8192 tokens nobody picked by hand: super-patch counts, keep ratios, signal mixes, payloads,
    # head sizes, launch modes; the signal handed over; then retrieval over units and attention on that cache
    rng = np.random.default_rng(9000 + i)
    P = int(rng.integers(257, 8193)) if i % 4 else int(rng.choice([257, 512, 4096, 6272, 8192]))
    hkv = int(rng.choice([1, 2, 4]))
    units = int(rng.integers(2, 7))
    kw = {"batch_chunks": int(rng.choice([1, 2])), "overlap_copy": int(rng.integers(0, 2)),
          "refine_margin": float(rng.choice([-1.0, 0.0, 10.0]))}
    w = _unit_workload(str(rng.choice(["bf16", "f32"])), P, int(rng.choice([1, 2, 7, 32])), float(rng.choice([0.05, 0.3, 0.8, 1.0])),
                       float(rng.choice([0.0, 0.5, 0.8, 1.0])), units, frames_per_segment=int(rng.choice([1, 2, 3])),
                       n_layers=int(rng.integers(1, 3)), n_kv_heads=hkv, n_q_heads=hkv * int(rng.choice([1, 2])),
                       head_dim=int(rng.choice([16, 32, 64, 128])))
    p = Pair(w, seed=9100 + i, chunk=int(rng.integers(1, 3)), with_q=False, gpu_kw=kw)
    p.ingest(att_seed=9200 + i)
    p.check_compress()
    p.check_retrieve(questions_for(w, [5, 9], 9300 + i), mk.MUKV_SEMI, 1, 2, 0.3)
    p.check_attend(0, 2, [[0, units - 1], [units - 1, -1]], [4, 2], True, seed=i)
    p.close()


# ------------- three independently compressed stores searched together (Sec. 3.3-3.4, Sec. 4.1) -----
def _three_stores(P, F, S, T, rhos, alphas, head, dtype, seed, gpu_kw=None):
    """One K/V stream of T time steps of F frames; store 0 takes the segments (units of F*P tokens), store 1
    the middle frame of every segment (P tokens), store 2 that frame's S super-patches (P // S tokens each).
    Every store has its own rho and alpha and is handed its attention signal.  Returns the Pairs and k, v."""
    base = W["tiny"].scaled(dtype=dtype, tokens_per_frame=P, frames_per_segment=F, n_frames=T * F, spike_prob=0.05, **head)
    k, v, _ = synth.SynthStream(base, seed, device="cpu", with_q=False).next_chunk(T * F)
    mid, u_p = F // 2, P // S
    tok = [torch.arange(T * F * P),
           torch.cat([(t * F + mid) * P + torch.arange(P) for t in range(T)]),
           torch.cat([(t * F + mid) * P + torch.arange(S * u_p) for t in range(T)])]
    pairs = []
    for i, unit in enumerate((F * P, P, u_p)):
        n_units = tok[i].numel() // unit
        w = base.scaled(tokens_per_frame=unit, frames_per_segment=1, superpatches_per_frame=1, keep_ratio=rhos[i],
                        alpha=alphas[i], n_frames=n_units, n_questions=3)
        p = Pair(w, seed=seed, chunk=n_units, with_q=False, gpu_kw=gpu_kw)
        ki, vi = k[:, :, tok[i]].contiguous(), v[:, :, tok[i]].contiguous()
        att = synth.handed_over_attention(n_units, unit, seed + 10 + i)
        p.orc.compress_chunk(np_view(ki), np_view(vi), att=att.numpy().astype(np.float64))
        kd, vd, ad = ki.cuda(), vi.cuda(), att.cuda()
        p.keep_alive += [kd, vd, ad]
        p.gpu.compress_chunk(kd, vd, att_signal=ad)
        pairs.append(p)
    torch.cuda.synchronize()
    return pairs, base


def _check_three_stores(pairs, base, qs, ks, lams, ups, n_global=0, rows_cap=None):
    B = len(qs)
    qt = torch.cat(qs).contiguous().cuda()
    offs = torch.tensor(np.concatenate([[0], np.cumsum([q.shape[0] for q in qs])]), dtype=torch.int32, device="cuda")
    g0 = pairs[0].gpu.retrieve_units(qt, offs, ks[0], n_global=n_global, want_g=True)
    got = [g0] + [p.gpu.retrieve_units(qt, offs, k, lam, g_in=g0["g"]) for p, k, lam in zip(pairs[1:], ks[1:], lams[1:])]
    kap = [p.orc.kappa for p in pairs]
    cap = rows_cap or sum(k * c for k, c in zip(ks, kap))
    ko, vo, nt = mk.gather_multi([p.gpu for p in pairs], [g["idx"] for g in got], ups, cap)
    torch.cuda.synchronize()
    for b in range(B):
        want = orc.retrieve_multi([p.orc for p in pairs], np_view(qs[b]), ks, lams, n_global=n_global)
        np.testing.assert_allclose(g0["g"][b].cpu().numpy(), want[0]["g"], rtol=0, atol=1e-14)
        for i in range(3):
            np.testing.assert_array_equal(got[i]["idx"][b].cpu().numpy(), want[i]["idx"], err_msg=f"store {i} question {b}")
            assert np.abs(got[i]["score"][b].cpu().numpy() - want[i]["score"]).max() <= 1e-5
        kw, vw, n = orc.gather_multi([p.orc for p in pairs], [w_["idx"] for w_ in want], ups, rows_cap=cap)
        assert int(nt[b]) == n
        np.testing.assert_array_equal(np_view(ko[b].cpu()), kw)
        np.testing.assert_array_equal(np_view(vo[b].cpu()), vw)
    return got


@pytest.mark.parametrize("dtype,head", [("f32", dict(n_layers=2, n_q_heads=4, n_kv_heads=2, head_dim=32)),
                                        ("bf16", dict(n_layers=2, n_q_heads=28, n_kv_heads=4, head_dim=128))])
def test_three_stores_retrieved_together(dtype, head):
    P, F, S, T = 24, 2, 3, 11
    pairs, base = _three_stores(P, F, S, T, (0.8, 0.25, 0.5), (0.8, 0.7, 0.5), head, dtype, seed=7700)
    qs = [synth.random_question(base, n, 7710 + i) for i, n in enumerate([5, 12, 3])]
    _check_three_stores(pairs, base, qs, [3, 5, 6], [0.0, 0.3, 0.3], [1, 1, S])
    _check_three_stores(pairs, base, qs, [3, 5, 6], [0.0, 0.9, 0.0], [1, 1, S], n_global=1)
    # more asked for than exists (padding), and an output too short for the context
    _check_three_stores(pairs, base, qs, [14, 20, 40], [0.0, 0.3, 0.3], [1, 1, S], rows_cap=50)
    # repeated and out-of-range entries in the lists given to the gather
    idx = [torch.tensor([[4, 4, -1, 99]] * 3, dtype=torch.int32, device="cuda"),
           torch.tensor([[10, 0, 10]] * 3, dtype=torch.int32, device="cuda"),
           torch.tensor([[32, 1, 33, 1, 7]] * 3, dtype=torch.int32, device="cuda")]
    ko, vo, nt = mk.gather_multi([p.gpu for p in pairs], idx, [1, 1, S], 200)
    torch.cuda.synchronize()
    kw, vw, n = orc.gather_multi([p.orc for p in pairs], [i[0].cpu().numpy() for i in idx], [1, 1, S], rows_cap=200)
    assert int(nt[0]) == n
    np.testing.assert_array_equal(np_view(ko[2].cpu()), kw)
    np.testing.assert_array_equal(np_view(vo[0].cpu()), vw)
    for p in pairs:
        p.close()


def test_three_stores_with_the_paper_hyper_parameters():
    # Sec. 4.1: P = 196, F = 4, S = 4; rho = 0.8 / 0.1 / 0.1, alpha = 0.8 / 0.7 / 0.5, k_g = 12 / 32 / 20 and
    # lambda_g = 0 / 0.3 / 0.3 for segment / frame / patch; Table 1: 8.3K tokens loaded per question
    # (12 * 627 + 32 * 19 + 20 * 4 = 8212), in the 7B head layout
    head = dict(n_layers=2, n_q_heads=28, n_kv_heads=4, head_dim=128)
    pairs, base = _three_stores(196, 4, 4, 40, (0.8, 0.1, 0.1), (0.8, 0.7, 0.5), head, "bf16", seed=7800)
    assert [p.orc.kappa for p in pairs] == [627, 19, 4]
    qs = [synth.random_question(base, n, 7810 + i) for i, n in enumerate([32, 16])]
    got = _check_three_stores(pairs, base, qs, [12, 32, 20], [0.0, 0.3, 0.3], [1, 1, 4])
    ko, vo, nt = mk.gather_multi([p.gpu for p in pairs], [g["idx"] for g in got], [1, 1, 4], 8212)
    torch.cuda.synchronize()
    assert nt.cpu().tolist() == [8212, 8212]
    for p in pairs:
        p.close()


def test_three_stores_argument_errors():
    head = dict(n_layers=1, n_q_heads=4, n_kv_heads=2, head_dim=32)
    pairs, base = _three_stores(12, 2, 3, 4, (0.8, 0.5, 0.5), (0.8, 0.7, 0.5), head, "f32", seed=7900)
    other = gpu_context(base.scaled(n_layers=2, n_frames=4), max_frames=4, max_chunk_frames=4)
    idx = torch.zeros(1, 2, dtype=torch.int32, device="cuda")
    with pytest.raises(mk.MuKVError) as e:                       # stores of different models
        mk.gather_multi([pairs[0].gpu, other], [idx, idx], [1, 1], 16)
    assert e.value.status == mk.MUKV_ERR_SHAPE
    with pytest.raises(mk.MuKVError) as e:                       # more entries than the plan holds
        mk.gather_multi([pairs[0].gpu], [torch.zeros(1, 3073, dtype=torch.int32, device="cuda")], [1], 16)
    assert e.value.status == mk.MUKV_ERR_UNSUPPORTED
    qt = synth.random_question(base, 4, 1).cuda()
    offs = torch.tensor([0, 4], dtype=torch.int32, device="cuda")
    g = torch.zeros(1, 64, dtype=torch.float64, device="cuda")
    with pytest.raises(mk.MuKVError) as e:                       # a store either supplies the global query or takes it
        mk.mukv_retrieve_units(pairs[1].gpu.h, qt.data_ptr(), offs.data_ptr(), 1, 2, 0.3, -1, g.data_ptr(), 0, g.data_ptr(),
                               idx.data_ptr(), None, None)
    assert e.value.status == mk.MUKV_ERR_INVALID_ARG
    other.close()
    for p in pairs:
        p.close()
