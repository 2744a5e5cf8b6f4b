"""GPU parity: the HIP path behind the C ABI against the CPU fp64 oracle on the same seeded
bytes.  Integer results (row indices, lengths, copied rows) must be bit-exact; floats within
the tolerances in gpu_util."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2503_09387_amd as vs
from gpu_util import (DEV, check_close, lens_array, oracle_prefill_rows, run_prefill, scale32,
                      torch_dtype, vs_shape, workspace)
from synth import (CONFIGS, AttnShape, cache_rows, carrier_embeddings, cfg1_inputs, decode_lengths, decode_step_inputs,
                   draw, frame_inputs, to_f64)

pytestmark = pytest.mark.gpu

QW = CONFIGS["cfg2"]["shape"]


@pytest.fixture(autouse=True)
def _reset_tuning():
    yield
    for knob in (0, 1, 2, 4):
        vs.set_tuning(knob, 0)


def same_bits(dev_t, host_t):
    return torch.equal(dev_t.cpu().view(torch.uint8), host_t.contiguous().view(torch.uint8))


# ---------------------------------------------------------------------------- cfg1
def test_cfg1_tiny_fp32_pool_prefill_compact():
    c = CONFIGS["cfg1"]
    s = c["shape"]
    x = cfg1_inputs(c)
    L, T = c["prefix"], c["n_visual"] + 1
    # carrier embedding
    e = x["e"].to(DEV)
    pooled = torch.empty(c["hidden"], dtype=torch.float32, device=DEV)
    vs.carrier_mean_pool(e, pooled, "f32")
    check_close(pooled, oracle.mean_pool(to_f64(x["e"])), "f32", "mean pool")
    # prefill
    out, cache, _ = run_prefill(s, x["k_c"], x["v_c"], L, x["q"], x["k_f"], x["v_f"], capacity=L + 1)
    ref = oracle_prefill_rows(s, x["q"], x["k_c"], x["v_c"], L, x["k_f"], x["v_f"])
    check_close(out, ref, "f32", "cfg1 prefill")
    # compaction
    row = vs.carrier_compact_append(vs_shape(s), cache, x["k_f"].to(DEV), x["v_f"].to(DEV))
    torch.cuda.synchronize()
    ok_k, ok_v = to_f64(x["k_c"]).copy(), to_f64(x["v_c"]).copy()
    ok_k, ok_v = np.concatenate([ok_k, np.zeros((1,) + ok_k.shape[1:])]), np.concatenate([ok_v, np.zeros((1,) + ok_v.shape[1:])])
    orow, olen = oracle.compact_append(ok_k, ok_v, L, to_f64(x["k_f"]), to_f64(x["v_f"]))
    assert (row, cache.len) == (orow, olen) == (16, 17)
    assert np.array_equal(cache.k.double().cpu().numpy(), ok_k) and np.array_equal(cache.v.double().cpu().numpy(), ok_v)
    # fused entry point gives the same bits
    out2, cache2, row2 = run_prefill(s, x["k_c"], x["v_c"], L, x["q"], x["k_f"], x["v_f"], capacity=L + 1, fused=True)
    assert row2 == 16 and cache2.len == 17
    assert torch.equal(out2, out) and torch.equal(cache2.k, cache.k) and torch.equal(cache2.v, cache.v)


# ---------------------------------------------------------------------------- cfg2
@pytest.mark.parametrize("fused", [False, True])
def test_cfg2_stream_of_64_frames(fused):
    c = CONFIGS["cfg2"]
    s, P0, F, T = c["shape"], c["prefix"], c["frames"], c["n_visual"] + 1
    pk, pv = cache_rows(c["seed"], s, P0, c["sigma"])
    cap = P0 + F
    kc = torch.zeros((cap, s.n_kv_heads, s.head_dim), dtype=torch.bfloat16, device=DEV)
    vc = torch.zeros_like(kc)
    kc[:P0].copy_(pk)
    vc[:P0].copy_(pv)
    cache = vs.Cache(kc, vc, P0)
    ws = workspace(s, T, cap, 0)
    ok, ov = np.zeros((cap, s.n_kv_heads, s.head_dim)), np.zeros((cap, s.n_kv_heads, s.head_dim))
    ok[:P0], ov[:P0] = to_f64(pk), to_f64(pv)
    olen = P0
    sh = vs_shape(s)
    worst = (0.0, 0.0)
    for f in range(F):
        q, kf, vf = frame_inputs(c["seed"], s, T, c["sigma"], frame=f)
        qd, kfd, vfd = q.to(DEV), kf.to(DEV), vf.to(DEV)
        out = torch.empty_like(qd)
        if fused:
            row = vs.frame_prefill_compact(sh, cache, qd, kfd, vfd, out, ws)
        else:
            vs.frame_prefill_attn(sh, cache, qd, kfd, vfd, out, ws)
            row = vs.carrier_compact_append(sh, cache, kfd, vfd)
        ref = oracle.frame_prefill(to_f64(q), ok[:olen], ov[:olen], to_f64(kf), to_f64(vf), scale32(s))
        orow, olen = oracle.compact_append(ok, ov, olen, to_f64(kf), to_f64(vf))
        assert (row, cache.len) == (orow, olen), f"frame {f}"
        torch.cuda.synchronize()
        e = check_close(out, ref, "bf16", f"cfg2 frame {f}")
        worst = (max(worst[0], e[0]), max(worst[1], e[1]))
    assert cache.len == 264
    assert np.array_equal(kc.double().cpu().numpy(), ok) and np.array_equal(vc.double().cpu().numpy(), ov)
    print(f"cfg2 worst max-abs {worst[0]:.2e} mean-abs {worst[1]:.2e}")


# ---------------------------------------------------------------------------- cfg3
def test_cfg3_whole_stream_all_frames_all_layers():
    """The whole long stream: 256 frames x 28 layers through vs_frame_prefill_compact, starting from
    4296 retained rows per layer.  Row index and length of EVERY (frame, layer) call are compared
    with oracle.compact_append run beside it, and at the end every cache byte (retained rows,
    the 256 appended carrier rows, untouched tail) with the oracle's arrays.  Floats are checked
    against the oracle on frames whose cache length is 0, 1 and 63 past a multiple of the kernel's
    64-row tile (and the first, a middle and the last frame), three layers, eight tokens each.
    The frames' Q/K/V come from a pool of 8 distinct frames per layer (frame f uses f % 8), as in
    bench.py: the draw of 7168 frame-layers would take minutes, and the retained state does not
    depend on which values move."""
    c = CONFIGS["cfg3"]
    s, T, NL, P0, F = c["shape"], c["n_visual"] + 1, c["layers"], c["prefix"], c["frames"]
    sh = vs_shape(s)
    cap = P0 + F
    POOL = 8
    ws = workspace(s, T, cap, 0)
    sample_layers = (0, 13, 27)
    float_frames = {0, 55, 56, 57, 128, 255}          # 4296 + f = 63, 0, 1 (mod 64) at f = 55, 56, 57
    assert [(P0 + f) % 64 for f in (55, 56, 57)] == [63, 0, 1]
    tokens = np.array([0, 1, 37, 84, 85, 127, 168, 169])
    tok_dev = torch.from_numpy(tokens).to(DEV)
    pool_host = [[frame_inputs(c["seed"], s, T, c["sigma"], frame=f, layer=l) for l in range(NL)] for f in range(POOL)]
    pool_dev = [[tuple(x.to(DEV) for x in fl) for fl in fr] for fr in pool_host]
    pool_kv64 = [[(to_f64(fl[1]), to_f64(fl[2])) for fl in fr] for fr in pool_host]
    caches, ok, ov, olen = [], [], [], []
    for l in range(NL):
        hk, hv = cache_rows(c["seed"], s, P0, c["sigma"], layer=l)
        kc = torch.zeros((cap, s.n_kv_heads, s.head_dim), dtype=torch.bfloat16, device=DEV)
        vc = torch.zeros_like(kc)
        kc[:P0].copy_(hk)
        vc[:P0].copy_(hv)
        caches.append(vs.Cache(kc, vc, P0))
        k64, v64 = np.zeros((cap, s.n_kv_heads, s.head_dim)), np.zeros((cap, s.n_kv_heads, s.head_dim))
        k64[:P0], v64[:P0] = to_f64(hk), to_f64(hv)
        ok.append(k64)
        ov.append(v64)
        olen.append(P0)
    outs = [torch.empty((T, s.n_q_heads, s.head_dim), dtype=torch.bfloat16, device=DEV) for _ in sample_layers]
    unchecked = torch.empty_like(outs[0])
    for f in range(F):
        pending = []
        for l in range(NL):
            qd, kfd, vfd = pool_dev[f % POOL][l]
            sampled = f in float_frames and l in sample_layers
            out = outs[sample_layers.index(l)] if sampled else unchecked
            if sampled:  # the oracle's view of the cache before this frame
                q, kf, vf = pool_host[f % POOL][l]
                ref = oracle.attention(to_f64(q)[tokens], np.concatenate([ok[l][:olen[l]], to_f64(kf)]),
                                       np.concatenate([ov[l][:olen[l]], to_f64(vf)]), olen[l] + tokens + 1, scale32(s))
                pending.append((l, out, ref))
            row = vs.frame_prefill_compact(sh, caches[l], qd, kfd, vfd, out, ws)
            orow, olen[l] = oracle.compact_append(ok[l], ov[l], olen[l], *pool_kv64[f % POOL][l])
            assert (row, caches[l].len) == (orow, olen[l]) == (P0 + f, P0 + f + 1), f"frame {f} layer {l}"
        if pending:
            torch.cuda.synchronize()
            for l, out, ref in pending:
                check_close(out[tok_dev], ref, "bf16", f"cfg3 whole stream, frame {f} layer {l}")
    torch.cuda.synchronize()
    for l in range(NL):
        assert caches[l].len == olen[l] == 4552
        assert np.array_equal(caches[l].k.double().cpu().numpy(), ok[l]), f"K cache of layer {l}"
        assert np.array_equal(caches[l].v.double().cpu().numpy(), ov[l]), f"V cache of layer {l}"


# ---------------------------------------------------------------------------- cfg4
def test_cfg4_decode_16_ragged_streams():
    """Full launch shape (16 streams, lengths U[512,8192]+128, capacity 8384); 2 of the 28 layers
    (each layer is the same launch), 6 of the 64 steps with floats checked on every one."""
    c = CONFIGS["cfg4"]
    s, S = c["shape"], c["streams"]
    sh = vs_shape(s)
    lens0 = decode_lengths(c["seed"], S, c["carrier_lo"], c["carrier_hi"], c["text_hist"])
    assert min(lens0) >= 640 and max(lens0) <= 8320
    cap = c["carrier_hi"] + c["text_hist"] + c["steps"]
    ws = workspace(s, 0, cap, S)
    for layer in (0, 27):
        ks = torch.zeros((S, cap, s.n_kv_heads, s.head_dim), dtype=torch.bfloat16, device=DEV)
        vsl = torch.zeros_like(ks)
        ok = [np.zeros((cap, s.n_kv_heads, s.head_dim)) for _ in range(S)]
        ov = [np.zeros((cap, s.n_kv_heads, s.head_dim)) for _ in range(S)]
        for i in range(S):
            hk, hv = cache_rows(c["seed"], s, lens0[i], c["sigma"], layer=layer, stream=i)
            ks[i, :lens0[i]].copy_(hk)
            vsl[i, :lens0[i]].copy_(hv)
            ok[i][:lens0[i]], ov[i][:lens0[i]] = to_f64(hk), to_f64(hv)
        lens = lens_array(lens0)
        olens = list(lens0)
        for step in range(6):
            q, kn, vn = decode_step_inputs(c["seed"], s, S, c["sigma"], step=step, layer=layer)
            out = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device=DEV)
            vs.decode_attn(sh, ks, vsl, lens, q.to(DEV), kn.to(DEV), vn.to(DEV), out, ws)
            ref = np.zeros((S, s.n_q_heads, s.head_dim))
            for i in range(S):
                ref[i], olens[i] = oracle.decode(to_f64(q[i]), ok[i], ov[i], olens[i], to_f64(kn[i]),
                                                 to_f64(vn[i]), scale32(s))
            assert list(lens) == olens, f"lengths after step {step}"
            torch.cuda.synchronize()
            check_close(out, ref, "bf16", f"cfg4 layer {layer} step {step}")
        for i in range(S):
            assert np.array_equal(ks[i].double().cpu().numpy(), ok[i])
            assert np.array_equal(vsl[i].double().cpu().numpy(), ov[i])


def test_cfg4_whole_decode_64_steps_28_layers():
    """All 64 steps on all 28 layers of the 16 ragged streams.  After every call the lengths are
    compared with the oracle's; at the end every appended row (64 per stream and layer) is compared
    bit for bit with what oracle.compact_append put there, and the rows in front of them and behind
    them with what was there before.  Floats against oracle.decode for all 16 streams at
    (layer, step) = (0, 0), (13, 31) and (27, 63), the last step included.
    The oracle's row copy works on a window of each stream's cache that starts at the stream's
    initial length (an append is the same operation wherever the row sits; whole caches in fp64
    would take 30 GB).  Four distinct layer slabs are drawn and copied to the 28 layers, as in
    bench.py; the inputs of every (step, layer) are drawn on their own."""
    c = CONFIGS["cfg4"]
    s, S, NL, steps = c["shape"], c["streams"], c["layers"], c["steps"]
    sh = vs_shape(s)
    lens0 = decode_lengths(c["seed"], S, c["carrier_lo"], c["carrier_hi"], c["text_hist"])
    cap = c["carrier_hi"] + c["text_hist"] + steps
    ws = workspace(s, 0, cap, S)
    DISTINCT = 4
    base_host, base_dev = [], []
    for l in range(DISTINCT):
        k = torch.zeros((S, cap, s.n_kv_heads, s.head_dim), dtype=torch.bfloat16)
        v = torch.zeros_like(k)
        for i in range(S):
            hk, hv = cache_rows(c["seed"], s, lens0[i], c["sigma"], layer=l, stream=i)
            k[i, :lens0[i]], v[i, :lens0[i]] = hk, hv
        base_host.append((k, v))
        base_dev.append((k.to(DEV), v.to(DEV)))
    slabs = [(base_dev[l % DISTINCT][0].clone(), base_dev[l % DISTINCT][1].clone()) for l in range(NL)]
    lens = [lens_array(lens0) for _ in range(NL)]
    # oracle state: the rows appended to (layer, stream), as a window starting at the initial length
    wk = [[np.zeros((steps, s.n_kv_heads, s.head_dim)) for _ in range(S)] for _ in range(NL)]
    wv = [[np.zeros((steps, s.n_kv_heads, s.head_dim)) for _ in range(S)] for _ in range(NL)]
    wlen = [[0] * S for _ in range(NL)]
    float_at = {(0, 0), (13, 31), (27, steps - 1)}
    out = torch.empty((S, s.n_q_heads, s.head_dim), dtype=torch.bfloat16, device=DEV)
    for step in range(steps):
        for l in range(NL):
            q, kn, vn = decode_step_inputs(c["seed"], s, S, c["sigma"], step=step, layer=l)
            kn64, vn64 = to_f64(kn), to_f64(vn)
            ref = None
            if (l, step) in float_at:
                ref = np.zeros((S, s.n_q_heads, s.head_dim))
                for i in range(S):
                    n0 = lens0[i]
                    k_all = np.concatenate([to_f64(base_host[l % DISTINCT][0][i, :n0]), wk[l][i][:step], np.zeros((1, s.n_kv_heads, s.head_dim))])
                    v_all = np.concatenate([to_f64(base_host[l % DISTINCT][1][i, :n0]), wv[l][i][:step], np.zeros((1, s.n_kv_heads, s.head_dim))])
                    ref[i], n_after = oracle.decode(to_f64(q[i]), k_all, v_all, n0 + step, kn64[i], vn64[i], scale32(s))
                    assert n_after == n0 + step + 1
            vs.decode_attn(sh, slabs[l][0], slabs[l][1], lens[l], q.to(DEV), kn.to(DEV), vn.to(DEV), out, ws)
            for i in range(S):
                row, wlen[l][i] = oracle.compact_append(wk[l][i], wv[l][i], wlen[l][i], kn64[i:i + 1], vn64[i:i + 1])
                assert row == step
            assert list(lens[l]) == [lens0[i] + wlen[l][i] for i in range(S)], f"lengths after step {step}, layer {l}"
            if ref is not None:
                torch.cuda.synchronize()
                check_close(out, ref, "bf16", f"cfg4 whole decode, layer {l} step {step}")
    torch.cuda.synchronize()
    for l in range(NL):
        kd, vd = slabs[l][0].cpu(), slabs[l][1].cpu()
        for i in range(S):
            n0 = lens0[i]
            assert lens[l][i] == n0 + steps
            assert np.array_equal(to_f64(kd[i, n0:n0 + steps]), wk[l][i]), f"appended K rows, layer {l} stream {i}"
            assert np.array_equal(to_f64(vd[i, n0:n0 + steps]), wv[l][i]), f"appended V rows, layer {l} stream {i}"
            assert torch.equal(kd[i, :n0], base_host[l % DISTINCT][0][i, :n0]) and torch.equal(vd[i, :n0], base_host[l % DISTINCT][1][i, :n0])
            assert not kd[i, n0 + steps:].any() and not vd[i, n0 + steps:].any()


# ---------------------------------------------------------------------------- cfg5
def test_cfg5_dense_and_compact_cache_same_frame():
    c = CONFIGS["cfg5"]
    s, T = c["shape"], c["n_visual"] + 1
    q, kf, vf = frame_inputs(c["seed"], s, T, c["sigma"])
    tokens = np.array([0, 2, 36, 37, 90, 128, 168, 169])
    for name, rows, stream in (("dense", c["dense_rows"], 0), ("compact", c["compact_rows"], 1)):
        hk, hv = cache_rows(c["seed"], s, rows, c["sigma"], stream=stream)
        out, _, _ = run_prefill(s, hk, hv, rows, q, kf, vf)
        if name == "compact":
            ref = oracle_prefill_rows(s, q, hk, hv, rows, kf, vf)
            check_close(out, ref, "bf16", "cfg5 compact")
        else:
            ref = oracle_prefill_rows(s, q, hk, hv, rows, kf, vf, tokens)
            check_close(out[torch.from_numpy(tokens).to(DEV)], ref, "bf16", "cfg5 dense (sampled tokens)")


# ---------------------------------------------------------------------------- prefill edges
@pytest.mark.parametrize("L,T,gain", [(0, 1, 1), (0, 5, 1), (1, 1, 1), (63, 2, 1), (64, 64, 1), (65, 170, 1),
                                      (200, 170, 8), (263, 170, 1), (1000, 19, 8), (4551, 170, 8), (130, 512, 1)])
@pytest.mark.parametrize("kv_groups", [0, 1, 2])  # 0: as dispatched (few keys: the kernel that splits nothing); else the other kernel
def test_prefill_bf16_shapes_and_peaked_softmax(L, T, gain, kv_groups):
    s = QW
    vs.set_tuning(vs.TUNE_PREFILL_KV_GROUPS, kv_groups)
    hk, hv = cache_rows(11, s, max(L, 1), 0.5)
    q, kf, vf = frame_inputs(11, s, T, 0.5, frame=L, layer=T % 7, q_gain=gain)
    out, _, _ = run_prefill(s, hk, hv, L, q, kf, vf)
    check_close(out, oracle_prefill_rows(s, q, hk, hv, L, kf, vf), "bf16", f"L={L} T={T} gain={gain}")
    if L == 0:  # a single visible key returns its V row exactly
        assert same_bits(out[0].reshape(s.n_kv_heads, s.group, -1)[:, 0], vf[0])


@pytest.mark.parametrize("hq,hkv", [(8, 8), (8, 1), (12, 4), (16, 2)])
@pytest.mark.parametrize("kv_groups", [0, 1, 2])
def test_prefill_other_head_groupings(hq, hkv, kv_groups):
    s = AttnShape(hq, hkv, 128, "bf16")
    vs.set_tuning(vs.TUNE_PREFILL_KV_GROUPS, kv_groups)
    L, T = 150, 70
    hk, hv = cache_rows(12, s, L, 0.5)
    q, kf, vf = frame_inputs(12, s, T, 0.5, q_gain=4)
    out, _, _ = run_prefill(s, hk, hv, L, q, kf, vf)
    check_close(out, oracle_prefill_rows(s, q, hk, hv, L, kf, vf), "bf16", f"Hq={hq} Hkv={hkv}")


@pytest.mark.parametrize("kv_groups", [1, 2])
def test_prefill_result_does_not_depend_on_the_split(kv_groups):
    s = QW
    L, T = 1500, 170
    hk, hv = cache_rows(13, s, L, 0.5)
    q, kf, vf = frame_inputs(13, s, T, 0.5, q_gain=4)
    ref = oracle_prefill_rows(s, q, hk, hv, L, kf, vf)
    vs.set_tuning(vs.TUNE_PREFILL_KV_GROUPS, kv_groups)
    outs = []
    for splits in (1, 2, 5, 12, 32):
        vs.set_tuning(vs.TUNE_PREFILL_SPLITS, splits)
        out, _, _ = run_prefill(s, hk, hv, L, q, kf, vf)
        check_close(out, ref, "bf16", f"splits={splits} kv_groups={kv_groups}")
        outs.append(out.float())
    for o in outs[1:]:
        assert (o - outs[0]).abs().max().item() <= 2 ** -7 * outs[0].abs().max().item()


@pytest.mark.parametrize("L,T,splits", [(4424, 170, 0), (1500, 170, 0), (1500, 170, 3), (3000, 300, 8), (700, 40, 2),
                                          # (300 tokens: more groups of 32 rows than compute units, so not the kernel that splits nothing)
                                          (100, 300, 0), (264, 170, 3), (100, 20, 2),
                                          # more than 8 splits (questions of a few tokens; several rounds of workgroups)
                                          (4552, 16, 0), (4552, 64, 0), (1500, 170, 12), (3000, 170, 32), (2100, 30, 9)])
def test_prefill_merge_inside_the_kernel_equals_the_second_kernel(L, T, splits):
    """Split results are merged inside the attention kernel, by the workgroups of a row tile together
    once the last of them has arrived (the library's choice) or by that last one alone, or by a
    second kernel: the same sums in the same order, so the same bits; also on repeated calls
    through one workspace (the arrival counters return to zero, launch numbers move on) and with
    the three ways taking turns.  Every case is split: with the second kernel a call is two launches."""
    s = QW
    hk, hv = cache_rows(31, s, L, 0.5)
    q, kf, vf = frame_inputs(31, s, T, 0.5, q_gain=4)
    ref = oracle_prefill_rows(s, q, hk, hv, L, kf, vf)
    ws = workspace(s, T, L, 0)
    vs.set_tuning(vs.TUNE_PREFILL_SPLITS, splits)
    vs.set_tuning(vs.TUNE_PREFILL_MERGE, 2)
    two_kernels, _, _ = run_prefill(s, hk, hv, L, q, kf, vf, ws=ws)
    check_close(two_kernels, ref, "bf16", f"second-kernel merge L={L} T={T} splits={splits}")
    dq, dk, dv, dcache = q.to(DEV), kf.to(DEV), vf.to(DEV), vs.Cache(hk.to(DEV), hv.to(DEV), L)
    spare = torch.empty_like(dq)
    assert _captured(lambda: vs.frame_prefill_attn(vs_shape(s), dcache, dq, dk, dv, spare, ws))[1] == 2
    for mode in (0, 0, 0, 1, 0, 1, 2, 0):
        vs.set_tuning(vs.TUNE_PREFILL_MERGE, mode)
        inside, _, _ = run_prefill(s, hk, hv, L, q, kf, vf, ws=ws)
        assert same_bits(inside, two_kernels.cpu()), f"merge mode {mode} differs from the second kernel's"
    vs.set_tuning(vs.TUNE_PREFILL_MERGE, 0)


@pytest.mark.parametrize("F,T,L,splits", [(2, 170, 4296, 0), (2, 170, 4296, 5), (3, 170, 2000, 4), (4, 60, 900, 2),
                                          (8, 21, 700, 3)])
def test_runs_of_frames_merge_inside_the_kernel_equals_the_second_kernel(F, T, L, splits):
    """The same for runs of frames: units are (KV head, frame, row tile), every frame reads its own
    number of retained rows; both ways of merging give the same bits, call after call."""
    s = QW
    sh = vs_shape(s)
    hk, hv = cache_rows(71, s, L, 0.5)
    q = draw(72, (F, T, s.n_q_heads, s.head_dim), 1.5, "bf16").to(DEV)
    kf = draw(73, (F, T, s.n_kv_heads, s.head_dim), 0.5, "bf16").to(DEV)
    vf = draw(74, (F, T, s.n_kv_heads, s.head_dim), 0.5, "bf16").to(DEV)
    kc = torch.zeros((L + F, s.n_kv_heads, s.head_dim), dtype=torch.bfloat16, device=DEV)
    vc = torch.zeros_like(kc)
    kc[:L].copy_(hk)
    vc[:L].copy_(hv)
    ws = torch.empty(vs.frames_workspace_bytes(sh, F, T, L + F), dtype=torch.uint8, device=DEV)
    vs.workspace_init(sh, ws)
    vs.set_tuning(vs.TUNE_PREFILL_SPLITS, splits)

    def run():
        cache = vs.Cache(kc, vc, L)
        out = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device=DEV)
        vs.frames_prefill_attn(sh, cache, q, kf, vf, out, ws)
        torch.cuda.synchronize()
        return out
    vs.set_tuning(vs.TUNE_PREFILL_MERGE, 2)
    two_kernels = run()
    assert bool(torch.isfinite(two_kernels.float()).all())
    for mode in (0, 0, 1, 0):
        vs.set_tuning(vs.TUNE_PREFILL_MERGE, mode)
        assert torch.equal(run().view(torch.int16), two_kernels.view(torch.int16)), f"merge mode {mode}"
    vs.set_tuning(vs.TUNE_PREFILL_MERGE, 0)


def test_prefill_placement_guard_reports_and_falls_back():
    """Every unit of an in-kernel-merge launch checks that its workgroups ran on one XCD.  With every other
    workgroup giving a neighbouring XCD as its own (tuning value 3) the units
    report themselves misplaced: the launch itself is still right (the real placement is
    unchanged), the next call launches nothing and returns VS_ERR_PLACEMENT, the calls after it merge
    with the second kernel and give the same bits, and a new vs_workspace_init probes again and
    brings the in-kernel merge back."""
    s, L, T = QW, 1500, 170
    hk, hv = cache_rows(75, s, L, 0.5)
    q, kf, vf = frame_inputs(75, s, T, 0.5, q_gain=4)
    ws = workspace(s, T, L, 0)
    good, _, _ = run_prefill(s, hk, hv, L, q, kf, vf, ws=ws)
    vs.set_tuning(vs.TUNE_PREFILL_MERGE, 3)
    flagged, _, _ = run_prefill(s, hk, hv, L, q, kf, vf, ws=ws)      # runs, reports, result still right
    vs.set_tuning(vs.TUNE_PREFILL_MERGE, 0)
    assert same_bits(flagged, good.cpu())
    with pytest.raises(vs.VSError) as err:
        run_prefill(s, hk, hv, L, q, kf, vf, ws=ws)
    assert err.value.code == 8
    for _ in range(2):                                                # second-kernel merge from now on
        after, _, _ = run_prefill(s, hk, hv, L, q, kf, vf, ws=ws)
        assert same_bits(after, good.cpu())
    ws2 = workspace(s, T, L, 0)                                       # probes the device again
    again, _, _ = run_prefill(s, hk, hv, L, q, kf, vf, ws=ws2)
    assert same_bits(again, good.cpu())
    run_prefill(s, hk, hv, L, q, kf, vf, ws=ws2)                      # and nothing is reported this time


def _captured(call):
    """The call captured into a graph, and how many nodes that has."""
    import os
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    hip = ctypes.CDLL(os.path.join(os.path.dirname(torch.__file__), "lib", "libamdhip64.so"))
    count = ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(count)) == 0
    graph.instantiate()
    return graph, count.value


def test_prefill_in_a_program_with_several_streams_and_graphs():
    """Once a process has used several streams or captured a graph, the device deals the ids of a stream from another
    XCD on.  Ids of one residue still share one, so the splits are merged inside the launch as before (one node
    per call), nothing is reported, and the bits are the same: eagerly, on other streams, and on every replay."""
    s, L, T = QW, 1500, 170
    sh = vs_shape(s)
    hk, hv = cache_rows(77, s, L, 0.5)
    q, kf, vf = (t.to(DEV) for t in frame_inputs(77, s, T, 0.5, q_gain=4))
    cache = vs.Cache(hk.to(DEV), hv.to(DEV), L)
    wss = [workspace(s, T, L, 0) for _ in range(5)]
    outs = [torch.empty_like(q) for _ in wss]

    def step(i):
        vs.frame_prefill_attn(sh, cache, q, kf, vf, outs[i], wss[i])

    step(0)
    torch.cuda.synchronize()
    good = outs[0].clone()

    def check(used):
        torch.cuda.synchronize()
        for i in used:
            assert torch.equal(outs[i].view(torch.int16), good.view(torch.int16))
            outs[i].fill_(float("nan"))

    streams = [torch.cuda.Stream() for _ in range(3)]
    for _ in range(4):
        for i, st in enumerate(streams):
            with torch.cuda.stream(st):
                step(1 + i)
            st.synchronize()
        check((1, 2, 3))
        step(0)
        check((0,))
    graph, nodes = _captured(lambda: step(4))
    assert nodes == 1
    for _ in range(4):
        graph.replay()
        check((4,))
        step(0)
        check((0,))
    assert _captured(lambda: step(4))[1] == 1  # (a report would have sent later calls to the second kernel)


def test_prefill_shared_merge_gives_up_waiting_and_reports():
    """In the shared merge the workgroups of a row tile wait for the last of them, looking at a word
    in memory a bounded number of times.  With tuning value 4 that number is zero: every kernel
    still ends, the workgroups that would have waited report through the host word (and leave their
    share unmerged), the next call launches nothing and returns VS_ERR_PLACEMENT, the
    calls after it merge with the second kernel and are right, and a new vs_workspace_init brings
    the in-kernel merge back."""
    s, L, T = QW, 1500, 170
    hk, hv = cache_rows(76, s, L, 0.5)
    q, kf, vf = frame_inputs(76, s, T, 0.5, q_gain=4)
    ws = workspace(s, T, L, 0)
    good, _, _ = run_prefill(s, hk, hv, L, q, kf, vf, ws=ws)
    vs.set_tuning(vs.TUNE_PREFILL_MERGE, 4)
    run_prefill(s, hk, hv, L, q, kf, vf, ws=ws)                       # ends; its output is incomplete
    vs.set_tuning(vs.TUNE_PREFILL_MERGE, 0)
    with pytest.raises(vs.VSError) as err:
        run_prefill(s, hk, hv, L, q, kf, vf, ws=ws)
    assert err.value.code == 8
    for _ in range(2):                                                # second-kernel merge from now on
        after, _, _ = run_prefill(s, hk, hv, L, q, kf, vf, ws=ws)
        assert same_bits(after, good.cpu())
    ws2 = workspace(s, T, L, 0)                                       # probes the device again
    for _ in range(2):
        again, _, _ = run_prefill(s, hk, hv, L, q, kf, vf, ws=ws2)
        assert same_bits(again, good.cpu())


@pytest.mark.parametrize("L,kv_groups", [(130, 0), (130, 1), (130, 2), (1500, 0), (1500, 1)])
@pytest.mark.parametrize("mode", ["all_low", "all_high", "rising", "falling", "jump"])
def test_prefill_extreme_score_ranges(mode, L, kv_groups):
    """Scaled scores far from 0 (in log2 units: around -400, around +400, climbing or falling by
    400 along the keys, or jumping by 60 in the middle): the speculative softmax reference has to
    be dropped and rebuilt, at the first sub-block and later ones, with the accumulators rescaled."""
    s = QW
    T = 170
    vs.set_tuning(vs.TUNE_PREFILL_KV_GROUPS, kv_groups)
    hk, hv = cache_rows(21, s, L, 0.5)
    q, kf, vf = frame_inputs(21, s, T, 0.5)
    n = L + T
    ramp = torch.arange(n, dtype=torch.float32) / n
    a = {"all_low": torch.full((n,), -10.0), "all_high": torch.full((n,), 10.0), "rising": 10.0 * ramp,
         "falling": -10.0 * ramp, "jump": 1.5 * (ramp > 0.5).float()}[mode]
    # k_j += a_j * u, q += 10 * u with u = 0.5 * ones: score_j moves by 0.1275 * 10 * a_j * 32 log2 units
    hk = (hk.float() + 0.5 * a[:L, None, None]).to(torch.bfloat16)
    kf = (kf.float() + 0.5 * a[L:, None, None]).to(torch.bfloat16)
    q = (q.float() + 5.0).to(torch.bfloat16)
    out, _, _ = run_prefill(s, hk, hv, L, q, kf, vf)
    check_close(out, oracle_prefill_rows(s, q, hk, hv, L, kf, vf), "bf16", f"{mode} L={L}")


@pytest.mark.parametrize("kv_groups", [1, 2])
@pytest.mark.parametrize("low", [1.0, 10.0, 38.0])
@pytest.mark.parametrize("value", [0.0, 2.0 ** -120, 2.0 ** -80])
def test_split_prefill_with_values_of_zero_or_next_to_it(value, low, kv_groups):
    """All scores `low` log2 units below 0 (a row's sum over a split's keys is then far below 1, its reciprocal large) and values
    of 0, or of next to nothing, in the keys of the first split or in all: a partial result is scaled by the
    reciprocal and by a power of two, which must not meet each other before they meet the values.  2 to 32 splits, all three merges."""
    s, T, L = AttnShape(8, 4, 128, "bf16"), 37, 2100
    hk, hv = cache_rows(71, s, L, 0.05)
    q, kf, vf = frame_inputs(71, s, T, 0.05)
    q = (q.float() + 1.0).to(torch.bfloat16)
    # (k_j - c against q + 1 moves score_j by 0.1275 * 128 * c log2 units)
    hk, kf = ((t.float() - low / 16.32).to(torch.bfloat16) for t in (hk, kf))
    vs.set_tuning(vs.TUNE_PREFILL_KV_GROUPS, kv_groups)
    for splits, merge in ((2, 0), (2, 1), (2, 2), (3, 0), (5, 1), (8, 0), (8, 2), (12, 0), (32, 0), (32, 2)):
        vs.set_tuning(vs.TUNE_PREFILL_SPLITS, splits)
        vs.set_tuning(vs.TUNE_PREFILL_MERGE, merge)
        for rows in (L // splits + 64, L):  # (the first split's keys are among the first, or all)
            v_c, v_f = hv.clone(), vf.clone()
            v_c[:rows] = value
            if rows == L:
                v_f[:] = value
            out, _, _ = run_prefill(s, hk, v_c, L, q, kf, v_f)
            what = f"V {value} in {rows} rows, {splits} splits, merge {merge}, {kv_groups} key groups"
            if rows == L and value < 2.0 ** -112:  # (below 2^-112 the power's inverse is 0 in fp32: such rows come out as 0)
                assert out.float().abs().max() <= value, what
            else:
                check_close(out, oracle_prefill_rows(s, q, hk, v_c, L, kf, v_f), "bf16", what, absolute=False)


@pytest.mark.parametrize("kv_groups", [1, 2])
@pytest.mark.parametrize("tiles,first_block,step", [(3, 2, 60.0), (4, 3, 60.0), (7, 4, 20.0), (7, 5, 20.0), (8, 6, 400.0), (8, 7, 400.0)])
def test_prefill_reference_left_behind_inside_the_loop_of_plain_steps(tiles, first_block, step, kv_groups):
    """Scores that jump at a chosen sub-block of 32 keys (even and odd ones, by `step` log2 units, and again two and three
    sub-blocks later), over so many whole tiles in one lane: the loop over plain steps is left behind either half of a step,
    the sub-block redone and the loop entered again, with an odd or even number of steps to go."""
    s, T = AttnShape(8, 4, 128, "bf16"), 70
    L = 64 * tiles * kv_groups + 5
    vs.set_tuning(vs.TUNE_PREFILL_KV_GROUPS, kv_groups)
    vs.set_tuning(vs.TUNE_PREFILL_SPLITS, 1)
    hk, hv = cache_rows(44, s, L, 0.5)
    q, kf, vf = frame_inputs(44, s, T, 0.5)
    block = torch.arange(L + T) // 32
    a = sum((block >= b).float() for b in (first_block, first_block + 2, first_block + 5)) * (step / 40.8)
    # (k_j += a_j u, q += 10 u with u = 0.5 ones: score_j moves by 0.1275 * 10 * a_j * 32 log2 units)
    hk = (hk.float() + 0.5 * a[:L, None, None]).to(torch.bfloat16)
    kf = (kf.float() + 0.5 * a[L:, None, None]).to(torch.bfloat16)
    q = (q.float() + 5.0).to(torch.bfloat16)
    out, _, _ = run_prefill(s, hk, hv, L, q, kf, vf)
    check_close(out, oracle_prefill_rows(s, q, hk, hv, L, kf, vf), "bf16", f"{tiles} tiles, block {first_block}, {kv_groups} key groups")


@pytest.mark.parametrize("kv_groups", [1, 2])
@pytest.mark.parametrize("far", [4, 0, -1])
def test_prefill_rows_of_which_one_lane_never_sums_anything(far, kv_groups):
    """A row's keys are shared out to two lanes by bit 2 of their number.  The keys with (far = 4) or without (0) that bit lie 200
    log2 units below the others, or first the ones and then, from the middle on, the others do (-1): a lane whose sum is 0
    goes through the loop of plain steps with its row, and its keys count from where they matter."""
    s, T = AttnShape(8, 4, 128, "bf16"), 70
    L = 64 * 8 * kv_groups + 5
    vs.set_tuning(vs.TUNE_PREFILL_KV_GROUPS, kv_groups)
    vs.set_tuning(vs.TUNE_PREFILL_SPLITS, 1)
    hk, hv = cache_rows(45, s, L, 0.5)
    q, kf, vf = frame_inputs(45, s, T, 0.5)
    j = torch.arange(L + T)
    low = (j & 4) == far if far >= 0 else ((j & 4) == 0) ^ (j % (64 * 8) >= 256)
    # (k_j += a_j u, q += 10 u with u = 0.5 ones: score_j moves by 0.1275 * 10 * a_j * 32 log2 units)
    a = low.float() * (-200.0 / 40.8)
    hk = (hk.float() + 0.5 * a[:L, None, None]).to(torch.bfloat16)
    kf = (kf.float() + 0.5 * a[L:, None, None]).to(torch.bfloat16)
    q = (q.float() + 5.0).to(torch.bfloat16)
    out, _, _ = run_prefill(s, hk, hv, L, q, kf, vf)
    check_close(out, oracle_prefill_rows(s, q, hk, hv, L, kf, vf), "bf16", f"bit 2 {far}, {kv_groups} key groups")


def test_prefill_uniform_scores_is_running_mean_at_full_size():
    """Q = 0: every row is the mean of its visible V rows (closed form, any size)."""
    s = QW
    L, T = 4296, 170
    hk, hv = cache_rows(14, s, L, 0.5)
    _, kf, vf = frame_inputs(14, s, T, 0.5)
    q = torch.zeros((T, s.n_q_heads, s.head_dim), dtype=torch.bfloat16)
    out, _, _ = run_prefill(s, hk, hv, L, q, kf, vf)
    v_all = np.concatenate([to_f64(hv), to_f64(vf)])
    csum = np.cumsum(v_all, axis=0)
    ref = np.stack([csum[L + t] / (L + t + 1) for t in range(T)])  # [T][Hkv][D]
    ref = np.repeat(ref, s.group, axis=1)
    check_close(out, ref, "bf16", "uniform scores")


def test_prefill_fp32_path_larger_shapes():
    for (hq, hkv, d, L, T) in [(4, 2, 128, 700, 9), (6, 3, 64, 0, 3), (8, 1, 64, 300, 40)]:
        s = AttnShape(hq, hkv, d, "f32")
        hk, hv = cache_rows(15, s, max(L, 1), 1.0)
        q, kf, vf = frame_inputs(15, s, T, 1.0)
        out, _, _ = run_prefill(s, hk, hv, L, q, kf, vf)
        check_close(out, oracle_prefill_rows(s, q, hk, hv, L, kf, vf), "f32", f"fp32 {hq}/{hkv}/{d} L={L}")


@pytest.mark.parametrize("dim,hq,hkv,L,T", [(64, 4, 1, 203, 128), (64, 4, 1, 203, 129), (128, 8, 2, 500, 64), (128, 8, 2, 500, 65),
                                            (128, 8, 8, 0, 70)])
def test_fp32_prefill_on_both_sides_of_the_chip(dim, hq, hkv, L, T):
    """Up to 512 workgroups and beyond, over one and several chunks of 256 keys."""
    s = AttnShape(hq, hkv, dim, "f32")
    hk, hv = cache_rows(43, s, max(L, 1), 1.0)
    q, kf, vf = frame_inputs(43, s, T, 1.0)
    out, _, _ = run_prefill(s, hk, hv, L, q, kf, vf)
    check_close(out, oracle_prefill_rows(s, q, hk, hv, L, kf, vf), "f32", f"fp32 {hq}/{hkv}/{dim} L={L} T={T}")


@pytest.mark.parametrize("path,L", [("prefill", 100), ("prefill, general kernel", 100), ("prefill", 1500), ("prefill, one split", 1500),
                                    ("prefill, general kernel, one split", 1500), ("fp32 prefill", 40),
                                    ("decode", 100), ("decode", 700), ("decode", 9300), ("fp32 decode", 300)])
def test_a_score_that_is_not_a_number_stays_in_its_row(path, L):
    """A query row that holds a NaN comes out as NaN; every other row is what it is without it, to a rounding (the
    softmax references of the rows of a wavefront may be refreshed at other tiles)."""
    s = AttnShape(28, 4, 128, "f32" if "fp32" in path else "bf16")
    sh, dt, T = vs_shape(s), torch_dtype(s.dtype), 1 if "decode" in path else 40
    hk, hv = cache_rows(45, s, L, 0.5)
    k, v = (torch.cat([t, torch.zeros_like(t[:1])]).to(DEV) for t in (hk, hv))
    q, kf, vf = (t.to(DEV) for t in frame_inputs(45, s, T, 0.5))
    if "general" in path:
        vs.set_tuning(vs.TUNE_PREFILL_KV_GROUPS, 1)
    if "one split" in path:
        vs.set_tuning(vs.TUNE_PREFILL_SPLITS, 1)
    ws = workspace(s, T, L + 1, 1)
    outs = []
    for bad in (False, True):
        qd = q.clone()
        if bad:
            qd[T // 2, 9, 17] = float("nan")
        out = torch.zeros(q.shape, dtype=dt, device=DEV)
        if "decode" in path:
            vs.decode_attn(sh, k[None], v[None], lens_array([L]), qd, None, None, out, ws)
        else:
            vs.frame_prefill_attn(sh, vs.Cache(k, v, L), qd, kf, vf, out, ws)
        torch.cuda.synchronize()
        outs.append(out)
    assert bool(torch.isfinite(outs[0]).all()) and bool(torch.isnan(outs[1][T // 2, 9]).all())
    outs[1][T // 2, 9] = outs[0][T // 2, 9]
    a, b = outs[0].float(), outs[1].float()
    assert bool((a - b).abs().max() <= 2 ** -7 * a.abs().max())


# ---------------------------------------------------------------------------- decode edges
def _decode_case(s, lens0, cap, seed, gain=1.0, with_new=True):
    S = len(lens0)
    dt = torch_dtype(s.dtype)
    sigma = 0.5 if s.dtype == "bf16" else 1.0
    ks = torch.zeros((S, cap, s.n_kv_heads, s.head_dim), dtype=dt, device=DEV)
    vsl = torch.zeros_like(ks)
    ok, ov = [], []
    for i in range(S):
        hk, hv = cache_rows(seed, s, max(lens0[i], 1), sigma, stream=i)
        ks[i, :lens0[i]].copy_(hk[:lens0[i]])
        vsl[i, :lens0[i]].copy_(hv[:lens0[i]])
        a, b = np.zeros((cap, s.n_kv_heads, s.head_dim)), np.zeros((cap, s.n_kv_heads, s.head_dim))
        a[:lens0[i]], b[:lens0[i]] = to_f64(hk[:lens0[i]]), to_f64(hv[:lens0[i]])
        ok.append(a)
        ov.append(b)
    q, kn, vn = decode_step_inputs(seed, s, S, sigma, q_gain=gain)
    lens = lens_array(lens0)
    out = torch.full(q.shape, float("nan"), dtype=dt, device=DEV)
    ws = workspace(s, 0, cap, S)
    vs.decode_attn(vs_shape(s), ks, vsl, lens, q.to(DEV), kn.to(DEV) if with_new else None,
                   vn.to(DEV) if with_new else None, out, ws)
    torch.cuda.synchronize()
    ref = np.zeros((S, s.n_q_heads, s.head_dim))
    for i in range(S):
        ref[i], n = oracle.decode(to_f64(q[i]), ok[i], ov[i], lens0[i], to_f64(kn[i]) if with_new else None,
                                  to_f64(vn[i]) if with_new else None, scale32(s))
        assert lens[i] == n
        assert np.array_equal(ks[i].double().cpu().numpy(), ok[i]) and np.array_equal(vsl[i].double().cpu().numpy(), ov[i])
    return out, ref, (q, kn, vn)


@pytest.mark.parametrize("lens0,gain", [([0], 1), ([1, 2, 30, 31, 32, 33, 126, 127, 128, 129, 1000, 5], 1),
                                        ([777], 8), ([8319, 640, 4000], 8)])
def test_decode_ragged_lengths(lens0, gain):
    out, ref, (q, kn, vn) = _decode_case(QW, lens0, 8384 if max(lens0) > 1000 else 1024, 21, gain)
    check_close(out, ref, "bf16", f"decode lens={lens0}")
    if lens0 == [0]:  # empty cache: the output is the new V row exactly
        assert same_bits(out[0].reshape(QW.n_kv_heads, QW.group, -1)[:, 0], vn[0])


def test_decode_without_new_row_and_many_streams():
    lens0 = [40 + 13 * i for i in range(70)]  # more than one launch worth of streams
    out, ref, _ = _decode_case(QW, lens0, 1024, 22, with_new=False)
    check_close(out, ref, "bf16", "decode, 70 streams, no append")


def test_decode_result_does_not_depend_on_the_chunking():
    ref_out = None
    for chunk in (128, 256, 1024, 8192):
        vs.set_tuning(vs.TUNE_DECODE_CHUNK_ROWS, chunk)
        out, ref, _ = _decode_case(QW, [3000, 129, 5000], 5120, 23, gain=4)
        check_close(out, ref, "bf16", f"chunk_rows={chunk}")
        if ref_out is None:
            ref_out = out.float()
        assert (out.float() - ref_out).abs().max().item() <= 2 ** -7 * ref_out.abs().max().item()


# (hq, hkv, lens): one share of 4 and of 8 tiles and one row more, a full chip of them; shares of 4 tiles up to
# 32 tiles; then 8 tiles, more than 8, 12 shares of a stream; ragged streams; other head counts; one stream that is
# over every limit
@pytest.mark.parametrize("hq,hkv,lens0", [
    (28, 4, [127]), (28, 4, [128]), (28, 4, [255]), (28, 4, [256]), (28, 4, [0, 31, 127, 5]), (28, 4, [100] * 64), (28, 4, [255] * 64),
    (28, 4, [700]), (28, 4, [1023, 1, 300]), (28, 4, [1024]), (28, 4, [3071, 200]), (28, 4, [700] * 16), (28, 4, [1500, 1400, 1000] * 3),
    (28, 4, [2900] * 7), (28, 4, [703] * 64), (8, 1, [3071, 17]), (16, 2, [1500, 60, 900]), (12, 6, [1500] * 4), (6, 6, [333, 2]),
    (8, 8, [255] * 32), (28, 4, [9300])])
@pytest.mark.parametrize("gain", [1, 8])
def test_decode_few_rows(hq, hkv, lens0, gain):
    """The decode step that merges inside its launch, at the edges of its plan."""
    s = AttnShape(hq, hkv, 128, "bf16")
    out, ref, _ = _decode_case(s, lens0, max(lens0) + 1, 27, gain, with_new=gain == 1 or 0 in lens0)
    check_close(out, ref, "bf16", f"decode Hq={hq} Hkv={hkv} lens={lens0[:4]} x{len(lens0)} gain={gain}")


def test_decode_few_rows_replayed():
    """The arrival counters are back where they started after every launch: a captured chain of steps of different
    plans over one workspace gives the same bits on every replay, with eager work of the program in between."""
    cap = 3200
    g = torch.Generator(device=DEV).manual_seed(5)
    k, v, q = (torch.randn(d, generator=g, device=DEV, dtype=torch.bfloat16) for d in ((16, cap, 4, 128), (16, cap, 4, 128), (16, 28, 128)))
    sh = vs_shape(QW)
    ws = vs.make_workspace(sh, 0, cap, 16, DEV)
    plans = [[700], [3000] * 4, [100] * 16, [700] * 16, [900]]
    outs = [torch.empty_like(q[:len(p)]) for p in plans]

    def steps():
        st = vs.current_stream_handle()
        for p, out in zip(plans, outs):
            n = len(p)
            vs.decode_attn(sh, k[:n], v[:n], lens_array(p), q[:n], None, None, out, ws, stream=st)

    steps()
    torch.cuda.synchronize()
    want = [o.clone() for o in outs]
    graph, nodes = _captured(steps)
    assert nodes == len(plans)
    for _ in range(8):
        for o in outs:
            o.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(o.view(torch.int16), w.view(torch.int16)) for o, w in zip(outs, want))
        steps()
    torch.cuda.synchronize()


@pytest.mark.parametrize("left", ["zeros", "ones", "sums", "other calls"])
def test_decode_over_a_control_block_that_holds_something_else(left):
    """Shared-out steps over a workspace that was never prepared, or has served other calls since, are right; and
    vs_workspace_init gives the bits of a fresh workspace again, also over counts that were left behind."""
    s, lens0, cap = QW, [700, 3000, 64, 1500], 3200
    sh, n = vs_shape(s), len(lens0)
    kv = [cache_rows(61, s, cap, 0.5, stream=i) for i in range(n)]
    k, v = (torch.stack([c[j] for c in kv]).to(DEV) for j in (0, 1))
    hq, _, _ = decode_step_inputs(61, s, n, 0.5, q_gain=4)
    q = hq.to(DEV)
    ws = vs.make_workspace(sh, 0, cap, n, DEV)

    def step():
        out = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device=DEV)
        vs.decode_attn(sh, k, v, lens_array(lens0), q, None, None, out, ws)
        torch.cuda.synchronize()
        return out

    fresh = step()
    ref = np.stack([oracle.decode(to_f64(hq[i]), to_f64(kv[i][0]), to_f64(kv[i][1]), m, None, None, scale32(s))[0]
                    for i, m in enumerate(lens0)])
    check_close(fresh, ref, "bf16", "decode, fresh workspace")
    if left == "zeros":
        ws.zero_()
    elif left == "ones":
        ws.fill_(0xFF)
    elif left == "sums":
        ws.view(torch.float32)[:] = torch.randn(ws.numel() // 4, device=DEV)
    else:  # a product's shares and a bank's cosines lie at the start of their workspaces
        w = draw(62, (512, 3584), 0.2, "bf16").to(DEV)
        o = torch.empty((170, 512), dtype=torch.bfloat16, device=DEV)
        assert 0 < vs.linear_workspace_bytes(170, 3584, 512) <= ws.numel()
        vs.linear(draw(63, (170, 3584), 1.0, "bf16").to(DEV), w, o, workspace=ws)
        e = draw(64, (128, 256), 1.0, "bf16").to(DEV)
        victim = torch.zeros(1, dtype=torch.int32, device=DEV)
        vs.memory_bank_push(vs.Bank(e, "bf16", 128), e[3].clone(), victim, ws)
    for _ in range(3):
        check_close(step(), ref, "bf16", f"decode, control block: {left}")
    ws[:4096].view(torch.int32).add_(3)  # counts that nobody will finish
    vs.workspace_init(sh, ws)
    for _ in range(2):
        assert torch.equal(step().view(torch.int16), fresh.view(torch.int16))


@pytest.mark.parametrize("n,rows,shared_out", [(1, 700, True), (4, 100, False), (4, 700, True)])
def test_decode_static_counts_nothing_in_its_array(n, rows, shared_out):
    """The library's own array cannot be cleared, so a call over it may not rely on what an earlier one left there:
    where rows are shared out, a second launch adds the shares (two nodes of a captured step, one with a
    workspace); where they are not, one launch does."""
    sh = vs_shape(QW)
    k, v, q = (torch.randn(d, device=DEV).to(torch.bfloat16) for d in ((n, 800, 4, 128), (n, 800, 4, 128), (n, 28, 128)))
    ws = vs.make_workspace(sh, 0, 800, n, DEV)
    out = torch.empty_like(q)
    own = lambda: vs.decode_attn_static(sh, k, v, lens_array([rows] * n), q, None, None, out)
    given = lambda: vs.decode_attn(sh, k, v, lens_array([rows] * n), q, None, None, out, ws)
    for call, nodes in ((given, 1), (own, 2 if shared_out else 1)):
        call()
        torch.cuda.synchronize()
        want = out.clone()
        graph, count = _captured(call)
        assert count == nodes
        for _ in range(3):
            out.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("hq,hkv", [(6, 3), (12, 6), (5, 5), (16, 2), (8, 1), (24, 8)])
@pytest.mark.parametrize("chunk", [0, 32])
def test_decode_other_kv_head_counts(hq, hkv, chunk):
    """KV head counts that are not multiples of 4 (a workgroup then takes 1 or 2 heads and its spare
    wavefronts take sub-ranges of the share), with the library's own shares and with the smallest
    ones (one tile per share: the most workgroups, the highest partial-result slots)."""
    s = AttnShape(hq, hkv, 128, "bf16")
    vs.set_tuning(vs.TUNE_DECODE_CHUNK_ROWS, chunk)
    lens0 = [3000, 1, 129, 64, 700, 33] + [40 + 37 * i for i in range(20)]
    out, ref, _ = _decode_case(s, lens0, 3072, 26, gain=4)
    check_close(out, ref, "bf16", f"decode Hq={hq} Hkv={hkv} chunk_rows={chunk}")


def test_decode_equals_one_token_prefill():
    s, L = QW, 900
    out, ref, (q, kn, vn) = _decode_case(s, [L], 1024, 24, gain=4)
    hk, hv = cache_rows(24, s, L, 0.5, stream=0)
    pre, _, _ = run_prefill(s, hk, hv, L, q[0:1], kn[0:1], vn[0:1])
    check_close(pre, ref, "bf16", "one-token prefill vs oracle decode")
    assert (pre.float() - out.float()).abs().max().item() <= 2 ** -7 * out.float().abs().max().item()


def test_decode_fp32_path():
    s = AttnShape(4, 2, 64, "f32")
    out, ref, _ = _decode_case(s, [5, 300, 1], 512, 25)
    check_close(out, ref, "f32", "fp32 decode")


def test_prefill_largest_run_and_head_ratio():
    """4096 tokens in one run (the limit), 8 query heads per KV head (the limit): 32768 query rows
    per KV head, 256 row tiles; sampled tokens against the oracle."""
    s = AttnShape(16, 2, 128, "bf16")
    L, T = 300, 4096
    hk, hv = cache_rows(71, s, L, 0.5)
    q, kf, vf = frame_inputs(71, s, T, 0.5, q_gain=2)
    tokens = np.array([0, 1, 63, 64, 127, 128, 1000, 2047, 2048, 3333, 4094, 4095])
    ref = oracle_prefill_rows(s, q, hk, hv, L, kf, vf, tokens)
    out, cache, row = run_prefill(s, hk, hv, L, q, kf, vf, capacity=L + 1, fused=True)
    check_close(out[torch.from_numpy(tokens).to(DEV)], ref, "bf16", "4096-token run, 8 heads per KV head")
    assert row == L and cache.len == L + 1 and same_bits(cache.k[L], kf[T - 1]) and same_bits(cache.v[L], vf[T - 1])
    assert bool(torch.isfinite(out.float()).all())
    c = vs.Cache(cache.k, cache.v, L)
    too_many = torch.empty((4097, s.n_q_heads, s.head_dim), dtype=torch.bfloat16, device=DEV)
    with pytest.raises(vs.VSError):
        vs.frame_prefill_attn(vs_shape(s), c, too_many, too_many, too_many, too_many, workspace(s, 4096, L + 1, 0))


def test_decode_longest_stream_mix():
    """64 streams in one launch (the most one launch takes), lengths from 1 row to 12000 rows."""
    s = QW
    lens0 = [12000, 1, 2, 31, 32, 33] + [int(x) for x in np.random.default_rng(9).integers(1, 3000, size=58)]
    out, ref, _ = _decode_case(s, lens0, 12008, 27, gain=4)
    check_close(out, ref, "bf16", "64 streams, up to 12000 rows")


# ---------------------------------------------------------------------------- the question after the video
@pytest.mark.parametrize("L,Tq,dtype,splits", [(4424, 32, "bf16", 0), (200, 7, "bf16", 0), (0, 19, "bf16", 0),
                                                (1500, 130, "bf16", 3), (700, 1, "bf16", 0), (300, 600, "bf16", 0),
                                                (150, 9, "f32", 0)])
def test_question_prefill_keeps_all_rows_and_decoding_continues(L, Tq, dtype, splits):
    """vs_question_prefill_append against the oracle's token-by-token evaluation: outputs, the Tq
    rows appended bit for bit, the length; then one decoding step on top of them."""
    s = QW if dtype == "bf16" else AttnShape(4, 2, 64, "f32")
    dt = torch_dtype(dtype)
    cap = L + Tq + 4
    hk, hv = cache_rows(61, s, L, 0.5)
    q, kt, vt = frame_inputs(61, s, Tq, 0.5, q_gain=4)
    Kc, Vc = np.zeros((cap, s.n_kv_heads, s.head_dim)), np.zeros((cap, s.n_kv_heads, s.head_dim))
    if L:
        Kc[:L], Vc[:L] = to_f64(hk), to_f64(hv)
    ref, n = oracle.query_prefill(to_f64(q), Kc, Vc, L, to_f64(kt), to_f64(vt), scale32(s))
    assert n == L + Tq
    k = torch.full((cap, s.n_kv_heads, s.head_dim), 7.0, dtype=dt, device=DEV)  # junk beyond len must not count
    v = torch.full_like(k, -7.0)
    if L:
        k[:L].copy_(hk)
        v[:L].copy_(hv)
    cache = vs.Cache(k, v, L)
    ws = workspace(s, Tq, cap, 1)
    vs.set_tuning(vs.TUNE_PREFILL_SPLITS, splits)
    out = torch.full(q.shape, float("nan"), dtype=dt, device=DEV)
    vs.question_prefill_append(vs_shape(s), cache, q.to(DEV), kt.to(DEV), vt.to(DEV), out, ws)
    torch.cuda.synchronize()
    vs.set_tuning(vs.TUNE_PREFILL_SPLITS, 0)
    check_close(out, ref, dtype, f"question L={L} Tq={Tq}")
    assert cache.len == L + Tq
    assert same_bits(cache.k[L:L + Tq], kt) and same_bits(cache.v[L:L + Tq], vt)
    assert bool((cache.k[L + Tq:] == 7.0).all()) and bool((cache.v[L + Tq:] == -7.0).all())
    if L:
        assert same_bits(cache.k[:L], hk) and same_bits(cache.v[:L], hv)
    # the answer's first token
    qd, kn, vn = decode_step_inputs(62, s, 1, 0.5, step=0)
    o_ref, n2 = oracle.decode(to_f64(qd[0]), Kc, Vc, n, to_f64(kn[0]), to_f64(vn[0]), scale32(s))
    lens = lens_array([cache.len])
    od = torch.empty((1, s.n_q_heads, s.head_dim), dtype=dt, device=DEV)
    vs.decode_attn(vs_shape(s), k[None], v[None], lens, qd.to(DEV), kn.to(DEV), vn.to(DEV), od, ws)
    torch.cuda.synchronize()
    check_close(od[0], o_ref, dtype, f"decoding step after the question, L={L} Tq={Tq}")
    assert lens[0] == n2 == L + Tq + 1


# ---------------------------------------------------------------------------- the frame's rows and their projections
def _projection_case(s, N, d, seed):
    e = draw(seed, (N, d), 1.0, "bf16")
    n_out = (s.n_q_heads + 2 * s.n_kv_heads) * s.head_dim
    w = draw(seed + 1, (n_out, d), d ** -0.5, "bf16")
    rq, rk, rv = oracle.frame_qkv(to_f64(e), to_f64(w), s.n_q_heads, s.n_kv_heads, s.head_dim)
    sh = vs_shape(s)
    q = torch.full((N + 1, s.n_q_heads, s.head_dim), float("nan"), dtype=torch.bfloat16, device=DEV)
    k = torch.full((N + 1, s.n_kv_heads, s.head_dim), float("nan"), dtype=torch.bfloat16, device=DEV)
    v = torch.full_like(k, float("nan"))
    c = torch.full((d,), float("nan"), dtype=torch.bfloat16, device=DEV)
    outs = []
    for rep in range(2):
        vs.frame_qkv_project(sh, e.to(DEV), w.to(DEV), q, k, v, c_out=c)
        torch.cuda.synchronize()
        outs.append((q.clone(), k.clone(), v.clone()))
    assert all(same_bits(a, b.cpu()) for a, b in zip(outs[1], outs[0])), "the same call twice gives the same bits"
    return (q, k, v, c), (rq, rk, rv), (e, w)


@pytest.mark.parametrize("N,d,heads", [(169, 3584, (28, 4)), (49, 256, (8, 2)), (1, 64, (8, 8)), (191, 448, (16, 2)),
                                        (16, 128, (8, 1)), (100, 1024, (12, 4)), (160, 64, (3, 1)), (17, 192, (7, 1))])
def test_frame_projection_matches_oracle(N, d, heads):
    """vs_frame_qkv_project against the oracle: every row incl. the carrier's, Q/K/V in the layouts
    the prefill takes; the carrier embedding equals vs_carrier_mean_pool bit for bit."""
    s = AttnShape(heads[0], heads[1], 128, "bf16")
    (q, k, v, c), (rq, rk, rv), (e, w) = _projection_case(s, N, d, 500 + N)
    check_close(q, rq, "bf16", f"Q N={N} d={d}")
    check_close(k, rk, "bf16", f"K N={N} d={d}")
    check_close(v, rv, "bf16", f"V N={N} d={d}")
    pooled = torch.empty(d, dtype=torch.bfloat16, device=DEV)
    vs.carrier_mean_pool(e.to(DEV), pooled, "bf16")
    torch.cuda.synchronize()
    assert same_bits(c, pooled.cpu())
    # without the embedding asked for, the same Q/K/V
    q2, k2, v2 = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
    vs.frame_qkv_project(vs_shape(s), e.to(DEV), w.to(DEV), q2, k2, v2)
    torch.cuda.synchronize()
    assert same_bits(q2, q.cpu()) and same_bits(k2, k.cpu()) and same_bits(v2, v.cpu())


@pytest.mark.parametrize("N,d,heads", [
    # rows at the edges of the 16-row groups and of the 64-row classes; d of one tile, of as many as the ring holds
    # (5, 6) and one more, odd and even; counts of workgroups that are no multiple of 8, and with no compute unit
    # left over for helpers
    (1, 64, (8, 1)), (15, 128, (5, 5)), (16, 320, (6, 3)), (17, 384, (6, 3)), (63, 448, (5, 5)), (64, 320, (8, 1)), (65, 64, (5, 5)),
    (112, 192, (6, 3)), (128, 384, (8, 8)), (129, 320, (5, 5)), (144, 128, (48, 8)), (161, 448, (40, 8)), (191, 384, (12, 6)),
    # 192 workgroups: with helpers, and with too few of them to pay; 12 workgroups: fewer helpers than idle compute units
    (191, 1280, (32, 8)), (100, 1280, (32, 8)), (169, 512, (1, 1)),
])
def test_frame_projection_row_groups_ring_and_helpers(N, d, heads):
    s = AttnShape(heads[0], heads[1], 128, "bf16")
    (q, k, v, c), (rq, rk, rv), (e, _) = _projection_case(s, N, d, 1500 + N)
    check_close(q, rq, "bf16", f"Q N={N} d={d}")
    check_close(k, rk, "bf16", f"K N={N} d={d}")
    check_close(v, rv, "bf16", f"V N={N} d={d}")
    pooled = torch.empty(d, dtype=torch.bfloat16, device=DEV)
    vs.carrier_mean_pool(e.to(DEV), pooled, "bf16")
    torch.cuda.synchronize()
    assert same_bits(c, pooled.cpu())


def test_frame_projection_feeds_the_prefill():
    """E and W in, attention out: projection, then prefill with compaction, against the oracle's
    projection followed by its prefill (inputs of the second stage rounded to bf16 on both sides)."""
    s, N, d, L = QW, 169, 3584, 300
    (q, k, v, c), (rq, rk, rv), _ = _projection_case(s, N, d, 91)
    hk, hv = cache_rows(92, s, L, 0.5)
    out, cache, row = run_prefill(s, hk, hv, L, q.cpu(), k.cpu(), v.cpu(), capacity=L + 1, fused=True)
    ref = oracle_prefill_rows(s, q.cpu(), hk, hv, L, k.cpu(), v.cpu())
    check_close(out, ref, "bf16", "prefill on projected rows")
    assert row == L and same_bits(cache.k[L], k[N].cpu()) and same_bits(cache.v[L], v[N].cpu())


# ---------------------------------------------------------------------------- pool, batched append
@pytest.mark.parametrize("n,d,dtype", [(169, 3584, "bf16"), (49, 256, "f32"), (1, 8, "bf16"), (7, 1000, "f32")])
def test_mean_pool(n, d, dtype):
    e = draw(31, (n, d), 1.0, dtype)
    out = torch.empty(d, dtype=torch_dtype(dtype), device=DEV)
    vs.carrier_mean_pool(e.to(DEV), out, dtype)
    torch.cuda.synchronize()
    ref = oracle.mean_pool(to_f64(e))
    got = out.double().cpu().numpy()
    if dtype == "f32":
        assert np.abs(got - ref).max() <= 1e-6
    else:  # one bf16 rounding of an fp32 mean
        assert np.all(np.abs(got - ref) <= np.abs(ref) * 2.0 ** -8 + 1e-30)


@pytest.mark.parametrize("n,d,dtype", [(191, 72, "bf16"), (192, 64, "bf16"), (193, 200, "bf16"), (385, 36, "f32"),
                                       (16, 72, "bf16"), (17, 36, "f32"), (64, 200, "bf16"), (65, 36, "f32"), (17, 32776, "bf16"),
                                       (200, 16388, "f32")])
def test_mean_pool_around_one_trip(n, d, dtype):
    """Row counts around what a thread requests at once (1, 4 or 12 rows of 16 row groups), ragged column blocks of both widths: bit for
    bit the sum in the documented order, 16 row groups in order and then their sums in order."""
    e = draw(32, (n, d), 1.0, dtype)
    out = torch.empty(d, dtype=torch_dtype(dtype), device=DEV)
    vs.carrier_mean_pool(e.to(DEV), out, dtype)
    parts = []
    for g in range(16):
        acc = torch.zeros(d)
        for r in range(g, n, 16):
            acc = acc + e[r].float()
        parts.append(acc)
    tot = parts[0]
    for part in parts[1:]:
        tot = tot + part
    assert same_bits(out, (tot / float(n)).to(torch_dtype(dtype)))


@pytest.mark.parametrize("dim,L,T,n_kept,overlap", [(64, 0, 1, 1, False), (64, 63, 50, 1, False), (128, 250, 9, 9, False),
                                                    (64, 16, 20, 20, True), (64, 16, 20, 1, True)])
def test_fp32_prefill_appends_in_its_launch(dim, L, T, n_kept, overlap):
    """The kept rows are copied by the attention launch; a run that lies where they go is copied after it."""
    s = AttnShape(4, 2, dim, "f32")
    hk, hv = cache_rows(41, s, max(L, 1), 1.0)
    q, kf, vf = frame_inputs(42, s, T, 1.0)
    k = torch.full((L + T + 3, 2, dim), 7.0, device=DEV)
    v = torch.full_like(k, -7.0)
    k[:L].copy_(hk[:L])
    v[:L].copy_(hv[:L])
    cache = vs.Cache(k, v, L)
    at = L + 1 if n_kept == 1 else L  # (the run's rows in the cache; all kept: they are where they go)
    kd, vd = (k[at:at + T], v[at:at + T]) if overlap else (torch.empty_like(kf, device=DEV), torch.empty_like(vf, device=DEV))
    kd.copy_(kf)
    vd.copy_(vf)
    out = torch.full(q.shape, float("nan"), device=DEV)
    ws = vs.make_workspace(vs_shape(s), T, L + T, 1, DEV)
    call = vs.question_prefill_append if n_kept == T and T > 1 else vs.frame_prefill_compact
    call(vs_shape(s), cache, q.to(DEV), kd, vd, out, ws)
    check_close(out, oracle_prefill_rows(s, q, hk, hv, L, kf, vf), "f32", f"fp32 append D={dim} L={L} T={T}")
    assert cache.len == L + n_kept
    assert same_bits(k[L:L + n_kept], kf[T - n_kept:]) and same_bits(v[L:L + n_kept], vf[T - n_kept:])
    if not overlap:
        assert bool((k[L + n_kept:] == 7).all()) and bool((v[L + n_kept:] == -7).all())


@pytest.mark.parametrize("call,F,T,L,at", [
    ("frame", 1, 170, 40, 0), ("frame", 1, 170, 1500, 0), ("frame", 1, 2000, 100, 0), ("frame", 1, 50, 300, 2), ("frame", 1, 1, 300, 0),
    ("question", 1, 37, 200, 0), ("question", 1, 37, 2000, 0), ("question", 1, 37, 2000, 5), ("question", 1, 900, 64, 1),
    ("frames", 3, 50, 700, 0), ("frames", 5, 2, 90, 0), ("frames", 12, 170, 64, 0), ("frames", 4, 33, 200, 3)])
def test_run_that_lies_in_the_cache_where_its_kept_rows_go(call, F, T, L, at):
    """A run projected straight into the cache, at row len + at: the same bits, in the outputs and the kept rows, as from
    tensors of its own.  (Long runs take several rounds of workgroups, which all read the run's first rows.)"""
    s = QW
    sh, rows = vs_shape(s), F * T
    hk, hv = cache_rows(44, s, L, 0.5)
    q, kf, vf = (t.to(DEV) for t in frame_inputs(44, s, rows, 0.5, q_gain=3))
    kept = {"frame": 1, "question": T, "frames": F}[call]
    need = vs.frames_workspace_bytes(sh, F, T, L + F) if call == "frames" else vs.workspace_bytes(sh, T, L, 0)
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    vs.workspace_init(sh, ws)
    got = []
    for in_cache in (False, True):
        k, v = (torch.full((L + at + rows + 2, s.n_kv_heads, s.head_dim), 3.0, dtype=torch.bfloat16, device=DEV) for _ in range(2))
        k[:L].copy_(hk)
        v[:L].copy_(hv)
        kd, vd = (k[L + at:L + at + rows], v[L + at:L + at + rows]) if in_cache else (kf, vf)
        if in_cache:
            kd.copy_(kf)
            vd.copy_(vf)
        cache = vs.Cache(k, v, L)
        out = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device=DEV)
        if call == "frames":
            vs.frames_prefill_attn(sh, cache, *(t.view(F, T, *t.shape[1:]) for t in (q, kd, vd, out)), ws)
        else:
            (vs.frame_prefill_compact if call == "frame" else vs.question_prefill_append)(sh, cache, q, kd, vd, out, ws)
        torch.cuda.synchronize()
        assert cache.len == L + kept
        got.append((out, k[:L + kept].clone(), v[:L + kept].clone()))
    for apart, inside in zip(*got):
        assert torch.equal(apart.view(torch.int16), inside.view(torch.int16))


@pytest.mark.parametrize("n_caches,pinned", [(28, False), (4096, False), (4095, True), (4096, True), (4097, True), (50, True)])
def test_batched_compaction(n_caches, pinned):
    s, T, cap = QW, 6, 5
    rng = np.random.default_rng(5)
    lens0 = rng.integers(0, cap, size=n_caches).tolist()
    if pinned:  # lengths in a pinned host tensor, row indices into a caller's array
        lens_t = torch.tensor(lens0, dtype=torch.int32).pin_memory()
        ks = torch.zeros((n_caches, cap, s.n_kv_heads, s.head_dim), dtype=torch.bfloat16, device=DEV)
        vsl = torch.zeros_like(ks)
        kf = draw(41, (n_caches, T, s.n_kv_heads, s.head_dim), 0.5, "bf16")
        vf = draw(42, (n_caches, T, s.n_kv_heads, s.head_dim), 0.5, "bf16")
        # rows into a pinned tensor (the device copy is taken from it), into a plain array, or
        # nowhere (then the call waits for the stream, lens being pinned)
        rows_c = [torch.zeros(n_caches, dtype=torch.int32).pin_memory(), (ctypes.c_int32 * n_caches)(), None][n_caches % 3]
        got = vs.carrier_compact_append_batched(vs_shape(s), ks, vsl, lens_t, kf.to(DEV), vf.to(DEV),
                                                workspace=workspace(s, 0, 0, n_caches), rows_out=rows_c)
        torch.cuda.synchronize()
        assert (got is rows_c if rows_c is not None else got == lens0) and lens_t.tolist() == [n + 1 for n in lens0]
        assert rows_c is None or [int(x) for x in rows_c] == lens0
        idx = torch.tensor(lens0)
        ar = torch.arange(n_caches)
        assert same_bits(ks[ar, idx], kf[:, T - 1]) and same_bits(vsl[ar, idx], vf[:, T - 1])
        assert int((ks != 0).any(dim=-1).any(dim=-1).sum()) == n_caches  # one row per cache, no other
        return
    ks = torch.zeros((n_caches, cap, s.n_kv_heads, s.head_dim), dtype=torch.bfloat16, device=DEV)
    vsl = torch.zeros_like(ks)
    kf = draw(41, (n_caches, T, s.n_kv_heads, s.head_dim), 0.5, "bf16")
    vf = draw(42, (n_caches, T, s.n_kv_heads, s.head_dim), 0.5, "bf16")
    lens = lens_array(lens0)
    ws = workspace(s, 0, 0, n_caches)
    rows = vs.carrier_compact_append_batched(vs_shape(s), ks, vsl, lens, kf.to(DEV), vf.to(DEV), workspace=ws)
    torch.cuda.synchronize()
    assert rows == lens0 and list(lens) == [n + 1 for n in lens0]
    want_k, want_v = torch.zeros(ks.shape, dtype=torch.bfloat16), torch.zeros(ks.shape, dtype=torch.bfloat16)
    for i in range(n_caches):
        want_k[i, lens0[i]] = kf[i, T - 1]
        want_v[i, lens0[i]] = vf[i, T - 1]
    assert same_bits(ks, want_k) and same_bits(vsl, want_v)


# ---------------------------------------------------------------------------- memory bank
@pytest.mark.parametrize("dtype,M,d,policy", [("bf16", 128, 3584, 0), ("f32", 16, 256, 0), ("bf16", 64, 3584, 1),
                                              ("bf16", 5, 8, 0), ("f32", 130, 64, 0)])
def test_memory_bank_stream(dtype, M, d, policy):
    """Carriers arrive one by one: the bank fills, then drops the older carrier of the most similar
    adjacent pair.  Victim indices against the fp64 oracle (the device sums in fp64 too, in another
    order: equal whenever the two best cosines differ by more than 1e-6, far above what the order of
    summation can move), embeddings and the K/V rows of three layers bit for bit."""
    s = AttnShape(4, 2, 64, "f32") if dtype == "f32" else QW
    n_layers, first, extra = 3, 5, 40
    n = M + extra
    emb = carrier_embeddings(7, n, d, dtype)
    kv = draw(99, (n, n_layers, 2, s.n_kv_heads, s.head_dim), 1.0, dtype)   # [carrier][layer][k|v]
    dt = torch_dtype(dtype)
    bank = vs.Bank(torch.zeros((M, d), dtype=dt, device=DEV), dtype)
    caches = [vs.Cache(torch.full((first + M + 2, s.n_kv_heads, s.head_dim), 7.0, dtype=dt, device=DEV),
                       torch.full((first + M + 2, s.n_kv_heads, s.head_dim), -7.0, dtype=dt, device=DEV), first)
              for _ in range(n_layers)]
    victim = torch.full((1,), -5, dtype=torch.int32, device=DEV)
    ws = torch.empty(vs.memory_bank_workspace_bytes(M), dtype=torch.uint8, device=DEV)
    # the oracle's state
    o_emb = np.zeros((M, d))
    o_k = [np.full((first + M + 2, s.n_kv_heads, s.head_dim), 7.0) for _ in range(n_layers)]
    o_v = [np.full((first + M + 2, s.n_kv_heads, s.head_dim), -7.0) for _ in range(n_layers)]
    o_n = 0
    near_ties = 0
    for t in range(n):
        e_dev = emb[t].to(DEV)
        rows = kv[t].to(DEV)
        vs.memory_bank_push(bank, e_dev, victim, ws, policy=policy)
        vs.carrier_evict_append(vs_shape(s), caches, first, M, rows[:, 0], rows[:, 1], victim)
        got = int(victim.cpu()[0])
        e64 = to_f64(emb[t])
        if o_n < M:
            assert got == -1
            want = -1
        else:
            want, cos = oracle.bank_victim(o_emb, e64, policy)
            top = np.sort(cos)[::-1]
            assert 0 <= got < M and cos[got] >= top[0] - 1e-6, f"carrier {t}: victim {got}, cosine {cos[got]} vs best {top[0]}"
            if top[0] - top[1] > 1e-6:
                assert got == want, f"carrier {t}: victim {got}, oracle {want}"
            else:
                near_ties += 1
        n2 = oracle.bank_apply(o_emb, 0, M, o_n, got, e64)
        for l in range(n_layers):
            oracle.bank_apply(o_k[l], first, M, o_n, got, to_f64(kv[t, l, 0]))
            oracle.bank_apply(o_v[l], first, M, o_n, got, to_f64(kv[t, l, 1]))
        o_n = n2
        assert bank.len == o_n and all(c.len == first + o_n for c in caches)
        if t % 13 == 0 or t >= n - 3:
            assert np.array_equal(bank.e.double().cpu().numpy(), o_emb), f"embeddings after carrier {t}"
            for l in range(n_layers):
                assert np.array_equal(caches[l].k.double().cpu().numpy(), o_k[l]), f"K rows of layer {l} after carrier {t}"
                assert np.array_equal(caches[l].v.double().cpu().numpy(), o_v[l]), f"V rows of layer {l} after carrier {t}"
    assert near_ties <= extra // 4


@pytest.mark.parametrize("dtype,M,d", [("bf16", 33, 4104), ("f32", 257, 2052), ("bf16", 258, 72), ("bf16", 600, 8), ("f32", 1, 4),
                                       ("bf16", 40, 512), ("bf16", 40, 520), ("f32", 40, 516)])
def test_memory_bank_at_the_edges_of_a_pass(dtype, M, d):
    """Banks around what one pass of the row move holds (256 rows), embeddings around what the cosines take
    through LDS at a time (8 KB) and around those they do not take through it (512 numbers): victims against the fp64 oracle, the moved rows bit for bit."""
    dt = torch_dtype(dtype)
    emb = carrier_embeddings(11, M + 6, d, dtype)
    bank = vs.Bank(emb[:M].clone().to(DEV), dtype, M)
    victim = torch.full((1,), -5, dtype=torch.int32, device=DEV)
    ws = torch.empty(vs.memory_bank_workspace_bytes(M), dtype=torch.uint8, device=DEV)
    dim = 64 if dtype == "f32" else 128
    shape = vs.Shape.make(4, 2, dim, dtype)
    rows = draw(12, (M + 6, 2, 2, dim), 1.0, dtype)
    cache = vs.Cache(rows[:M, 0].contiguous().to(DEV), rows[:M, 1].contiguous().to(DEV), M)
    want, want_k, want_v = emb[:M].clone(), rows[:M, 0].clone(), rows[:M, 1].clone()
    for t in range(M, M + 6):
        vs.memory_bank_push(bank, emb[t].to(DEV), victim, ws)
        k_new, v_new = (rows[t:t + 1, i].contiguous().to(DEV) for i in (0, 1))
        vs.carrier_evict_append(shape, [cache], 0, M, k_new, v_new, victim)
        got = int(victim.cpu()[0])
        expect, cos = oracle.bank_victim(to_f64(want), to_f64(emb[t]))
        assert got == expect or abs(cos[got] - cos[expect]) <= 1e-6
        move = lambda rows_, new: torch.cat([rows_[:got], rows_[got + 1:], new[None]])
        want, want_k, want_v = move(want, emb[t]), move(want_k, rows[t, 0]), move(want_v, rows[t, 1])
        assert same_bits(bank.e, want) and same_bits(cache.k, want_k) and same_bits(cache.v, want_v)
        assert cache.len == M and bank.len == M


def test_memory_bank_ties_and_zero_vectors():
    """Equal cosines: the smallest index goes; a zero vector has cosine 0 and never wins over a
    positive one."""
    M, d = 6, 16
    e = torch.zeros((M, d), dtype=torch.float32)
    e[0, 0] = 1.0
    e[1, 1] = 2.0
    e[2, 1] = 0.5          # pair (1, 2): cosine 1
    e[3, 2] = 1.0
    e[4, 3] = 3.0
    e[5, 3] = 1.0          # pair (4, 5): cosine 1 as well
    new = torch.zeros(d)
    bank = vs.Bank(e.to(DEV), "f32", M)
    victim = torch.zeros(1, dtype=torch.int32, device=DEV)
    ws = torch.empty(vs.memory_bank_workspace_bytes(M), dtype=torch.uint8, device=DEV)
    vs.memory_bank_push(bank, new.to(DEV), victim, ws)
    assert int(victim.cpu()[0]) == 1 == oracle.bank_victim(e.double().numpy(), new.double().numpy())[0]
    want = e.double().numpy().copy()
    oracle.bank_apply(want, 0, M, M, 1, new.double().numpy())
    assert np.array_equal(bank.e.double().cpu().numpy(), want)


def test_memory_bank_rejects_bad_arguments():
    s = QW
    e = torch.zeros((4, 8), dtype=torch.bfloat16, device=DEV)
    victim = torch.zeros(1, dtype=torch.int32, device=DEV)
    ws = torch.empty(256, dtype=torch.uint8, device=DEV)
    bank = vs.Bank(e, "bf16")
    with pytest.raises(vs.VSError) as err:
        vs.memory_bank_push(bank, e[0], victim, ws, policy=3)
    assert err.value.code == 2
    with pytest.raises(vs.VSError) as err:
        vs.memory_bank_push(bank, e[0], victim, ws[:8])
    assert err.value.code == 5 and bank.len == 0
    k = torch.zeros((6, s.n_kv_heads, s.head_dim), dtype=torch.bfloat16, device=DEV)
    cache = vs.Cache(k, k.clone(), 2)
    rows = torch.zeros((1, s.n_kv_heads, s.head_dim), dtype=torch.bfloat16, device=DEV)
    with pytest.raises(vs.VSError) as err:       # prefix + bank does not fit the cache
        vs.carrier_evict_append(vs_shape(s), [cache], 2, 5, rows, rows, victim)
    assert err.value.code == 4 and cache.len == 2
    with pytest.raises(vs.VSError) as err:       # fewer rows than the prefix
        vs.carrier_evict_append(vs_shape(s), [cache], 3, 2, rows, rows, victim)
    assert err.value.code == 2


def test_stream_with_memory_bank_prefill_reads_the_bank():
    """Frames arrive at a bank of 4 carriers behind a 3-row prefix, two layers: every frame's
    prefill attends to [prefix | carriers held], then its carrier is pushed (evicting one once the
    bank is full).  Outputs against the oracle run over the oracle's own bank; victims, lengths and
    retained rows as the oracle has them."""
    s = QW
    M, first, n_layers, frames, T, d = 4, 3, 2, 10, 21, 64
    emb = carrier_embeddings(17, frames, d, "bf16")
    dt = torch.bfloat16
    caches, o_k, o_v = [], [], []
    for l in range(n_layers):
        hk, hv = cache_rows(40 + l, s, first, 0.5)
        k = torch.zeros((first + M, s.n_kv_heads, s.head_dim), dtype=dt, device=DEV)
        v = torch.zeros_like(k)
        k[:first].copy_(hk)
        v[:first].copy_(hv)
        caches.append(vs.Cache(k, v, first))
        ok, ov = np.zeros((first + M, s.n_kv_heads, s.head_dim)), np.zeros((first + M, s.n_kv_heads, s.head_dim))
        ok[:first], ov[:first] = to_f64(hk), to_f64(hv)
        o_k.append(ok)
        o_v.append(ov)
    bank = vs.Bank(torch.zeros((M, d), dtype=dt, device=DEV), "bf16")
    o_emb, o_n = np.zeros((M, d)), 0
    victim = torch.zeros(1, dtype=torch.int32, device=DEV)
    bws = torch.empty(vs.memory_bank_workspace_bytes(M), dtype=torch.uint8, device=DEV)
    ws = workspace(s, T, first + M, 0)
    for f in range(frames):
        rows_k = torch.empty((n_layers, s.n_kv_heads, s.head_dim), dtype=dt, device=DEV)
        rows_v = torch.empty_like(rows_k)
        o_rows = []
        for l in range(n_layers):
            q, kf, vf = frame_inputs(500 + 10 * f + l, s, T, 0.5, q_gain=2)
            out = torch.full(q.shape, float("nan"), dtype=dt, device=DEV)
            vs.frame_prefill_attn(vs_shape(s), caches[l], q.to(DEV), kf.to(DEV), vf.to(DEV), out, ws)
            L = first + o_n
            ref = oracle.frame_prefill(to_f64(q), o_k[l][:L], o_v[l][:L], to_f64(kf), to_f64(vf), scale32(s))
            check_close(out, ref, "bf16", f"frame {f} layer {l} over {o_n} carriers")
            rows_k[l].copy_(kf[T - 1])
            rows_v[l].copy_(vf[T - 1])
            o_rows.append((to_f64(kf[T - 1]), to_f64(vf[T - 1])))
        vs.memory_bank_push(bank, emb[f].to(DEV), victim, bws)
        vs.carrier_evict_append(vs_shape(s), caches, first, M, rows_k, rows_v, victim)
        got = int(victim.cpu()[0])
        e64 = to_f64(emb[f])
        if o_n == M:
            want, cos = oracle.bank_victim(o_emb, e64)
            top = np.sort(cos)[::-1]
            assert got == want or top[0] - top[1] <= 1e-6
        else:
            assert got == -1
        for l in range(n_layers):
            oracle.bank_apply(o_k[l], first, M, o_n, got, o_rows[l][0])
            oracle.bank_apply(o_v[l], first, M, o_n, got, o_rows[l][1])
        o_n = oracle.bank_apply(o_emb, 0, M, o_n, got, e64)
        assert bank.len == o_n and all(c.len == first + o_n for c in caches)
    for l in range(n_layers):
        assert np.array_equal(caches[l].k.double().cpu().numpy(), o_k[l]) and np.array_equal(caches[l].v.double().cpu().numpy(), o_v[l])


# ---------------------------------------------------------------------------- run of several frames
@pytest.mark.parametrize("F,T,L,splits", [(1, 170, 300, 0), (4, 170, 1500, 0), (8, 170, 4296, 0), (3, 21, 0, 0),
                                          (6, 40, 70, 0), (2, 170, 4296, 5), (64, 20, 500, 0)])
def test_run_of_frames_with_semantic_mask(F, T, L, splits):
    """Several frames in one call: outputs against the oracle's definition of the mask, the carriers
    appended in frame order bit for bit, and the same as feeding the frames one call at a time."""
    s = QW
    hk, hv = cache_rows(61, s, L, 0.5)
    q = draw(62, (F, T, s.n_q_heads, s.head_dim), 0.5 * 3, "bf16")
    kf = draw(63, (F, T, s.n_kv_heads, s.head_dim), 0.5, "bf16")
    vf = draw(64, (F, T, s.n_kv_heads, s.head_dim), 0.5, "bf16")
    ref = oracle.frames_prefill(to_f64(q), to_f64(hk) if L else None, to_f64(hv) if L else None, to_f64(kf), to_f64(vf),
                                scale32(s))
    dt = torch.bfloat16

    def fresh_cache():
        k = torch.zeros((L + F, s.n_kv_heads, s.head_dim), dtype=dt, device=DEV)
        v = torch.zeros_like(k)
        if L:
            k[:L].copy_(hk)
            v[:L].copy_(hv)
        return vs.Cache(k, v, L)

    vs.set_tuning(vs.TUNE_PREFILL_SPLITS, splits)
    cache = fresh_cache()
    ws = torch.empty(vs.frames_workspace_bytes(vs_shape(s), F, T, L + F), dtype=torch.uint8, device=DEV)
    vs.workspace_init(vs_shape(s), ws)
    out = torch.full(q.shape, float("nan"), dtype=dt, device=DEV)
    vs.frames_prefill_attn(vs_shape(s), cache, q.to(DEV), kf.to(DEV), vf.to(DEV), out, ws)
    torch.cuda.synchronize()
    assert cache.len == L + F
    check_close(out, ref, "bf16", f"run of {F} frames of {T} over {L} rows")
    assert same_bits(cache.k[L:], kf[:, T - 1]) and same_bits(cache.v[L:], vf[:, T - 1])
    if L:
        assert same_bits(cache.k[:L], hk) and same_bits(cache.v[:L], hv)
    # one call per frame gives the same values up to the rounding of differently split sums
    c2 = fresh_cache()
    ws1 = workspace(s, T, L + F, 0)
    for a in range(F):
        o1 = torch.full(q.shape[1:], float("nan"), dtype=dt, device=DEV)
        vs.frame_prefill_compact(vs_shape(s), c2, q[a].to(DEV), kf[a].to(DEV), vf[a].to(DEV), o1, ws1)
        torch.cuda.synchronize()
        d = (o1.float() - out[a].float()).abs().max().item()
        assert d <= 2 ** -7 * out[a].float().abs().max().item() + 1e-6, f"frame {a}: {d}"
    assert torch.equal(c2.k, cache.k) and torch.equal(c2.v, cache.v) and c2.len == cache.len


def test_prefill_random_shapes_sweep():
    """Seeded sweep over cache lengths, run lengths, head groupings, forced splits and key-group
    counts: exercises every way the key tiles can fall onto the (split, key group) lanes (fewer
    tiles than lanes, frame tiles on several lanes, a lane made of frame tiles only, ...)."""
    rng = np.random.default_rng(2024)
    groupings = [(28, 4), (8, 8), (8, 1), (12, 4), (16, 2)]
    for case in range(96):
        hq, hkv = groupings[rng.integers(len(groupings))]
        s = AttnShape(hq, hkv, 128, "bf16")
        L = int(rng.choice([0, 1, 63, 64, 65, 127, 200, 449, 512, 1000, 1733]))
        T = int(rng.choice([1, 2, 9, 19, 37, 64, 101, 170, 257]))
        splits = int(rng.choice([0, 0, 1, 2, 3, 5, 8, 13, 32]))
        kvg = int(rng.choice([0, 0, 1, 2]))
        gain = float(rng.choice([1, 1, 6]))
        vs.set_tuning(vs.TUNE_PREFILL_SPLITS, splits)
        vs.set_tuning(vs.TUNE_PREFILL_KV_GROUPS, kvg)
        hk, hv = cache_rows(700 + case, s, L, 0.5)
        q, kf, vf = frame_inputs(700 + case, s, T, 0.5, q_gain=gain)
        out, cache, row = run_prefill(s, hk, hv, L, q, kf, vf, fused=bool(case & 1))
        ref = oracle_prefill_rows(s, q, hk, hv, L, kf, vf)
        bound = oracle_prefill_rows(s, q, hk, hv.abs(), L, kf, vf.abs())
        check_close(out, ref, "bf16", f"case {case}: Hq/Hkv {hq}/{hkv} L={L} T={T} splits={splits} kv_groups={kvg} gain={gain}",
                    abs_v_out=bound)
        if case & 1:
            assert row == L and cache.len == L + 1 and same_bits(cache.k[L], kf[T - 1]) and same_bits(cache.v[L], vf[T - 1])


@pytest.mark.parametrize("kv_groups,splits", [(2, 1), (2, 2), (1, 1), (1, 3)])
def test_prefill_rows_whose_first_tile_is_masked_beside_rows_that_are_redone(kv_groups, splits):
    """A lane that starts with a tile some of its rows do not see at all, while others need the exact redo of
    that tile (peaked scores): the former must keep a usable reference for the tiles that follow."""
    s, L, T = AttnShape(12, 4, 128, "bf16"), 200, 101
    hk, hv = cache_rows(726, s, L, 0.5)
    q, kf, vf = frame_inputs(726, s, T, 0.5, q_gain=6)
    vs.set_tuning(vs.TUNE_PREFILL_KV_GROUPS, kv_groups)
    vs.set_tuning(vs.TUNE_PREFILL_SPLITS, splits)
    out, _, _ = run_prefill(s, hk, hv, L, q, kf, vf)
    ref = oracle_prefill_rows(s, q, hk, hv, L, kf, vf)
    check_close(out, ref, "bf16", f"first tile masked, kv_groups={kv_groups} splits={splits}")


@pytest.mark.parametrize("hq,hkv,L,T", [
    # units (KV heads x row tiles) that do not divide evenly over the XCDs, with keys enough to be split up to
    # what an XCD holds; one key group and two; more than 8 splits and fewer
    (28, 4, 4552, 37), (28, 4, 3000, 19), (28, 4, 1600, 37), (28, 4, 1200, 128), (12, 6, 1600, 170), (16, 2, 2500, 9),
    (24, 8, 1600, 100), (28, 4, 1100, 192), (28, 4, 1500, 330),
])
def test_prefill_plans_over_units_and_keys(hq, hkv, L, T):
    s = AttnShape(hq, hkv, 128, "bf16")
    hk, hv = cache_rows(1300 + T, s, L, 0.5)
    q, kf, vf = frame_inputs(1300 + T, s, T, 0.5, q_gain=3)
    out, cache, row = run_prefill(s, hk, hv, L, q, kf, vf, fused=True)
    ref = oracle_prefill_rows(s, q, hk, hv, L, kf, vf)
    check_close(out, ref, "bf16", f"plan Hq/Hkv {hq}/{hkv} L={L} T={T}")
    assert row == L and cache.len == L + 1 and same_bits(cache.k[L], kf[T - 1]) and same_bits(cache.v[L], vf[T - 1])


@pytest.mark.parametrize("gain", [1, 12])
@pytest.mark.parametrize("hq,hkv,L,T", [
    # key counts at the edges of blocks of 32 and of rounds of four blocks, blocks that straddle cache and frame,
    # packed rows at the edges of groups of 32, no cache, one token, row counts up to 7 rounds (the last ones taken: below)
    (28, 4, 0, 1), (28, 4, 0, 32), (28, 4, 1, 31), (28, 4, 31, 1), (28, 4, 32, 33), (28, 4, 33, 95), (8, 1, 95, 4), (8, 8, 96, 32),
    (16, 2, 127, 33), (12, 6, 128, 128), (24, 8, 200, 170), (28, 4, 264, 170), (28, 4, 342, 170), (28, 4, 511, 2), (28, 4, 700, 192),
])
def test_prefill_short_key_sequences(hq, hkv, L, T, gain):
    s = AttnShape(hq, hkv, 128, "bf16")
    hk, hv = cache_rows(1400 + L, s, L, 0.5)
    q, kf, vf = frame_inputs(1400 + L, s, T, 0.5, q_gain=gain)
    out, cache, row = run_prefill(s, hk, hv, L, q, kf, vf, fused=True)
    ref = oracle_prefill_rows(s, q, hk, hv, L, kf, vf)
    bound = oracle_prefill_rows(s, q, hk, hv.abs(), L, kf, vf.abs())
    check_close(out, ref, "bf16", f"short keys Hq/Hkv {hq}/{hkv} L={L} T={T} gain={gain}", abs_v_out=bound)
    assert row == L and cache.len == L + 1 and same_bits(cache.k[L], kf[T - 1]) and same_bits(cache.v[L], vf[T - 1])


def partial_row_tiles(ws, s):
    """How many (row tile, split) partial results a call has left in a workspace whose scratch area held 0xff before: 128 rows of
    128 fp16 numbers and of 4 fp32 ones each, none of which is ever stored as that (partial_area says where it starts)."""
    return int((partial_area(ws, s) != -1).sum()) / (128 * (64 + 4))


def partial_area(ws, s):
    ctrl = ((64 * s.n_kv_heads * 4 + 127) // 128 + 256 * s.n_kv_heads) * 128
    return ws[ctrl:ctrl + (ws.numel() - ctrl) // 4 * 4].view(torch.int32)


@pytest.mark.parametrize("hq,hkv,T,rounds", [(28, 4, 10, 5), (28, 4, 37, 6), (28, 4, 100, 7), (28, 4, 170, 8), (8, 8, 1, 5), (8, 8, 4, 5),
                                             (8, 8, 5, 6), (32, 32, 1, 6), (32, 32, 5, 7)])
@pytest.mark.parametrize("beyond", [0, 1])
def test_prefill_on_both_sides_of_the_short_kernels_range(hq, hkv, T, rounds, beyond):
    """The last key count that the kernel for few keys takes (so many rounds of 128) and the next one, which is split and leaves
    partial results in the workspace."""
    s, L = AttnShape(hq, hkv, 128, "bf16"), 128 * rounds + beyond - T
    hk, hv = cache_rows(1500 + T, s, L, 0.5)
    q, kf, vf = frame_inputs(1500 + T, s, T, 0.5, q_gain=3)
    ws = workspace(s, T, L + 1, 1)
    partial_area(ws, s).fill_(-1)
    out, cache, row = run_prefill(s, hk, hv, L, q, kf, vf, ws=ws, fused=True)
    assert (partial_row_tiles(ws, s) > 0) == bool(beyond)
    bound = oracle_prefill_rows(s, q, hk, hv.abs(), L, kf, vf.abs())
    check_close(out, oracle_prefill_rows(s, q, hk, hv, L, kf, vf), "bf16", f"{hq}/{hkv} T={T} L={L}", abs_v_out=bound)
    assert row == L and cache.len == L + 1 and same_bits(cache.k[L], kf[T - 1]) and same_bits(cache.v[L], vf[T - 1])


def check_whole_and_split(ws, s, F, T):
    """The units behind the whole rounds of every XCD, and no others, have left partial results, 2 to 8 each."""
    units = -(-T * (s.n_q_heads // s.n_kv_heads) // 128) * s.n_kv_heads * F
    per_xcd = -(-units // 8)
    split = sum(max(0, min(per_xcd, units - x * per_xcd) - per_xcd // 32 * 32) for x in range(8))
    assert split > 0 and partial_row_tiles(ws, s) in [split * n for n in range(2, 9)]


@pytest.mark.parametrize("F,T,L,hq,hkv", [
    (33, 124, 600, 8, 8), (39, 60, 900, 16, 8), (35, 117, 577, 8, 8), (9, 170, 1500, 28, 4),
    (12, 192, 600, 28, 4),                            # 66 units per XCD: two whole rounds in front
    (33, 124, 32700 - 124, 8, 8), (33, 124, 33000, 8, 8),  # 512 tiles of keys and more
])
def test_run_of_frames_with_whole_and_split_units(F, T, L, hq, hkv):
    """More units than compute units, and a last round of few: those are split, the others whole.  Against the oracle
    (some frames), the kept rows bit for bit, three times through one workspace with the same bits, whatever is said about merges, and
    close to the result where all units are split alike."""
    s = AttnShape(hq, hkv, 128, "bf16")
    hk, hv = cache_rows(65, s, L, 0.5)
    q = draw(66, (F, T, hq, 128), 0.5, "bf16")
    kf, vf = (draw(k, (F, T, hkv, 128), 0.5, "bf16") for k in (67, 68))
    ws = torch.empty(vs.frames_workspace_bytes(vs_shape(s), F, T, L + F), dtype=torch.uint8, device=DEV)
    vs.workspace_init(vs_shape(s), ws)
    partial_area(ws, s).fill_(-1)
    qd, kd, vd = q.to(DEV), kf.to(DEV), vf.to(DEV)

    def run():
        k, v = (torch.zeros((L + F, hkv, 128), dtype=torch.bfloat16, device=DEV) for _ in "kv")
        k[:L].copy_(hk)
        v[:L].copy_(hv)
        out = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device=DEV)
        vs.frames_prefill_attn(vs_shape(s), vs.Cache(k, v, L), qd, kd, vd, out, ws)
        torch.cuda.synchronize()
        assert same_bits(k[L:], kf[:, T - 1]) and same_bits(v[L:], vf[:, T - 1])
        return out

    first = run()
    check_whole_and_split(ws, s, F, T)
    tokens = [0, T // 2, T - 1] if L > 2000 else list(range(T))
    for f in (0, F // 2, F - 1):
        k_all, v_all = torch.cat([hk, kf[:f, T - 1]]), torch.cat([hv, vf[:f, T - 1]])
        check_close(first[f][tokens], oracle_prefill_rows(s, q[f], k_all, v_all, L + f, kf[f], vf[f], tokens), "bf16", f"frame {f} of {F}")
    assert all(same_bits(run(), first.cpu()) for _ in range(2))
    for merge in (1, 2):
        vs.set_tuning(vs.TUNE_PREFILL_MERGE, merge)
        assert same_bits(run(), first.cpu())
    vs.set_tuning(vs.TUNE_PREFILL_MERGE, 0)
    vs.set_tuning(vs.TUNE_PREFILL_SPLITS, 2)
    assert (run().float() - first.float()).abs().max() <= 2 ** -7 * first.float().abs().max()


def test_run_of_frames_with_whole_and_split_units_waits_for_nobody():
    """The workgroups of a split unit start when those of whole units have ended, which may be any time where the launch has part of
    the device: with waits given up at once the result is complete all the same, and nothing is reported."""
    s, F, T, L = AttnShape(8, 8, 128, "bf16"), 33, 124, 600
    hk, hv = (t.to(DEV) for t in cache_rows(65, s, L, 0.5))
    q, kf, vf = (draw(k, (F, T, 8, 128), 0.5, "bf16").to(DEV) for k in (66, 67, 68))
    ws = torch.empty(vs.frames_workspace_bytes(vs_shape(s), F, T, L + F), dtype=torch.uint8, device=DEV)
    vs.workspace_init(vs_shape(s), ws)
    outs = []
    for merge in (0, 4, 3, 0):
        vs.set_tuning(vs.TUNE_PREFILL_MERGE, merge)
        k, v = (torch.cat([t, torch.zeros_like(t[:F])]) for t in (hk, hv))
        outs.append(torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device=DEV))
        vs.frames_prefill_attn(vs_shape(s), vs.Cache(k, v, L), q, kf, vf, outs[-1], ws)
        torch.cuda.synchronize()
    assert torch.isfinite(outs[0]).all() and all(same_bits(o, outs[0].cpu()) for o in outs[1:])


def test_long_question_with_whole_and_split_units():
    """The same for one long run whose rows are all kept: 264 units of 2100 tokens."""
    s, T, L = AttnShape(16, 8, 128, "bf16"), 2100, 512
    hk, hv = cache_rows(69, s, L, 0.5)
    q, kt, vt = frame_inputs(69, s, T, 0.5)
    k, v = (torch.zeros((L + T, 8, 128), dtype=torch.bfloat16, device=DEV) for _ in "kv")
    k[:L].copy_(hk)
    v[:L].copy_(hv)
    out = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device=DEV)
    ws = workspace(s, T, L + T, 0)
    partial_area(ws, s).fill_(-1)
    vs.question_prefill_append(vs_shape(s), vs.Cache(k, v, L), q.to(DEV), kt.to(DEV), vt.to(DEV), out, ws)
    torch.cuda.synchronize()
    check_whole_and_split(ws, s, 1, T)
    assert same_bits(k[L:], kt) and same_bits(v[L:], vt) and same_bits(k[:L], hk) and same_bits(v[:L], hv)
    tokens = [0, 1, 63, 64, 1023, 1024, 2047, 2048, 2099]  # 64 tokens are a row tile; the last tile's units are split
    check_close(out[tokens], oracle_prefill_rows(s, q, hk, hv, L, kt, vt, tokens), "bf16", "long question")


def test_runs_of_frames_random_shapes_sweep():
    rng = np.random.default_rng(77)
    for case in range(24):
        hq, hkv = [(28, 4), (8, 8), (8, 1)][rng.integers(3)]
        s = AttnShape(hq, hkv, 128, "bf16")
        F = int(rng.choice([1, 2, 3, 5, 9, 17]))
        T = int(rng.choice([1, 3, 19, 40, 101]))
        L = int(rng.choice([0, 5, 64, 130, 700]))
        splits = int(rng.choice([0, 0, 2, 4, 7]))
        vs.set_tuning(vs.TUNE_PREFILL_SPLITS, splits)
        hk, hv = cache_rows(900 + case, s, L, 0.5)
        q = draw(1000 + case, (F, T, hq, 128), 1.0, "bf16")
        kf = draw(1100 + case, (F, T, hkv, 128), 0.5, "bf16")
        vf = draw(1200 + case, (F, T, hkv, 128), 0.5, "bf16")
        ref = oracle.frames_prefill(to_f64(q), to_f64(hk) if L else None, to_f64(hv) if L else None, to_f64(kf),
                                    to_f64(vf), scale32(s))
        k = torch.zeros((L + F, hkv, 128), dtype=torch.bfloat16, device=DEV)
        v = torch.zeros_like(k)
        if L:
            k[:L].copy_(hk)
            v[:L].copy_(hv)
        cache = vs.Cache(k, v, L)
        ws = torch.empty(max(vs.frames_workspace_bytes(vs_shape(s), F, T, L + F), 1 << 24), dtype=torch.uint8, device=DEV)
        vs.workspace_init(vs_shape(s), ws)
        out = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device=DEV)
        vs.frames_prefill_attn(vs_shape(s), cache, q.to(DEV), kf.to(DEV), vf.to(DEV), out, ws)
        torch.cuda.synchronize()
        bound = oracle.frames_prefill(to_f64(q), to_f64(hk) if L else None, np.abs(to_f64(hv)) if L else None, to_f64(kf),
                                      np.abs(to_f64(vf)), scale32(s))
        check_close(out, ref, "bf16", f"case {case}: Hq/Hkv {hq}/{hkv} F={F} T={T} L={L} splits={splits}", abs_v_out=bound)
        assert cache.len == L + F and same_bits(cache.k[L:], kf[:, T - 1]) and same_bits(cache.v[L:], vf[:, T - 1])


def test_package_used_before_torch_is_imported():
    """A fresh process that touches the library before it imports torch (here: a tuning call)
    must still find the device afterwards: library and torch share one HIP runtime, torch's,
    whichever of the two the program names first."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    code = (
        "import sys; sys.path.insert(0, %r)\n"
        "import paper_2503_09387_amd as vs\n"
        "vs.set_tuning(vs.TUNE_PREFILL_SPLITS, 0)\n"
        "import torch\n"
        "sh = vs.Shape.make(28, 4, 128, 'bf16', 0.0883883)\n"
        "ws = vs.make_workspace(sh, 8, 64, 2, 'cuda:0')\n"
        "e = torch.ones((4, 64), dtype=torch.float32, device='cuda:0'); c = torch.empty(64, device='cuda:0')\n"
        "vs.carrier_mean_pool(e, c, 'f32'); torch.cuda.synchronize()\n"
        "assert bool((c == 1).all())\n"
        "print('ok')\n" % root)
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr
