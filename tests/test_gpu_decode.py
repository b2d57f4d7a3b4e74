"""GPU parity: baklava_decode_attn against the fp64 oracle (Eq. 1 / Eq. 7), element by element."""
import numpy as np
import pytest
import torch

from oracle import baklava_oracle as O
from paper_2502_13176_amd import binding as B
from paper_2502_13176_amd import synth

pytestmark = pytest.mark.gpu


def _h():
    import gpu_harness
    return gpu_harness


def _kernels_for(w):
    ks = []
    if w.G <= 8:
        ks.append(B.KERNEL_VALU)
    if w.dtype == "bf16" and w.D == 128:
        ks.append(B.KERNEL_MFMA)
    return ks


def test_tiny_workload_full_cache():
    H = _h()
    w = synth.WORKLOADS["tiny"]
    rng = np.random.Generator(np.random.PCG64(w.seed))
    arena = H.make_arena(w)
    st = H.fill_from_host(arena, w, [w.ctx] * arena.n_caches, rng, scores="uniform")
    q, q64 = H.make_q(w, rng, w.L)
    out = H.gpu_decode(arena, w, q)
    err = H.check_decode_against_oracle(arena, w, st, q64, out)
    print(f"tiny: max-abs error {err:.3e}", flush=True)
    arena.close()


@pytest.mark.parametrize("kernel", [B.KERNEL_VALU, B.KERNEL_MFMA])
@pytest.mark.parametrize("chunk", [256, 1024, 4096, 16384])
def test_llama_single_layer_at_full_size(kernel, chunk):
    """LLaMA-3-8B-shaped layer, context 8192, budgets summing to half of 8*8192, caches at budget."""
    H = _h()
    w = synth.WORKLOADS["llama1"]
    rng = np.random.Generator(np.random.PCG64(w.seed))
    budgets = synth.budgets_for(w, B.alloc_proportional)
    arena = H.make_arena(w, budgets)
    arena.set_option(B.OPT_KERNEL, kernel)
    H.set_chunk(arena, chunk)
    lens = [budgets[c % w.Hkv] for c in range(arena.n_caches)]
    st = H.fill_from_host(arena, w, lens, rng)
    q, q64 = H.make_q(w, rng, w.L)
    out = H.gpu_decode(arena, w, q)
    err = H.check_decode_against_oracle(arena, w, st, q64, out)
    print(f"llama1 kernel={kernel} chunk={chunk}: max-abs error {err:.3e}", flush=True)
    arena.close()


RAGGED_LENS = [1, 2, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 257, 1000, 1023, 1025, 2500]


@pytest.mark.parametrize("dtype,D,Hq,Hkv", [
    ("bf16", 128, 8, 2), ("bf16", 128, 7, 1), ("bf16", 128, 2, 2), ("bf16", 128, 16, 2), ("bf16", 128, 16, 1),
    ("bf16", 64, 8, 2), ("f32", 64, 4, 2), ("f32", 128, 7, 1), ("f32", 128, 2, 1),
])
def test_ragged_lengths_all_shapes(dtype, D, Hq, Hkv):
    """Lengths around every tile boundary of both kernels, several layers and sequences, with a
    layer sub-range launch as well as the whole stack."""
    H = _h()
    w = synth.shrink(synth.WORKLOADS["llama1"], name="ragged", L=2, Hq=Hq, Hkv=Hkv, D=D, batch=2, dtype=dtype,
                     seed=77, sink=1, recent=1, slack=0)
    rng = np.random.Generator(np.random.PCG64(w.seed))
    n_caches = w.L * w.batch * w.Hkv
    budgets = [4096] * (w.L * w.Hkv)
    lens = [RAGGED_LENS[(3 * c + 1) % len(RAGGED_LENS)] for c in range(n_caches)]
    arena = H.make_arena(w, budgets)
    st = H.fill_from_host(arena, w, lens, rng)
    q, q64 = H.make_q(w, rng, w.L)
    for kernel in _kernels_for(w):
        arena.set_option(B.OPT_KERNEL, kernel)
        for chunk in (256, 512, 4096):
            H.set_chunk(arena, chunk)
            out = H.gpu_decode(arena, w, q)
            H.check_decode_against_oracle(arena, w, st, q64, out)
        # second layer alone
        out1 = H.gpu_decode(arena, w, q[1:2], layer_begin=1, layer_count=1)
        H.check_decode_against_oracle(arena, w, st, q64[1:2], out1, caches=range(n_caches // 2, n_caches),
                                          layer_begin=1)
        # item targets below the item count at 256-row runs: runs grow (per layer / over the model)
        # until few items are left, down to one item per cache
        H.set_chunk(arena, 256)
        for target in (1, 7, 23):
            arena.set_option(B.OPT_TARGET_ITEMS, target)
            arena.set_option(B.OPT_TARGET_ITEMS_WHOLE, target)
            out = H.gpu_decode(arena, w, q)
            H.check_decode_against_oracle(arena, w, st, q64, out)
            out1 = H.gpu_decode(arena, w, q[1:2], layer_begin=1, layer_count=1)
            H.check_decode_against_oracle(arena, w, st, q64[1:2], out1, caches=range(n_caches // 2, n_caches),
                                          layer_begin=1)
        arena.set_option(B.OPT_TARGET_ITEMS, 0)
        arena.set_option(B.OPT_TARGET_ITEMS_WHOLE, 0)
    arena.close()


@pytest.mark.parametrize("kernel", [B.KERNEL_VALU, B.KERNEL_MFMA])
def test_result_does_not_depend_on_split_factor(kernel):
    H = _h()
    w = synth.shrink(synth.WORKLOADS["llama1"], name="split", Hq=8, Hkv=2, seed=5, slack=0)
    rng = np.random.Generator(np.random.PCG64(w.seed))
    budgets = [7000, 3333]
    arena = H.make_arena(w, budgets)
    arena.set_option(B.OPT_KERNEL, kernel)
    st = H.fill_from_host(arena, w, budgets, rng)
    q, q64 = H.make_q(w, rng, w.L)
    outs = []
    for chunk in (8192, 3584, 1024, 256):      # 1, 2, 7 and 28 splits of the long cache
        H.set_chunk(arena, chunk)
        outs.append(H.gpu_decode(arena, w, q))
        H.check_decode_against_oracle(arena, w, st, q64, outs[-1])
    for o in outs[1:]:
        assert np.max(np.abs(o - outs[0])) <= 1e-5
    arena.close()


@pytest.mark.parametrize("kernel", [B.KERNEL_VALU, B.KERNEL_MFMA])
def test_peaked_and_large_logits(kernel):
    """A few keys scaled up so single rows dominate the softmax, and logits of magnitude ~80:
    the running-max rescaling must stay finite and accurate."""
    H = _h()
    w = synth.shrink(synth.WORKLOADS["llama1"], name="peaked", Hq=8, Hkv=2, seed=9, slack=0)
    rng = np.random.Generator(np.random.PCG64(w.seed))
    budgets = [3000, 1500]
    arena = H.make_arena(w, budgets)
    arena.set_option(B.OPT_KERNEL, kernel)
    st = H.fill_from_host(arena, w, budgets, rng, peaked=True)
    q, q64 = H.make_q(w, rng, w.L)
    H.check_decode_against_oracle(arena, w, st, q64, H.gpu_decode(arena, w, q))
    st = H.fill_from_host(arena, w, budgets, rng, scale=7.0)
    q, q64 = H.make_q(w, rng, w.L, scale=7.0)
    H.check_decode_against_oracle(arena, w, st, q64, H.gpu_decode(arena, w, q))
    # ascending logits: the running maximum changes in every slab
    n = 2048
    K = np.zeros((n, w.D), dtype=np.float32)
    K[:, 0] = np.linspace(-40, 40, n)
    Vv = rng.standard_normal((n, w.D)).astype(np.float32)
    arena2 = H.make_arena(synth.shrink(w, Hq=4, Hkv=1), [n])
    arena2.set_option(B.OPT_KERNEL, kernel)
    w2 = synth.shrink(w, Hq=4, Hkv=1)
    st2 = H.HostState(1)
    st2.K[0], st2.V[0] = synth.f32_to_bf16_bits(K), synth.f32_to_bf16_bits(Vv)
    arena2.k[:n].copy_(H.to_device_storage(st2.K[0], "bf16", arena2.device))
    arena2.v[:n].copy_(H.to_device_storage(st2.V[0], "bf16", arena2.device))
    arena2.set_lengths([n])
    qq = np.zeros((1, 1, 4, w.D), dtype=np.float32)
    qq[..., 0] = [11.0, -11.0, 3.0, 0.5]
    qs = synth.f32_to_bf16_bits(qq)
    H.check_decode_against_oracle(arena2, w2, st2, synth.storage_to_f64(qs, "bf16"), H.gpu_decode(arena2, w2, qs))
    arena.close()
    arena2.close()


def test_error_paths():
    H = _h()
    w = synth.shrink(synth.WORKLOADS["llama1"], name="err", Hq=4, Hkv=2, seed=3, slack=2)
    arena = H.make_arena(w, [300, 200])
    q = torch.zeros((1, 1, 4, 128), dtype=torch.bfloat16, device=arena.device)
    out = torch.zeros((1, 1, 4, 128), dtype=torch.float32, device=arena.device)
    with pytest.raises(B.BaklavaError) as e:           # empty caches
        arena.decode_attn(0, 1, q, out)
    assert e.value.status == B.ESTATE
    with pytest.raises(B.BaklavaError) as e:
        arena.decode_attn(0, 2, q, out)
    assert e.value.status == B.EINVAL
    with pytest.raises(B.BaklavaError) as e:
        arena.set_lengths([303, 1])
    assert e.value.status == B.ECAPACITY
    arena.set_lengths([302, 1])
    kn = torch.zeros((1, 2, 128), dtype=torch.bfloat16, device=arena.device)
    with pytest.raises(B.BaklavaError) as e:           # cache 0 is full
        arena.append(0, 1, kn, kn, 5)
    assert e.value.status == B.ECAPACITY
    assert arena.lengths().tolist() == [302, 1]
    with pytest.raises(B.BaklavaError) as e:
        H.set_chunk(arena, 100)
    assert e.value.status == B.EINVAL
    arena.reset()
    assert arena.lengths().tolist() == [0, 0]
    torch.cuda.synchronize()
    assert arena.len.cpu().tolist() == [0, 0]
    arena.close()


@pytest.mark.parametrize("kernel", [B.KERNEL_VALU, B.KERNEL_MFMA])
def test_fused_append_at_item_boundaries(kernel):
    """baklava_append_decode_attn with the new row landing first / last in a work item, in a new
    work item of its own, and in an empty cache; the result must equal append followed by
    attention, and the oracle."""
    H = _h()
    w = synth.shrink(synth.WORKLOADS["llama1"], name="fusedb", L=1, Hq=8, Hkv=2, batch=4, seed=41, slack=600)
    rng = np.random.Generator(np.random.PCG64(w.seed))
    budgets = [500, 300]
    arena = H.make_arena(w, budgets)
    arena.set_option(B.OPT_KERNEL, kernel)
    H.set_chunk(arena, 256)
    lens = [0, 255, 256, 257, 511, 512, 513, 767]
    st = H.fill_from_host(arena, w, lens, rng)
    for step in range(3):
        q, q64 = H.make_q(w, rng, 1)
        knew = synth.payload(rng, (1, w.batch, w.Hkv, w.D), w.dtype)
        vnew = synth.payload(rng, (1, w.batch, w.Hkv, w.D), w.dtype)
        outd = torch.full((1, w.batch, w.Hq, w.D), float("nan"), dtype=torch.float32, device=arena.device)
        arena.append_decode_attn(0, 1, H.to_device_storage(knew, w.dtype, arena.device),
                                 H.to_device_storage(vnew, w.dtype, arena.device), 900 + step,
                                 H.to_device_storage(q, w.dtype, arena.device), outd)
        torch.cuda.synchronize()
        out = outd.cpu().numpy().astype(np.float64)
        post = H.download(arena, w)
        assert arena.lengths().tolist() == [n + step + 1 for n in lens]
        assert arena.len.cpu().tolist() == arena.lengths().tolist()
        for c in range(arena.n_caches):
            b, h = divmod(c, w.Hkv)
            assert np.array_equal(post.K[c][:-1], st.K[c]) and np.array_equal(post.V[c][:-1], st.V[c])
            assert np.array_equal(post.K[c][-1], knew[0, b, h]) and np.array_equal(post.V[c][-1], vnew[0, b, h])
            assert post.pos[c][-1] == 900 + step and post.score[c][-1] == 0.0
        H.check_decode_against_oracle(arena, w, post, q64, out)
        st = post
    arena.close()


def test_stream_probe_modes():
    """The measurement aid: the copy really copies, the read-only sweeps leave both buffers alone,
    unknown modes and odd sizes are refused."""
    dev = torch.device("cuda:0")
    n = (1 << 22) + 4096 + 16                      # not a multiple of the probe's block size
    src = torch.randint(0, 255, (n,), dtype=torch.uint8, device=dev)
    dst = torch.zeros((n,), dtype=torch.uint8, device=dev)
    B.stream_probe(dst, src, n, 0)
    torch.cuda.synchronize()
    assert torch.equal(dst, src)
    keep = dst.clone()
    for mode in (1, 2, 3):
        B.stream_probe(dst, src, n, mode)
    torch.cuda.synchronize()
    assert torch.equal(dst, keep)
    for bad in (lambda: B.stream_probe(dst, src, n, 4), lambda: B.stream_probe(dst, src, n - 8, 0),
                lambda: B.stream_probe(dst, src, 0, 1)):
        with pytest.raises(B.BaklavaError) as e:
            bad()
        assert e.value.status == B.EINVAL


@pytest.mark.parametrize("kernel", [B.KERNEL_VALU, B.KERNEL_MFMA])
@pytest.mark.parametrize("mode", [1, 2])
def test_kernel_timing_record(kernel, mode):
    """The measurement aid behind the roofline figure: both ways of timing the attention kernel count
    every launch, report a positive time that a host clock around the same calls bounds from above,
    leave the results alone, and the record is empty again after it has been read."""
    import time
    H = _h()
    w = synth.shrink(synth.WORKLOADS["llama1"], name="timed", L=3, Hq=8, Hkv=2, batch=2, seed=43, slack=64)
    rng = np.random.Generator(np.random.PCG64(w.seed))
    arena = H.make_arena(w, [700, 300] * w.L, track=True)       # the tracked instance of the kernel is timed too
    lens = [int(arena.cap_host[c]) - 1 - 37 * (c % 3) for c in range(arena.n_caches)]
    st = H.fill_from_host(arena, w, lens, rng, scores="uniform")
    arena.set_option(B.OPT_KERNEL, kernel)
    H.set_chunk(arena, 256)
    q, q64 = H.make_q(w, rng, w.L)
    ref = H.gpu_decode(arena, w, q)
    arena.set_option(B.OPT_TIME_KERNEL, mode)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    outs = [H.gpu_decode(arena, w, q) for _ in range(3)]           # one launch over all layers each
    qd = H.to_device_storage(q, w.dtype, arena.device)
    out_l = torch.empty((1, w.batch, w.Hq, w.D), dtype=torch.float32, device=arena.device)
    for l in range(w.L):
        arena.decode_attn(l, 1, qd[l:l + 1], out_l)
    torch.cuda.synchronize()
    wall_ms = (time.perf_counter() - t0) * 1e3
    with pytest.raises(B.BaklavaError) as e:                        # a record in one mode is read before the mode changes
        arena.set_option(B.OPT_TIME_KERNEL, 3 - mode)
    assert e.value.status == B.ESTATE
    ms, launches = arena.profile_read()
    assert launches == 3 + w.L and 0.0 < ms <= wall_ms
    assert arena.profile_read() == (0.0, 0)
    arena.set_option(B.OPT_TIME_KERNEL, 0)
    for o in outs:
        assert np.array_equal(o, ref)
    H.check_decode_against_oracle(arena, w, st, q64, ref)
    with pytest.raises(B.BaklavaError):
        arena.set_option(B.OPT_TIME_KERNEL, 3)
    arena.close()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("G", [5, 8])
@pytest.mark.parametrize("batch", [1, 30])
def test_fp32_matrix_kernel_slabs(D, G, batch):
    """fp32 rows for five query heads and more: lengths around a wavefront's slab (16 or 32 rows), a workgroup's (128 or
    256, half that where several workgroups share a compute unit) and a work item, outputs and tracked scores against the
    oracle.  Bound: a logit is a sum of D products over at most 2 + log2(D) roundings of at most 2^-24 of the sum of their
    sizes, so with |q|.|k| <= S (in log2 units) a weight is off by 2^-24 (2 + log2 D) S ln 2 and an output by that times
    the largest |v|; the sums over n rows add 2^-24 (n / 8 + 8) likewise, here less than as much again."""
    H = _h()
    w = synth.shrink(synth.WORKLOADS["tiny"], name="slabs", L=1, Hq=5 * G, Hkv=5, D=D, batch=batch, ctx=2048, seed=47 + G,
                     slack=0)
    rng = np.random.Generator(np.random.PCG64(w.seed))
    arena = H.make_arena(w, [40, 130, 257, 520, 1100], track=True)
    edges = [1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1099, 1100]
    lens = [([e for e in edges if e <= arena.cap_host[c]] * 30)[-1 - c // 5] for c in range(arena.n_caches)]
    st = H.fill_from_host(arena, w, lens, rng)
    q, q64 = H.make_q(w, rng, 1)
    out = H.gpu_decode(arena, w, q)
    post = H.download(arena, w)
    for c in range(arena.n_caches):
        _, b, hs = H.q_rows_of_cache(w, c)
        k, v = st.K[c].astype(np.float64), st.V[c].astype(np.float64)
        ref, p = O.decode_attn(q64[0, b, hs], k, v)
        size = float(np.max(np.abs(q64[0, b, hs]) @ np.abs(k).T)) / np.sqrt(D)
        tol = 2.0 ** -24 * 2 * (2 + np.log2(D)) * size * max(1.0, float(np.max(np.abs(v))))
        assert np.max(np.abs(out[0, b, hs] - ref)) <= tol, (c, lens[c])
        assert np.max(np.abs(post.score[c] - p.sum(axis=0))) <= G * tol, (c, lens[c])
    # the vector kernel on the same call
    arena.set_option(B.OPT_KERNEL, B.KERNEL_VALU)
    assert np.max(np.abs(H.gpu_decode(arena, w, q) - out)) <= 1e-5
    arena.close()


F32_MATRIX = [("f32", D, G, B.KERNEL_AUTO) for D in (64, 128) for G in (5, 8)]


@pytest.mark.parametrize("dtype,D,G,kernel", [(*shape, B.KERNEL_VALU) for shape in (
    ("f32", 64, 1), ("f32", 64, 4), ("f32", 128, 3), ("f32", 128, 8), ("bf16", 64, 1), ("bf16", 64, 5), ("bf16", 64, 8),
    ("bf16", 128, 1))] + F32_MATRIX)
def test_kernel_tiles_and_rising_logits(dtype, D, G, kernel):
    """The vector kernel's workgroups of 16 and of 8 wavefronts and the fp32 matrix kernel: lengths around a
    wavefront's and a workgroup's tile, with logits that climb along the cache by little and by 40 a row, so that
    every tile raises the maximum, and the scores that the vector kernel's second pass or the kept logits add."""
    H = _h()
    lens = [1, 15, 17, 32, 33, 127, 128, 129, 255, 257, 511, 512, 513, 1025]
    w = synth.shrink(synth.WORKLOADS["tiny"], name="valu", L=1, Hq=G * len(lens), Hkv=len(lens), D=D, batch=1,
                     dtype=dtype, seed=91, sink=1, recent=1, slack=0)
    rng = np.random.Generator(np.random.PCG64(w.seed + G))
    arena = H.make_arena(w, [2048] * len(lens), track=True)
    arena.set_option(B.OPT_KERNEL, kernel)
    q, q64 = H.make_q(w, rng, w.L)
    for step in (0.0, 0.02, 40.0):                 # natural units of the logit per row
        st = H.fill_from_host(arena, w, lens, rng)
        for c, n in enumerate(lens):
            # a component along the group's first query row that grows with the row
            u = q64[0, 0, c * G] / np.dot(q64[0, 0, c * G], q64[0, 0, c * G]) * np.sqrt(D)
            x = synth.storage_to_f64(st.K[c], dtype) + (step * np.minimum(np.arange(n), 30 if step > 1 else n))[:, None] * u
            st.K[c] = x.astype(np.float32) if dtype == "f32" else synth.f32_to_bf16_bits(x.astype(np.float32))
            o = int(arena.off_host[c])
            arena.k[o:o + n].copy_(H.to_device_storage(st.K[c], dtype, arena.device))
        # An fp32 logit of s (log2 units) carries an error of a few s * 2^-24, and so, relatively, do the weights:
        # about 1e-4 at the ~1700 of the steepest climb, 1e-6 to 3e-6 at the ~10 and ~40 of the others.
        tol, score_tol = (H.ATTN_TOL, 2e-3) if step > 1 else (4e-6, 4e-6)
        H.check_decode_against_oracle(arena, w, st, q64, H.gpu_decode(arena, w, q), tol=tol)
        post = H.download(arena, w)
        for c, n in enumerate(lens):
            l, b, hs = H.q_rows_of_cache(w, c)
            _, p = O.decode_attn(q64[l, b, hs], synth.storage_to_f64(st.K[c], dtype), synth.storage_to_f64(st.V[c], dtype))
            assert np.max(np.abs(post.score[c] - p.sum(0))) <= score_tol, (step, n)
            assert abs(post.score[c].astype(np.float64).sum() - G) <= G * score_tol, (step, n)
    arena.close()


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f32", 128), ("bf16", 64)])
@pytest.mark.parametrize("G", [1, 3, 8])
def test_scores_from_the_logits_of_a_call(dtype, D, G):
    """Tracked calls that leave no record keep their logits in LDS until a work item ends: work items longer than
    that area holds, launches of one and of several workgroups per compute unit, ragged ends, caches with one work
    item and with several.  The scores of two calls against the oracle's weights."""
    H = _h()
    ring = [1, 33, 255, 511, 513, 1281, 2560, 2561, 6000]
    many = [1 + (37 * i) % 700 for i in range(300)]
    for lens, chunk in ((ring, 8192), (ring, 256), (many, 256)):
        w = synth.shrink(synth.WORKLOADS["tiny"], name="logits", L=1, Hq=G * len(lens), Hkv=len(lens), D=D, batch=1,
                         dtype=dtype, seed=97, sink=1, recent=1, slack=0)
        rng = np.random.Generator(np.random.PCG64(w.seed + G))
        arena = H.make_arena(w, [max(8, n) for n in lens], track=True)
        H.set_chunk(arena, chunk)
        st = H.fill_from_host(arena, w, lens, rng)
        want = [np.zeros(n) for n in lens]
        for _ in range(2):
            q, q64 = H.make_q(w, rng, w.L)
            H.gpu_decode(arena, w, q)
            for c in range(0, len(lens), 1 if lens is ring else 7):
                l, b, hs = H.q_rows_of_cache(w, c)
                _, p = O.decode_attn(q64[l, b, hs], synth.storage_to_f64(st.K[c], dtype), synth.storage_to_f64(st.V[c], dtype))
                want[c] += p.sum(0)
        post = H.download(arena, w)
        for c in range(0, len(lens), 1 if lens is ring else 7):
            # 2 G weights of at most 1, each from a logit of at most about 16 with an error of a few units of 2^-24
            assert np.max(np.abs(post.score[c] - want[c])) <= 2 * G * 2.0 ** -19, (lens[c], chunk)
        for c in range(len(lens)):
            assert abs(post.score[c].astype(np.float64).sum() - 2 * G) <= 2 * G * 2.0 ** -17, (lens[c], chunk)
        arena.close()


@pytest.mark.parametrize("splits", [[2, 3, 8, 9, 15, 16], [2, 4, 5, 6, 7, 8], [1, 2, 17, 31, 63, 64, 65, 128, 129, 255, 256, 257, 300]])
@pytest.mark.parametrize("dtype,D,track", [("bf16", 128, False), ("bf16", 128, True), ("bf16", 64, False), ("f32", 64, True)])
def test_merge_of_many_work_items(splits, dtype, D, track):
    """Caches of up to 300 work items, around the numbers of splits that a thread group, a wavefront's lanes and its
    registers hold, merged by 256 and by 1024 threads: outputs (and scores) against the oracle."""
    H = _h()
    G = 3
    lens = [256 * k - 5 for k in splits]
    w = synth.shrink(synth.WORKLOADS["tiny"], name="merge", L=1, Hq=G * len(lens), Hkv=len(lens), D=D, batch=1, dtype=dtype,
                     seed=98, sink=1, recent=1, slack=0)
    rng = np.random.Generator(np.random.PCG64(w.seed + len(splits)))
    arena = H.make_arena(w, lens, track=track)
    for target in (B.OPT_TARGET_ITEMS, B.OPT_TARGET_ITEMS_WHOLE):
        arena.set_option(target, 0)                # runs of exactly 256 rows
    H.set_chunk(arena, 512)
    H.set_chunk(arena, 256)
    st = H.fill_from_host(arena, w, lens, rng, peaked=True)
    q, q64 = H.make_q(w, rng, w.L)
    # two bf16 terms per weight leave up to 2^-16 of a value of about 4, fp32 weights a few units of 2^-24 of the logits
    H.check_decode_against_oracle(arena, w, st, q64, H.gpu_decode(arena, w, q), tol=1e-4 if D == 128 else 64 * 2.0 ** -22)
    if track:
        post = H.download(arena, w)
        for c in range(arena.n_caches):
            l, b, hs = H.q_rows_of_cache(w, c)
            _, p = O.decode_attn(q64[l, b, hs], synth.storage_to_f64(st.K[c], dtype), synth.storage_to_f64(st.V[c], dtype))
            assert np.max(np.abs(post.score[c] - p.sum(0))) <= G * 2.0 ** -16
    arena.close()


def _two_term_attention(q, K, V):
    """Attention in 64 bits but for the weights, which are cut to two bf16 terms (high part and residual)."""
    s = (q @ K.T) * (np.log2(np.e) / np.sqrt(K.shape[1]))
    p = np.exp2(s - s.max(1, keepdims=True)).astype(np.float32)
    hi = (p.view(np.uint32) & np.uint32(0xFFFF0000)).view(np.float32)
    cut = hi.astype(np.float64) + synth.storage_to_f64(synth.f32_to_bf16_bits(p - hi), "bf16")
    return (cut @ V) / p.astype(np.float64).sum(1, keepdims=True)


@pytest.mark.parametrize("Hq,Hkv", [(2, 2), (6, 2), (7, 1), (16, 2)])
def test_matrix_kernel_with_half_size_rows(Hq, Hkv):
    """bf16 rows of 64 elements on the matrix cores (what automatic choice takes): lengths around the
    slabs and workgroup strides of its eight wavefronts, several schedules, against the oracle and the vector
    kernel, element by element to 256 ulps of 1, and over all outputs to the error of fp32 weights: three bf16
    terms per weight are exact, and the bound lies below what two terms leave on the same inputs."""
    H = _h()
    lens = [1, 2, 31, 32, 33, 63, 65, 255, 256, 257, 511, 513, 1000, 2500]
    w = synth.shrink(synth.WORKLOADS["llama1"], name="half", L=2, Hq=Hq, Hkv=Hkv, D=64, batch=7, dtype="bf16",
                     seed=92 + Hq, sink=1, recent=1, slack=0)
    rng = np.random.Generator(np.random.PCG64(w.seed))
    n_caches = w.L * w.batch * w.Hkv
    arena = H.make_arena(w, [4096] * (w.L * w.Hkv))
    st = H.fill_from_host(arena, w, [lens[(5 * c + 3) % len(lens)] for c in range(n_caches)], rng, peaked=True)
    q, q64 = H.make_q(w, rng, w.L)
    ref, two = np.zeros((2, *q64.shape))
    for c in range(n_caches):
        l, b, hs = H.q_rows_of_cache(w, c)
        K, V = synth.storage_to_f64(st.K[c], "bf16"), synth.storage_to_f64(st.V[c], "bf16")
        ref[l, b, hs], two[l, b, hs] = O.decode_attn(q64[l, b, hs], K, V)[0], _two_term_attention(q64[l, b, hs], K, V)
    rel = lambda x: np.linalg.norm(x - ref) / np.linalg.norm(ref)
    # fp32 logits of about 10 to 40 in log2 units and fp32 sums leave 1e-7 to 3e-7, two terms 9e-7 and more
    bound = 4e-7
    assert rel(two) > 2 * bound
    arena.set_option(B.OPT_KERNEL, B.KERNEL_VALU)
    vector = H.gpu_decode(arena, w, q)
    assert rel(vector) <= bound
    arena.set_option(B.OPT_KERNEL, B.KERNEL_AUTO)
    for chunk in (256, 512, 4096):
        H.set_chunk(arena, chunk)
        out = H.gpu_decode(arena, w, q)
        H.check_decode_against_oracle(arena, w, st, q64, out, tol=64 * 2.0 ** -24 * 4)
        assert np.max(np.abs(out - vector)) <= 64 * 2.0 ** -24 * 4
        assert rel(out) <= bound
        out1 = H.gpu_decode(arena, w, q[1:2], layer_begin=1, layer_count=1)
        H.check_decode_against_oracle(arena, w, st, q64[1:2], out1, caches=range(n_caches // 2, n_caches), layer_begin=1,
                                      tol=64 * 2.0 ** -24 * 4)
    with pytest.raises(B.BaklavaError):          # forcing it is still for rows of 128 elements only
        arena.set_option(B.OPT_KERNEL, B.KERNEL_MFMA)
    arena.close()


@pytest.mark.parametrize("dtype,D,G,kernel", [("bf16", 64, 4, B.KERNEL_AUTO), ("bf16", 64, 4, B.KERNEL_VALU),
                                              ("bf16", 128, 4, B.KERNEL_MFMA), ("bf16", 128, 4, B.KERNEL_VALU),
                                              ("f32", 64, 8, B.KERNEL_VALU), ("f32", 128, 3, B.KERNEL_AUTO)] + F32_MATRIX)
def test_rows_whose_logits_are_minus_infinity(dtype, D, G, kernel):
    """Keys of the type's lowest value (a mask) give logits of -inf: such rows carry no weight, wherever they
    fill a wavefront's first rows, a work item's, or all but one row of a cache."""
    H = _h()
    lens = [40, 300, 700, 1300]
    masked = [39, 64, 512, 1299]                   # rows in front
    w = synth.shrink(synth.WORKLOADS["llama1"], name="masked", L=1, Hq=4 * G, Hkv=4, D=D, batch=1, dtype=dtype, seed=94, sink=1,
                     recent=1, slack=0)
    rng = np.random.Generator(np.random.PCG64(w.seed))
    arena = H.make_arena(w, [2048] * 4)
    arena.set_option(B.OPT_KERNEL, kernel)
    st = H.fill_from_host(arena, w, lens, rng)
    for c, n in enumerate(masked):
        st.K[c][:n] = 0xFF7F if dtype == "bf16" else np.finfo(np.float32).min   # -3.4e38, times queries above zero
        o = int(arena.off_host[c])
        arena.k[o:o + lens[c]].copy_(H.to_device_storage(st.K[c], w.dtype, arena.device))
    q, q64 = H.make_q(w, rng, w.L)
    q, q64 = q & 0x7FFF if dtype == "bf16" else np.abs(q), np.abs(q64)
    for chunk in (256, 512, 2048):
        H.set_chunk(arena, chunk)
        H.check_decode_against_oracle(arena, w, st, q64, H.gpu_decode(arena, w, q))
    arena.close()


@pytest.mark.parametrize("dtype,D,G,kernel", [(*shape, B.KERNEL_VALU) for shape in (
    ("f32", 64, 1), ("f32", 128, 4), ("f32", 64, 8), ("bf16", 64, 2), ("bf16", 128, 8))] + F32_MATRIX)
def test_values_near_the_ends_of_the_range(dtype, D, G, kernel):
    """The vector kernel and the fp32 matrix kernel on values whose plain sum over the rows just fits fp32 and on values close to the
    smallest normal number, with logits that rise along the cache by less than 8 in log2 units: weights above
    1 would overflow the one, weights far below 1 would lose the other."""
    H = _h()
    n = 1025
    w = synth.shrink(synth.WORKLOADS["tiny"], name="range", L=1, Hq=G, Hkv=1, D=D, batch=1, dtype=dtype, seed=95, sink=1,
                     recent=1, slack=0)
    rng = np.random.Generator(np.random.PCG64(w.seed + G))
    arena = H.make_arena(w, [n])
    arena.set_option(B.OPT_KERNEL, kernel)
    H.set_chunk(arena, 2048)                       # one work item
    st = H.fill_from_host(arena, w, [n], rng)
    q = np.zeros((1, 1, G, D), dtype=np.float32)
    q[..., 0] = np.sqrt(D)
    K = np.zeros((n, D), dtype=np.float32)
    K[256:, 0] = 5.375                             # 7.75 in log2 units
    u = 1 + rng.random((n, D), dtype=np.float32)
    store = (lambda x: x) if dtype == "f32" else synth.f32_to_bf16_bits
    arena.k[:n].copy_(H.to_device_storage(store(K), dtype, arena.device))
    for scale in (1e35, 2.0 ** -125):
        V = store((u * np.float32(scale)).astype(np.float32))
        arena.v[:n].copy_(H.to_device_storage(V, dtype, arena.device))
        out = H.gpu_decode(arena, w, store(q))[0, 0]
        ref, _ = O.decode_attn(synth.storage_to_f64(store(q), dtype)[0, 0], K.astype(np.float64), synth.storage_to_f64(V, dtype))
        # 2^-125 and weights of 1 and 2^-7.75: a product's rounding at 2^-149 is at most 2^-17 of the smaller
        assert np.max(np.abs(out / ref - 1)) <= 2e-5, scale
    arena.close()


@pytest.mark.parametrize("dtype,D,G,kernel", [("bf16", 64, 4, B.KERNEL_AUTO), ("bf16", 64, 4, B.KERNEL_VALU),
                                              ("f32", 128, 8, B.KERNEL_VALU)] + F32_MATRIX)
def test_infinite_values(dtype, D, G, kernel):
    """bf16 rows of 64 elements and fp32 rows: an infinite element of V makes that element of the outputs infinite, also in
    the row with the largest weight (1, which needs one bf16 term only), and leaves the others alone.  On the fp32 matrix
    kernel in the cache's last row too, which stands in for the rows past the end."""
    H = _h()
    n = 700
    w = synth.shrink(synth.WORKLOADS["llama1"], name="inf", L=1, Hq=G, Hkv=1, D=D, batch=1, dtype=dtype, seed=96, sink=1,
                     recent=1, slack=0)
    rng = np.random.Generator(np.random.PCG64(w.seed))
    arena = H.make_arena(w, [n])
    arena.set_option(B.OPT_KERNEL, kernel)
    st = H.fill_from_host(arena, w, [n], rng)
    q, q64 = H.make_q(w, rng, w.L)
    K = synth.storage_to_f64(st.K[0], dtype)
    _, p = O.decode_attn(q64[0, 0], K, synth.storage_to_f64(st.V[0], dtype))
    inf, minus_inf = (0x7F80, 0xFF80) if dtype == "bf16" else (np.inf, -np.inf)
    for g in range(G):
        st.V[0][np.argmax(p[g]), g] = inf
        st.V[0][np.argsort(p[g])[n // 2], 8 + g] = minus_inf
    last = kernel == B.KERNEL_AUTO and dtype == "f32"
    if last:
        st.V[0][n - 1, 20] = inf
    arena.v[:n].copy_(H.to_device_storage(st.V[0], dtype, arena.device))
    ref, _ = O.decode_attn(q64[0, 0], K, synth.storage_to_f64(st.V[0], dtype))
    assert np.isinf(ref).sum() == (2 * G + last) * G
    for chunk in (256, 1024):
        H.set_chunk(arena, chunk)
        out = H.gpu_decode(arena, w, q)[0, 0]
        assert np.array_equal(np.isinf(ref), np.isinf(out)) and np.array_equal(ref[np.isinf(ref)], out[np.isinf(ref)])
        fin = np.isfinite(ref)
        assert np.max(np.abs(out[fin] - ref[fin])) <= 4e-6
    arena.close()


@pytest.mark.parametrize("dtype,D,G", [("bf16", 128, 4), ("bf16", 128, 16), ("bf16", 64, 2), ("f32", 64, 1), ("f32", 64, 3), ("f32", 128, 4), ("f32", 128, 5)])
@pytest.mark.parametrize("track", [False, True])
def test_short_runs_of_small_launches(dtype, D, G, track):
    """The default schedules of layers that runs of 256 or 512 rows would not fill the chip with: runs of 64 rows and
    more, lengths around them, layers of split and of unsplit caches, against the oracle, per layer and all at once; a
    run length set to the default's shortest is followed."""
    H = _h()
    lens = [64, 65, 63, 1, 513, 640, 577, 2, 1000, 1089, 704, 129, 300, 256, 200, 320]  # four layers of four caches
    w = synth.shrink(synth.WORKLOADS["llama1"], name="runs", L=4, Hq=2 * G, Hkv=2, D=D, batch=2, dtype=dtype, seed=97 + G,
                     sink=1, recent=1, slack=0)
    rng = np.random.Generator(np.random.PCG64(w.seed))
    budgets = [max(lens[4 * l + h], lens[4 * l + 2 + h]) + 3 for l in range(w.L) for h in range(2)]
    arena = H.make_arena(w, budgets, track=track)
    st = H.fill_from_host(arena, w, lens, rng)
    q, q64 = H.make_q(w, rng, w.L)
    ref_w = np.zeros(arena.total_tokens)
    for c in range(arena.n_caches):
        l, b, hs = H.q_rows_of_cache(w, c)
        _, p = O.decode_attn(q64[l, b, hs], synth.storage_to_f64(st.K[c], dtype), synth.storage_to_f64(st.V[c], dtype))
        ref_w[arena.off_host[c]:arena.off_host[c] + lens[c]] = p.sum(0)
    tol = 5 * 2.0 ** -17  # two bf16 terms of a weight leave 2^-17 of it, elements of V are below 5
    calls = 0
    for chunk in (None, 512):
        if chunk:
            arena.set_option(B.OPT_CHUNK_TOKENS, chunk)
        H.check_decode_against_oracle(arena, w, st, q64, H.gpu_decode(arena, w, q), tol=tol)
        for l in range(w.L):
            out = H.gpu_decode(arena, w, q[l:l + 1], layer_begin=l, layer_count=1)
            H.check_decode_against_oracle(arena, w, st, q64[l:l + 1], out, caches=range(4 * l, 4 * l + 4), layer_begin=l, tol=tol)
        calls += 2
    if track:
        got = H.download(arena, w).score
        for c in range(arena.n_caches):
            o = int(arena.off_host[c])
            assert np.max(np.abs(got[c] - calls * ref_w[o:o + lens[c]])) <= 2e-6 * calls * G  # fp32 logits of up to 16 in log2 units
    arena.close()


@pytest.mark.parametrize("batch", [64, 65, 96, 97])
def test_work_items_of_whole_model_launches(batch):
    """Numbers of caches around the lines at which a launch over all layers aims at two, three and five work items per
    compute unit, ragged lengths, against the oracle."""
    H = _h()
    w = synth.shrink(synth.WORKLOADS["llama1"], name="whole", L=1, Hq=4, Hkv=2, D=64, batch=batch, seed=120 + batch, sink=1,
                     recent=1, slack=0)
    rng = np.random.Generator(np.random.PCG64(w.seed))
    arena = H.make_arena(w, [1300, 700])
    lens = [int(rng.integers(1, 1301 if c % 2 == 0 else 701)) for c in range(arena.n_caches)]
    st = H.fill_from_host(arena, w, lens, rng)
    q, q64 = H.make_q(w, rng, 1)
    # three bf16 terms of a weight are exact: fp32 logits, weights and sums of up to 1300 rows
    H.check_decode_against_oracle(arena, w, st, q64, H.gpu_decode(arena, w, q), tol=64 * 2.0 ** -24 * 4)
    arena.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_tracked_launch_over_many_caches_beside_a_long_one(dtype):
    """65536 caches, one of 131072 rows: work items times the tiles of the longest one are more threads than a grid
    dimension holds.  A tracked call and a fused one over all of them: outputs, scores, lengths on both sides."""
    n, long_rows = 65536, 131072
    arena = B.Arena(1, n, n, 64, 1, dtype, [1] * (n - 1) + [long_rows], 1, 0, 0, B.POLICY_SCORE, True)
    gen = torch.Generator(device=arena.device)
    gen.manual_seed(41)
    for t in (arena.k, arena.v):
        t.normal_(generator=gen)
    lens = np.asarray(arena.cap_host) - 1
    arena.set_lengths(lens)
    q, kn, vn = (torch.randn((1, 1, n, 64), generator=gen, device=arena.device).to(arena.k.dtype) for _ in range(3))
    out = torch.full((1, 1, n, 64), float("nan"), dtype=torch.float32, device=arena.device)
    off = torch.from_numpy(arena.off_host[:-1]).to(arena.device)
    o = int(arena.off_host[-1])

    def long_cache(m):
        p = torch.softmax(arena.k[o:o + m].double() @ q[0, 0, -1].double() / 8.0, 0)
        return p @ arena.v[o:o + m].double(), p

    arena.decode_attn(0, 1, q, out)
    ref, p = long_cache(long_rows)
    assert torch.equal(out[0, 0, :-1], arena.v[off].float())                     # one row: all of its weight
    assert torch.equal(arena.score[off], torch.ones(n - 1, device=arena.device))
    # fp32 sums of 131072 weights and logits of up to about 10: well inside 2^-16
    assert (out[0, 0, -1].double() - ref).abs().max() <= 2.0 ** -16
    assert (arena.score[o:o + long_rows].double() - p).abs().max() <= 2.0 ** -16
    arena.append_decode_attn(0, 1, kn, vn, 7, q, out)
    assert arena.lengths().tolist() == arena.len.cpu().tolist() == (lens + 1).tolist()
    ref, p2 = long_cache(long_rows + 1)
    assert (out[0, 0, -1].double() - ref).abs().max() <= 2.0 ** -16
    p2[:long_rows] += p
    assert (arena.score[o:o + long_rows + 1].double() - p2).abs().max() <= 2.0 ** -15
    two = torch.softmax((torch.stack([arena.k[off], arena.k[off + 1]]).double() * q[0, 0, :-1].double()).sum(2) / 8.0, 0)
    want = two[0, :, None] * arena.v[off].double() + two[1, :, None] * arena.v[off + 1].double()
    assert (out[0, 0, :-1].double() - want).abs().max() <= 2.0 ** -16
    assert (arena.score[off].double() - 1 - two[0]).abs().max() <= 2.0 ** -16
    assert (arena.score[off + 1].double() - two[1]).abs().max() <= 2.0 ** -16
    arena.close()


@pytest.mark.parametrize("dtype,D,G,track", [("bf16", 128, 4, False), ("bf16", 128, 4, True), ("bf16", 64, 2, True), ("f32", 64, 2, True), ("f32", 128, 4, False)])
def test_launches_over_several_layers(dtype, D, G, track):
    """Launches over some of the layers: short runs fill the chip for one layer or two, over more layers the launch
    takes the longer ones it would take if they had been asked for (bit for bit), against the oracle, with steps that
    append and a flush of the range in between."""
    H = _h()
    L, rows = 9, [1500, 700, 2600, 513, 3100, 64, 4000, 1999]
    w = synth.shrink(synth.WORKLOADS["llama1"], name="several", L=L, Hq=8 * G, Hkv=8, D=D, batch=1, dtype=dtype, seed=131,
                     sink=1, recent=1, slack=4)
    budgets = [rows[(h + l) % 8] for l in range(L) for h in range(8)]
    arenas = [H.make_arena(w, budgets, track=track) for _ in range(2)]
    arenas[1].set_option(B.OPT_CHUNK_TOKENS, 512)                 # the default's shortest run, asked for
    states = [H.fill_from_host(a, w, budgets, np.random.Generator(np.random.PCG64(132)), scores="zero") for a in arenas]
    rng = np.random.Generator(np.random.PCG64(133))
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for lb, lc in ((0, 8), (1, 8), (1, 2), (3, 1)):
        q, q64 = H.make_q(w, rng, lc)
        outs = [H.gpu_decode(a, w, q, layer_begin=lb, layer_count=lc) for a in arenas]
        H.check_decode_against_oracle(arenas[0], w, states[0], q64, outs[0], caches=range(8 * lb, 8 * (lb + lc)), layer_begin=lb,
                                      tol=5 * 2.0 ** -17)  # two bf16 terms of a weight leave 2^-17 of it, elements of V are below 5
        if lc == 8 and cus == 256:
            assert np.array_equal(outs[0], outs[1])
        for a in arenas:
            a.flush_scores(lb, lc)
    kn, vn = (H.to_device_storage(synth.payload(rng, (8, 1, 8, D), dtype), dtype, arenas[0].device) for _ in range(2))
    q = H.to_device_storage(H.make_q(w, rng, 8)[0], dtype, arenas[0].device)
    out = [torch.empty((8, 1, 8 * G, D), dtype=torch.float32, device=q.device) for _ in range(2)]
    for t in range(3):
        for a, o in zip(arenas, out):
            a.append_decode_attn(1, 8, kn, vn, 9000 + t, q, o)
        if cus == 256:
            assert torch.equal(out[0], out[1])
    got, want = (H.download(a, w) for a in arenas)
    for c in range(arenas[0].n_caches):
        # at most 7 calls of G weights, each from an fp32 logit of up to 16 in log2 units
        assert np.max(np.abs(got.score[c] - want.score[c])) <= 2e-6 * 7 * G
        assert np.array_equal(got.K[c], want.K[c]) and np.array_equal(got.pos[c], want.pos[c])
    for a in arenas:
        a.close()


@pytest.mark.parametrize("whole", [False, True])
def test_item_target_set_to_its_default_is_followed(whole):
    """An item target that equals the default ends the default's short runs like any other: the same work items (and
    bits) as after a detour over another target."""
    H = _h()
    L = 1 if whole else 2
    w = synth.shrink(synth.WORKLOADS["llama1"], name="target", L=L, Hq=8, Hkv=2, batch=1, seed=141, sink=1, recent=1, slack=0)
    budgets = [900, 2100, 700, 3000][:2 * L]
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    option, default = (B.OPT_TARGET_ITEMS_WHOLE, 2 * cus) if whole else (B.OPT_TARGET_ITEMS, cus)
    q = H.make_q(w, np.random.Generator(np.random.PCG64(142)), 1)[0]
    outs = []
    for targets in ([], [default], [default + 1, default]):
        arena = H.make_arena(w, budgets)
        H.fill_from_host(arena, w, budgets, np.random.Generator(np.random.PCG64(143)))
        for t in targets:
            arena.set_option(option, t)
        outs.append(H.gpu_decode(arena, w, q, layer_begin=0, layer_count=1))
        arena.close()
    assert np.array_equal(outs[1], outs[2])
    assert not np.array_equal(outs[0], outs[1])      # (short runs, so other sums)
