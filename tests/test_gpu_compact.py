"""GPU parity: baklava_compact against the oracle's eviction -- kept-index lists and lengths
bit-exact, moved K/V/score/pos rows bit-identical to the rows they came from."""
import ctypes as C

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


def run_compact_and_check(arena, w, st, policy=B.POLICY_SCORE, layer_begin=0, layer_count=None, want_lists=True):
    H = _h()
    layer_count = w.L if layer_count is None else layer_count
    kept_dev = torch.full((arena.total_tokens,), -1, dtype=torch.int32, device=arena.device) if want_lists else None
    arena.compact(layer_begin, layer_count, kept_dev)
    torch.cuda.synchronize()
    after = H.download(arena, w)
    dev_len = arena.len.cpu().numpy()
    host_len = arena.lengths()
    cpl = w.batch * w.Hkv
    for c in range(arena.n_caches):
        n = st.K[c].shape[0]
        in_range = layer_begin * cpl <= c < (layer_begin + layer_count) * cpl
        if not in_range:
            assert dev_len[c] == n and host_len[c] == n
            assert np.array_equal(after.K[c], st.K[c]) and np.array_equal(after.V[c], st.V[c])
            continue
        b = int(arena.budget_host[(c // cpl) * w.Hkv + c % w.Hkv])
        recent = w.recent
        kept = O.compact_select(st.score[c], n, b, w.sink, recent, policy)
        assert dev_len[c] == len(kept) == min(n, b), f"cache {c}"
        assert host_len[c] == len(kept)
        if want_lists:
            o = int(arena.off_host[c])
            got = kept_dev[o:o + len(kept)].cpu().numpy()
            assert np.array_equal(got, np.asarray(kept, dtype=np.int32)), f"cache {c}: kept list differs"
        # rows moved bit-exactly
        assert np.array_equal(after.K[c], st.K[c][kept]), f"cache {c}: K rows"
        assert np.array_equal(after.V[c], st.V[c][kept]), f"cache {c}: V rows"
        assert np.array_equal(after.score[c].view(np.uint32), st.score[c][kept].view(np.uint32))
        assert np.array_equal(after.pos[c], st.pos[c][kept])
    return after


def test_tiny_workload_decode_compact_decode():
    """One decode over the full 256-row caches, eviction to budgets {64, 192} from U(0,1) scores,
    one decode over the compacted caches: all three results against the oracle."""
    H = _h()
    w = synth.WORKLOADS["tiny"]
    rng = np.random.Generator(np.random.PCG64(w.seed))
    arena = H.make_arena(w)
    st = H.fill_from_host(arena, w, [w.ctx] * arena.n_caches, rng, scores="uniform")
    q, q64 = H.make_q(w, rng, w.L)
    H.check_decode_against_oracle(arena, w, st, q64, H.gpu_decode(arena, w, q))
    after = run_compact_and_check(arena, w, st)
    assert arena.lengths().tolist() == [64, 192]
    q2, q264 = H.make_q(w, rng, w.L)
    H.check_decode_against_oracle(arena, w, after, q264, H.gpu_decode(arena, w, q2))
    # a second compaction changes nothing
    again = run_compact_and_check(arena, w, after)
    for c in range(arena.n_caches):
        assert np.array_equal(again.K[c], after.K[c])
    arena.close()


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("f32", 64), ("bf16", 64), ("f32", 128)])
def test_ragged_compaction_all_row_sizes(dtype, D):
    H = _h()
    w = synth.shrink(synth.WORKLOADS["llama32"], name="cmp", L=3, Hq=8, Hkv=4, D=D, batch=2, dtype=dtype,
                     seed=21, sink=4, recent=16, slack=700)
    rng = np.random.Generator(np.random.PCG64(w.seed))
    budgets = [20, 21, 100, 128, 129, 300, 511, 512, 513, 1000, 33, 64]
    arena = H.make_arena(w, budgets)
    cpl = w.batch * w.Hkv
    lens = []
    for c in range(arena.n_caches):
        b = budgets[(c // cpl) * w.Hkv + c % w.Hkv]
        extra = [0, 1, 64, 700, 127, 129, 333, -5][c % 8]      # at, just over, far over and under budget
        lens.append(max(1, b + extra))
    st = H.fill_from_host(arena, w, lens, rng, scores="uniform")
    after = run_compact_and_check(arena, w, st, layer_begin=1, layer_count=1)      # one layer only
    after = run_compact_and_check(arena, w, after)                                 # then everything
    arena.close()


def test_ties_zero_scores_and_signed_zero():
    """All-equal scores (ties everywhere), coarse scores with many ties, and -0.0 vs +0.0."""
    H = _h()
    w = synth.shrink(synth.WORKLOADS["llama32"], name="ties", L=1, Hq=6, Hkv=3, batch=1, seed=22, sink=2,
                     recent=3, slack=3000)
    rng = np.random.Generator(np.random.PCG64(w.seed))
    budgets = [40, 700, 1500]
    arena = H.make_arena(w, budgets)
    lens = [900, 2600, 4400]
    st = H.fill_from_host(arena, w, lens, rng, scores="zero")
    # cache 0: all zero; cache 1: coarse grid; cache 2: zeros of both signs plus a few values
    s1 = (rng.integers(0, 5, lens[1]) / 4).astype(np.float32)
    s2 = np.where(rng.random(lens[2]) < 0.5, np.float32(0.0), np.float32(-0.0)).astype(np.float32)
    s2[rng.integers(0, lens[2], 50)] = rng.random(50).astype(np.float32)
    s2[rng.integers(0, lens[2], 20)] = -rng.random(20).astype(np.float32)
    for c, s in ((1, s1), (2, s2)):
        o = int(arena.off_host[c])
        arena.score[o:o + lens[c]].copy_(torch.from_numpy(s).to(arena.device))
        st.score[c] = s
    run_compact_and_check(arena, w, st)
    arena.close()


def test_streaming_policy():
    H = _h()
    w = synth.shrink(synth.WORKLOADS["llama32"], name="stream", L=2, Hq=4, Hkv=2, batch=2, seed=23, sink=4,
                     recent=0, slack=500)
    rng = np.random.Generator(np.random.PCG64(w.seed))
    budgets = [100, 257, 64, 4]
    arena = H.make_arena(w, budgets, policy=B.POLICY_STREAMING)
    cpl = w.batch * w.Hkv
    lens = [budgets[(c // cpl) * w.Hkv + c % w.Hkv] + (c * 37) % 400 for c in range(arena.n_caches)]
    st = H.fill_from_host(arena, w, lens, rng, scores="uniform")
    after = run_compact_and_check(arena, w, st, policy=B.POLICY_STREAMING)
    for c in range(arena.n_caches):
        b = budgets[(c // cpl) * w.Hkv + c % w.Hkv]
        if lens[c] > b:
            expect = list(range(min(4, b))) + list(range(lens[c] - (b - 4), lens[c]))
            assert after.pos[c].tolist() == expect
    arena.close()


def test_budget_equal_sink_plus_recent_keeps_no_middle_row():
    H = _h()
    w = synth.shrink(synth.WORKLOADS["llama32"], name="edge", L=1, Hq=2, Hkv=1, batch=1, seed=24, sink=4,
                     recent=16, slack=100)
    rng = np.random.Generator(np.random.PCG64(w.seed))
    arena = H.make_arena(w, [20])
    st = H.fill_from_host(arena, w, [120], rng, scores="uniform")
    after = run_compact_and_check(arena, w, st)
    assert after.pos[0].tolist() == [0, 1, 2, 3] + list(range(104, 120))
    arena.close()


def test_infeasible_budget_is_refused_at_creation():
    H = _h()
    w = synth.shrink(synth.WORKLOADS["llama32"], name="bad", L=1, Hq=2, Hkv=1, batch=1, sink=4, recent=16)
    with pytest.raises(B.BaklavaError) as e:
        H.make_arena(w, [19])
    assert e.value.status == B.EINFEASIBLE


@pytest.mark.parametrize("slack", [1, 64, 700])
def test_long_caches_move_in_many_tiles(slack):
    """Caches of 16 to 51 tiles of the move (256 rows): budgets of one row less than whole tiles, of whole tiles and of one
    row more, rows that move by fewer and by more than a tile has, from random places and all from the front."""
    H = _h()
    w = synth.shrink(synth.WORKLOADS["llama32"], name="far", L=1, Hq=8, Hkv=4, batch=2, seed=25, sink=4,
                     recent=16, slack=slack)
    rng = np.random.Generator(np.random.PCG64(w.seed + slack))
    budgets = [4095, 4096, 4097, 13000]
    arena = H.make_arena(w, budgets)
    lens = [b + slack for b in budgets] + [b + max(1, slack // 2) for b in budgets]
    st = H.fill_from_host(arena, w, lens, rng, scores="uniform")
    after = run_compact_and_check(arena, w, st)
    # evictions concentrated at the very front: every later row shifts by the full amount
    st2 = H.fill_from_host(arena, w, lens, rng, scores="uniform")
    for c in range(arena.n_caches):
        s = np.ones(lens[c], dtype=np.float32)
        s[4:4 + 2 * slack] = 0.0
        o = int(arena.off_host[c])
        arena.score[o:o + lens[c]].copy_(torch.from_numpy(s).to(arena.device))
        st2.score[c] = s
    run_compact_and_check(arena, w, st2)
    arena.close()


@pytest.mark.parametrize("layers,slack", [(1, 1), (1, 127), (1, 5000), (24, 200), (24, 6000)])
def test_move_of_fewer_and_of_more_tiles_than_compute_units(layers, slack):
    """One layer has about 100 tiles of the move, so every workgroup takes at most one, 24 have 2300, so each takes several
    and waits for tiles that others hold: evictions of fewer and of more rows than a tile has, from random places and
    all from the front, beside caches that one workgroup moves."""
    H = _h()
    w = synth.shrink(synth.WORKLOADS["llama32"], name="tickets", L=layers, Hq=6, Hkv=6, batch=1, seed=27, sink=4,
                     recent=16, slack=slack)
    rng = np.random.Generator(np.random.PCG64(w.seed + slack))
    budgets = [127, 128, 129, 2047, 2049, 20001] * layers
    arena = H.make_arena(w, budgets)
    lens = [b + slack - (c % 3) * (slack // 3) for c, b in enumerate(budgets)]
    st = H.fill_from_host(arena, w, lens, rng, scores="uniform")
    for c in range(1, arena.n_caches, 2):
        st.score[c][4:4 + slack] = 0.0          # evicted rows all at the front: every later row moves
        o = int(arena.off_host[c])
        arena.score[o:o + lens[c]].copy_(torch.from_numpy(st.score[c]).to(arena.device))
    run_compact_and_check(arena, w, st)
    arena.close()


@pytest.mark.parametrize("dtype,D,tile", [("bf16", 64, 512), ("bf16", 128, 256), ("f32", 128, 128)])
@pytest.mark.parametrize("slack", [1, 255, 257, 5000])
def test_move_tiles_wait_for_one_another(dtype, D, tile, slack):
    """The move takes its rows in tiles, each of which may be overwritten once the tiles before it have been read:
    destination ranges of one row less, exactly and one row more than whole tiles, rows that move by less than a tile and
    by many, from random places and all from the front, beside caches (the first one among them) that stay as they are."""
    H = _h()
    w = synth.shrink(synth.WORKLOADS["llama32"], name="tiles", L=3, Hq=5, Hkv=5, D=D, dtype=dtype, batch=1, seed=29,
                     sink=0, recent=0, slack=slack)
    rng = np.random.Generator(np.random.PCG64(w.seed + slack))
    budgets = [60, tile - 1, tile, 2 * tile + 1, 40 * tile] * w.L
    arena = H.make_arena(w, budgets)
    lens = [b if c % 5 == 0 else b + slack for c, b in enumerate(budgets)]
    st = H.fill_from_host(arena, w, lens, rng, scores="uniform")
    for c in range(5, 10):
        st.score[c][:slack] = 0.0
        o = int(arena.off_host[c])
        arena.score[o:o + lens[c]].copy_(torch.from_numpy(st.score[c]).to(arena.device))
    after = run_compact_and_check(arena, w, st, layer_begin=1, layer_count=2)
    for c in range(5, 15):
        st.K[c], st.V[c], st.score[c], st.pos[c] = after.K[c], after.V[c], after.score[c], after.pos[c]
    run_compact_and_check(arena, w, st)
    arena.close()


@pytest.mark.parametrize("policy", [B.POLICY_SCORE, B.POLICY_STREAMING])
@pytest.mark.parametrize("never,tiled_rows", [("cap", None), ("cap + 1", None), (10**6, 8192), (2**31 - 1, None), (2**31 - 1, 8192)])
def test_budgets_at_and_above_the_capacity(policy, never, tiled_rows):
    """A budget that is not below the capacity is a cache that never evicts, on every way the selection takes (one
    workgroup, several, tile by tile), in front of, between and behind caches that do.  A layer of such caches alone
    leaves 20 bytes of a result each in the workspace, and nothing is written behind the workspace."""
    H = _h()
    w = synth.shrink(synth.WORKLOADS["llama32"], name="never", L=3, Hq=6, Hkv=6, D=64, batch=1, seed=33, sink=2,
                     recent=0 if policy == B.POLICY_STREAMING else 3, slack=40)
    rows = [24, 300, 130, 17000, 70000, 24]
    arena = H.make_arena(w, rows * w.L, policy=policy)
    arena.close()
    cap = np.asarray(arena.cap_host, dtype=np.int64)
    unlimited = [True] * 6 + [True, False, True, False, True, False] + [False, True, False, True, False, True]
    arena.budget_host = np.array([{"cap": cap[c], "cap + 1": cap[c] + 1}.get(never, never) if u else rows[c % 6]
                                  for c, u in enumerate(unlimited)]).astype(np.int32)
    arena.budget.copy_(torch.from_numpy(arena.budget_host).to(arena.device))
    d, i32, i64 = arena.desc, C.POINTER(C.c_int32), C.POINTER(C.c_int64)
    cap_p, budget_p = arena.cap_host.ctypes.data_as(i32), arena.budget_host.ctypes.data_as(i32)
    ws_bytes = B.lib().baklava_workspace_bytes(C.byref(d), cap_p, budget_p)
    ws = torch.full((ws_bytes + (1 << 20),), 0xFF, dtype=torch.uint8, device=arena.device)
    d.workspace, d.workspace_bytes = ws.data_ptr(), ws_bytes
    ctx = C.c_void_p()
    assert B.lib().baklava_create(C.byref(d), arena.off_host.ctypes.data_as(i64), cap_p, None, budget_p, C.byref(ctx)) == B.OK
    arena.ctx = ctx
    if tiled_rows:
        arena.set_option(B.OPT_TILED_SELECT_ROWS, tiled_rows)
    rng = np.random.Generator(np.random.PCG64(w.seed))
    st = H.fill_from_host(arena, w, cap.tolist(), rng, scores="uniform")
    before = ws.clone()
    run_compact_and_check(arena, w, st, policy, layer_begin=0, layer_count=1, want_lists=False)
    assert int((ws != before).sum()) <= 20 * 6
    after = run_compact_and_check(arena, w, st, policy, layer_begin=2, layer_count=1)
    run_compact_and_check(arena, w, after, policy)
    assert bool((ws[ws_bytes:] == 0xFF).all())
    arena.close()


@pytest.mark.parametrize("dtype,D", [("bf16", 64), ("bf16", 128), ("f32", 128)])
@pytest.mark.parametrize("budgets", [[20, 127, 128, 64], [20, 127, 128, 129], [129, 3000, 128, 20], [129, 700, 128, 3000],
                                     [129, 700, 128, 3000, 511, 512, 513], [128, 3, 20, 128, 127],
                                     [255, 256, 20, 129], [257, 256, 3000, 600]])
@pytest.mark.parametrize("slack", [1, 129, 1000])
def test_short_caches_apart_from_tiles(dtype, D, budgets, slack):
    """A workgroup moves a cache of up to 128 rows of budget (256 of 128 bytes) where a quarter of all caches or more have no
    more: all of them, that many, exactly a quarter and fewer, some of them within their budget, by the whole and by one
    layer."""
    H = _h()
    n = len(budgets)
    w = synth.shrink(synth.WORKLOADS["llama32"], name="short", L=2, Hq=n, Hkv=n, D=D, dtype=dtype, batch=3, seed=34, sink=1,
                     recent=2, slack=slack)
    rng = np.random.Generator(np.random.PCG64(w.seed + slack))
    arena = H.make_arena(w, budgets + budgets[::-1])
    lens = [max(1, int(x) - slack * (c % 5 == 0) - (c % 3 == 1) * (slack // 2)) for c, x in enumerate(arena.cap_host)]
    st = H.fill_from_host(arena, w, lens, rng, scores="uniform")
    after = run_compact_and_check(arena, w, st, layer_begin=1, layer_count=1)
    run_compact_and_check(arena, w, after)
    arena.close()


@pytest.mark.parametrize("longer", [None, 5, 261])
def test_move_of_more_caches_than_a_launch_serves(longer):
    """8190 + 5 caches of a few rows, alone and beside others of more than 256: the move takes 8192 per launch."""
    H = _h()
    w = synth.shrink(synth.WORKLOADS["llama32"], name="many", L=1, Hq=5, Hkv=5, D=64, batch=1639, seed=30, sink=1,
                     recent=2, slack=3)
    rng = np.random.Generator(np.random.PCG64(w.seed))
    budgets = [3, 4, 5, 9, 17] if longer is None else [259, longer, 4, 260, 259]
    arena = H.make_arena(w, budgets)
    st = H.fill_from_host(arena, w, [budgets[c % 5] + c % 4 for c in range(arena.n_caches)], rng, scores="uniform")
    run_compact_and_check(arena, w, st)
    arena.close()


@pytest.mark.parametrize("scores", ["uniform", "equal", "coarse", "signed", "infinite"])
def test_caches_ranked_in_registers(scores):
    """Caches ranked from registers in blocks of 1024 rows: up to 16384 rows of capacity by one workgroup, beyond (so few
    of them) by one per 8192 rows, tile by tile beyond 65536: middles of one row less, exactly and one row more than a
    block, capacities on both sides of the two limits, one and all but one middle row to keep, ties that span wavefronts
    and blocks, scores of the type's extremes."""
    H = _h()
    w = synth.shrink(synth.WORKLOADS["tiny"], name="held", L=1, Hq=12, Hkv=12, batch=1, seed=28, sink=3,
                     recent=5, slack=1100)
    rng = np.random.Generator(np.random.PCG64(w.seed))
    budgets = [9, 63, 1030, 1031, 1032, 2055, 15284, 15285, 40000, 64436, 64437, 8]
    arena = H.make_arena(w, budgets)
    lens = [10, 72, 1031 + 8, 1033, 1032 + 1024, 2055 + 1, 16384, 16385, 41100, 65536, 65537, 1108]
    st = H.fill_from_host(arena, w, lens, rng, scores="uniform")
    for c, n in enumerate(lens):
        if scores == "equal":
            s = np.full(n, -0.5, dtype=np.float32)
        elif scores == "coarse":
            s = (rng.integers(0, 3, n) / 2).astype(np.float32)
        elif scores == "signed":
            s = (rng.standard_normal(n) * np.exp(rng.standard_normal(n) * 8)).astype(np.float32)
        elif scores == "infinite":
            big = np.finfo(np.float32).max
            s = rng.choice(np.array([-np.inf, -big, -0.0, 0.0, 1e-45, big, np.inf], dtype=np.float32), n)
        else:
            continue
        o = int(arena.off_host[c])
        arena.score[o:o + n].copy_(torch.from_numpy(s).to(arena.device))
        st.score[c] = s
    run_compact_and_check(arena, w, st)
    arena.close()


@pytest.mark.parametrize("free,n_narrow", [(4, 24), (4, 25), (0, 1), (60, 1), (-100, 200)])
def test_wide_and_narrow_caches_in_one_launch_or_two(free, n_narrow):
    """Wide caches that leave `free` compute units idle in their last round, beside up to six narrow ones for each (one
    launch) and more (two)."""
    sink, recent, slack = 3, 5, 40
    n_wide = torch.cuda.get_device_properties(0).multi_processor_count - free
    rng = np.random.Generator(np.random.PCG64(291))
    budgets = rng.permutation([16385 - slack + i % 3 for i in range(n_wide)] + [8 + 37 * i % 3000 for i in range(n_narrow)])
    n = len(budgets)
    arena = B.Arena(1, n, n, 64, 1, "bf16", [int(b) for b in budgets], slack, sink, recent, B.POLICY_SCORE, False,
                    workspace_fill=0xFF)
    lens = [int(c) - i % 45 for i, c in enumerate(arena.cap_host)]
    lens = [max(1, x) for x in lens]
    s = rng.standard_normal(arena.total_tokens).astype(np.float32)
    arena.score.copy_(torch.from_numpy(s).to(arena.device))
    arena.set_lengths(lens)
    kept_dev = torch.full((arena.total_tokens,), -1, dtype=torch.int32, device=arena.device)
    arena.compact(0, 1, kept_dev)
    got = kept_dev.cpu().numpy()
    assert arena.lengths().tolist() == arena.len.cpu().tolist() == [min(x, int(b)) for x, b in zip(lens, budgets)]
    for c in range(n):
        o = int(arena.off_host[c])
        kept = O.compact_select(s[o:o + lens[c]], lens[c], int(budgets[c]), sink, recent)
        assert np.array_equal(got[o:o + len(kept)], np.asarray(kept, dtype=np.int32)), f"cache {c}"
    arena.close()


@pytest.mark.parametrize("scores", ["uniform", "equal", "coarse", "signed", "infinite"])
def test_wide_caches_ranked_by_one_workgroup_each(scores):
    """Beside so many caches of more than 16384 rows that sharing them would not pay, one workgroup ranks each from its
    registers: the middles, capacities and scores of the test above in that form."""
    H = _h()
    sink, recent, slack, n_more = 3, 5, 1100, 125
    budgets = [9, 63, 1030, 1031, 1032, 2055, 15284, 15285, 40000, 64436, 64437, 8, 17500, 31700] + [15285] * n_more
    lens = [10, 72, 1031 + 8, 1033, 1032 + 1024, 2055 + 1, 16384, 16385, 41100, 65536, 65537, 1108, 18438, 32776] + [16385] * n_more
    n = len(budgets)
    arena = B.Arena(1, n, n, 64, 1, "bf16", budgets, slack, sink, recent, B.POLICY_SCORE, False, workspace_fill=0xFF)
    wide = [int(c) for c in arena.cap_host if 16384 < c <= 65536]
    assert 2 * sum(-(-c // 8192) for c in wide) > 3 * torch.cuda.get_device_properties(0).multi_processor_count
    gen = torch.Generator(device=arena.device)
    gen.manual_seed(281)
    arena.k.normal_(generator=gen)
    arena.v.normal_(generator=gen)
    arena.pos.copy_(torch.arange(arena.total_tokens, device=arena.device).to(torch.int32))
    rng = np.random.Generator(np.random.PCG64(282))
    big = np.finfo(np.float32).max
    total = arena.total_tokens
    s = {"uniform": lambda: rng.random(total), "equal": lambda: np.full(total, -0.5), "coarse": lambda: rng.integers(0, 3, total) / 2,
         "signed": lambda: rng.standard_normal(total) * np.exp(rng.standard_normal(total) * 8),
         "infinite": lambda: rng.choice(np.array([-np.inf, -big, -0.0, 0.0, 1e-45, big, np.inf], dtype=np.float32), total)}[scores]()
    s = s.astype(np.float32)
    arena.score.copy_(torch.from_numpy(s).to(arena.device))
    arena.set_lengths(lens)
    before = {name: getattr(arena, name).clone() for name in ("k", "v", "score", "pos")}
    kept_dev = torch.full((total,), -1, dtype=torch.int32, device=arena.device)
    arena.compact(0, 1, kept_dev)
    assert arena.lengths().tolist() == arena.len.cpu().tolist() == [min(x, b) for x, b in zip(lens, budgets)]
    for c in list(range(14)) + [n - 2, n - 1]:
        o = int(arena.off_host[c])
        kept = np.asarray(O.compact_select(s[o:o + lens[c]], lens[c], budgets[c], sink, recent))
        assert np.array_equal(kept_dev[o:o + len(kept)].cpu().numpy(), kept.astype(np.int32)), f"cache {c}"
        idx = torch.from_numpy(kept + o).to(arena.device)
        for name in ("k", "v", "score", "pos"):
            got, want = getattr(arena, name)[o:o + len(kept)], before[name][idx]
            assert torch.equal(got.view(torch.int16 if got.dtype == torch.bfloat16 else torch.int32),
                               want.view(torch.int16 if got.dtype == torch.bfloat16 else torch.int32)), f"cache {c}: {name}"
    arena.close()


@pytest.mark.parametrize("policy", [B.POLICY_SCORE, B.POLICY_STREAMING])
@pytest.mark.parametrize("scores", ["uniform", "equal", "coarse", "signed_zero"])
def test_caches_selected_tile_by_tile(scores, policy):
    """Caches beyond 8192 rows of capacity are ranked by several workgroups (tiles of 8192 rows, one
    kernel per radix pass): lengths at, just over and far over the budget, live lengths that end
    inside the first, a middle and the last tile, ties that span tiles (the older row must win across
    a tile boundary), short caches in the same launch, a launch over one layer only."""
    H = _h()
    w = synth.shrink(synth.WORKLOADS["llama32"], name="tiles", L=2, Hq=4, Hkv=4, batch=1, seed=26, sink=4,
                     recent=16, slack=300)
    rng = np.random.Generator(np.random.PCG64(w.seed + policy))
    budgets = [8100, 8192, 8193, 20, 16300, 16384, 24581, 500]
    extra = [300, 1, 150, 77, 0, 300, 299, 37]
    arena = H.make_arena(w, budgets, policy=policy)
    arena.set_option(B.OPT_TILED_SELECT_ROWS, 8192)       # the smallest threshold: six of the eight caches are tiled
    assert sum(1 for c in arena.cap_host if c > 8192) == 6
    lens = [b + e for b, e in zip(budgets, extra)]
    st = H.fill_from_host(arena, w, lens, rng, scores="uniform")
    if scores != "uniform":
        for c in range(arena.n_caches):
            n = lens[c]
            if scores == "equal":
                s = np.full(n, 0.25, dtype=np.float32)
            elif scores == "coarse":
                s = (rng.integers(0, 7, n) / 8).astype(np.float32)
            else:
                s = np.where(rng.random(n) < 0.5, np.float32(0.0), np.float32(-0.0)).astype(np.float32)
                s[rng.integers(0, n, 40)] = rng.random(40).astype(np.float32)
                s[rng.integers(0, n, 40)] = -rng.random(40).astype(np.float32)
            o = int(arena.off_host[c])
            arena.score[o:o + n].copy_(torch.from_numpy(s).to(arena.device))
            st.score[c] = s
    after = run_compact_and_check(arena, w, st, policy=policy, layer_begin=1, layer_count=1)   # tiles of layer 1 only
    after = run_compact_and_check(arena, w, after, policy=policy)                              # then both layers
    run_compact_and_check(arena, w, after, policy=policy)                                      # nothing left to evict
    arena.close()


@pytest.mark.parametrize("policy", [B.POLICY_SCORE, B.POLICY_STREAMING])
@pytest.mark.parametrize("scores", ["uniform", "equal", "coarse", "signed_zero", "negative", "close", "ends"])
def test_few_caches_ranked_by_several_workgroups(scores, policy):
    """Caches of 41020 to 65536 rows of capacity (six to eight tiles), few enough that each is ranked by one workgroup per
    8192 rows: live lengths at the edges of a tile, in the first, a middle and the last tile and at the budget, no
    survivors in the middle, ties across tiles, more keys that share their leading bits than LDS holds (equal and close
    scores), scores of both signs and at the ends of the type."""
    H = _h()
    w = synth.shrink(synth.WORKLOADS["tiny"], name="spread", L=2, Hq=5, Hkv=5, batch=1, seed=27, sink=4, recent=16,
                     slack=41000)
    rng = np.random.Generator(np.random.PCG64(w.seed + policy))
    budgets = [20, 500, 8192, 16000, 24536, 21, 8150, 300, 24535, 12000]
    arena = H.make_arena(w, budgets, policy=policy)
    lens = [41020, 8193, 49192, 16001, 65536, 24577, 8150, 41300, 65535, 30000]
    assert max(arena.cap_host) == 65536 and all(n <= c for n, c in zip(lens, arena.cap_host))
    st = H.fill_from_host(arena, w, lens, rng, scores="uniform")
    if scores != "uniform":
        for c, n in enumerate(lens):
            if scores == "equal":
                s = np.full(n, 0.25, dtype=np.float32)
            elif scores == "coarse":
                s = (rng.integers(0, 7, n) / 8).astype(np.float32)
            elif scores == "negative":
                s = (rng.random(n) * 2 - 1.5).astype(np.float32)
            elif scores == "close":
                s = np.float32(0.75) + (rng.integers(0, 3000, n) * 2.0 ** -24).astype(np.float32)
            elif scores == "ends":
                s = rng.choice(np.array([-np.inf, -3.4e38, -1e-45, -0.0, 0.0, 1e-45, 3.4e38, np.inf], dtype=np.float32), n)
            else:
                s = np.where(rng.random(n) < 0.5, np.float32(0.0), np.float32(-0.0)).astype(np.float32)
                s[rng.integers(0, n, 40)] = rng.random(40).astype(np.float32)
                s[rng.integers(0, n, 40)] = -rng.random(40).astype(np.float32)
            o = int(arena.off_host[c])
            arena.score[o:o + n].copy_(torch.from_numpy(s).to(arena.device))
            st.score[c] = s
    after = run_compact_and_check(arena, w, st, policy=policy, layer_begin=1, layer_count=1)
    after = run_compact_and_check(arena, w, after, policy=policy)
    run_compact_and_check(arena, w, after, policy=policy)                                      # nothing left to evict
    arena.close()


@pytest.mark.parametrize("policy", [B.POLICY_SCORE, B.POLICY_STREAMING])
@pytest.mark.parametrize("scores", ["uniform", "equal", "coarse", "ends"])
def test_shared_caches_beside_short_ones(scores, policy):
    """Caches of up to 16384 rows of capacity, ranked by one workgroup, in one launch with caches of three to eight tiles
    ranked by several: capacities of whole tiles and one row more, full and short live lengths, one of two layers and
    both, and a range without a shared cache."""
    H = _h()
    w = synth.shrink(synth.WORKLOADS["tiny"], name="beside", L=3, Hq=5, Hkv=5, batch=1, seed=30, sink=6, recent=20, slack=700)
    rng = np.random.Generator(np.random.PCG64(w.seed + policy))
    caps = [16384, 16385, 24576, 24577, 900, 32768, 32769, 8192, 5000, 40960, 16384, 8193, 730, 1024, 2000]
    arena = H.make_arena(w, [c - 700 for c in caps], policy=policy)
    lens = [16384, 16385, 24576, 24001, 900, 32768, 32069, 7900, 4300, 8193, 16383, 8193, 30, 1000, 1500]
    st = H.fill_from_host(arena, w, lens, rng, scores="uniform")
    for c, n in enumerate(lens):
        if scores == "equal":
            st.score[c] = np.full(n, 0.25, dtype=np.float32)
        elif scores == "coarse":
            st.score[c] = (rng.integers(0, 5, n) / 4 - 0.5).astype(np.float32)
        elif scores == "ends":
            st.score[c] = rng.choice(np.array([-np.inf, -3.4e38, -1e-45, -0.0, 0.0, 1e-45, 3.4e38, np.inf], dtype=np.float32), n)
        o = int(arena.off_host[c])
        arena.score[o:o + n].copy_(torch.from_numpy(st.score[c]).to(arena.device))
    after = run_compact_and_check(arena, w, st, policy=policy, layer_begin=1, layer_count=1)
    after = run_compact_and_check(arena, w, after, policy=policy, layer_begin=2, layer_count=1)   # no shared cache
    after = run_compact_and_check(arena, w, after, policy=policy, layer_begin=0, layer_count=2)
    run_compact_and_check(arena, w, after, policy=policy)                                      # nothing left to evict
    arena.close()


@pytest.mark.parametrize("share", [0.3, 0.7, 1.0])
def test_lowest_key_among_several_workgroups(share):
    """Scores whose bits are all ones have the lowest key there is, which places without a row hold too.  Rows with it
    that survive are the oldest ones, like rows of -inf if nothing else is below them, also where a cache is ranked by
    several workgroups and its first rows, the sinks, leave the first one fewer than 8192."""
    H = _h()
    w = synth.shrink(synth.WORKLOADS["tiny"], name="lowest", L=1, Hq=3, Hkv=3, batch=1, seed=29, sink=37, recent=5, slack=4000)
    rng = np.random.Generator(np.random.PCG64(w.seed))
    lens = [20481, 33000, 60000]
    arena = H.make_arena(w, [n - 4000 for n in lens])
    st = H.fill_from_host(arena, w, lens, rng, scores="uniform")
    kept_dev = torch.full((arena.total_tokens,), -1, dtype=torch.int32, device=arena.device)
    for c, n in enumerate(lens):
        ones = rng.random(n) < share
        o = int(arena.off_host[c])
        bits = np.where(ones, np.uint32(0xffffffff), st.score[c].view(np.uint32))
        arena.score[o:o + n].copy_(torch.from_numpy(bits.view(np.float32)).to(arena.device))
        st.score[c] = np.where(ones, np.float32(-np.inf), st.score[c])
    arena.compact(0, 1, kept_dev)
    after = H.download(arena, w)
    for c, n in enumerate(lens):
        kept = np.asarray(O.compact_select(st.score[c], n, n - 4000, w.sink, w.recent), dtype=np.int32)
        o = int(arena.off_host[c])
        assert np.array_equal(kept_dev[o:o + len(kept)].cpu().numpy(), kept), f"cache {c}"
        assert np.array_equal(after.K[c], st.K[c][kept]) and np.array_equal(after.pos[c], st.pos[c][kept])
    arena.close()


@pytest.mark.parametrize("seed", list(range(500, 512)))
def test_seeded_random_evictions(seed):
    """Random cache sizes on both sides of the threshold for tile-by-tile selection, random budgets, sink
    and recent windows, live lengths and score distributions (continuous, few distinct values, all equal,
    signed zeros, negative values), both policies, a random layer range first and all layers after it."""
    H = _h()
    r = np.random.Generator(np.random.PCG64(seed))
    policy = B.POLICY_STREAMING if seed % 4 == 0 else B.POLICY_SCORE
    L, Hkv, batch = int(r.integers(1, 4)), int(r.integers(1, 4)), int(r.integers(1, 3))
    sink = int(r.integers(0, 6))
    recent = 0 if policy == B.POLICY_STREAMING else int(r.integers(0, 40))
    slack = int(r.choice([1, 50, 700, 9000]))
    w = synth.shrink(synth.WORKLOADS["tiny"], name=f"evict{seed}", L=L, Hq=Hkv, Hkv=Hkv, batch=batch, seed=seed,
                     sink=sink, recent=recent, slack=slack)
    budgets = [int(max(sink + recent + 1, round(float(np.exp(r.uniform(np.log(16), np.log(30000))))))) for _ in range(L * Hkv)]
    arena = H.make_arena(w, budgets, policy=policy)
    threshold = int(r.choice([8192, 12000, 36864]))
    arena.set_option(B.OPT_TILED_SELECT_ROWS, threshold)
    cap = arena.cap_host
    lens = [int(cap[c]) if r.random() < 0.3 else int(r.integers(0, int(cap[c]) + 1)) for c in range(arena.n_caches)]
    st = H.fill_from_host(arena, w, lens, r, scores="uniform")
    kind = str(r.choice(["uniform", "coarse", "equal", "signed_zero", "negative"]))
    print(f"seed {seed}: policy={policy} L={L} Hkv={Hkv} batch={batch} sink={sink} recent={recent} slack={slack} "
          f"threshold={threshold} scores={kind} budgets={budgets}", flush=True)
    if kind != "uniform":
        for c in range(arena.n_caches):
            n = lens[c]
            if n == 0:
                continue
            if kind == "equal":
                s = np.full(n, 0.25, dtype=np.float32)
            elif kind == "coarse":
                s = (r.integers(0, 5, n) / 4).astype(np.float32)
            elif kind == "negative":
                s = (r.random(n) * 2 - 1).astype(np.float32)
            else:
                s = np.where(r.random(n) < 0.5, np.float32(0.0), np.float32(-0.0)).astype(np.float32)
                s[r.integers(0, n, 8)] = r.random(8).astype(np.float32)
            o = int(arena.off_host[c])
            arena.score[o:o + n].copy_(torch.from_numpy(s).to(arena.device))
            st.score[c] = s
    lb = int(r.integers(0, L))
    lc = int(r.integers(1, L - lb + 1))
    after = run_compact_and_check(arena, w, st, policy=policy, layer_begin=lb, layer_count=lc)
    after = run_compact_and_check(arena, w, after, policy=policy)
    run_compact_and_check(arena, w, after, policy=policy, want_lists=False)
    arena.close()
