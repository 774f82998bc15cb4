"""GPU parity at the places where a kernel's split of the work can go wrong: tile and group edges, segments that share
bitmap words or tiles' groups, remainders, and the sizes at which a call changes its path.  Everything is compared bit for
bit: the oracle defines every result to the bit (order of sums, single roundings, tie rules, random words)."""
import numpy as np
import pytest

import oracle
from paper_1709_09393_amd import binding, workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev():
    if not torch.cuda.is_available():
        pytest.fail("GPU test selected but torch.cuda.is_available() is False")
    return torch.device("cuda:0")


def to_dev(a):
    a = np.ascontiguousarray(a)
    return torch.from_numpy(a.view(np.int32) if a.dtype == np.uint32 else a).to(dev())


def u32(t):
    return t.cpu().numpy().view(np.uint32)


def offsets(sizes):
    return [0] + [int(x) for x in np.cumsum(sizes)]


# segments inside one bitmap word, across words, empty cores, many tiles, a last word that is not full
SEGMENTS = {
    "inside_one_word": [1, 2, 3, 5, 7, 11, 1, 1, 30],
    "words_shared_by_long_tiles": [4096 + 17, 31, 8192 + 1, 3, 4095, 64, 4097],
    "groups_and_segments_interleave": [5 * 4096 + 100, 40, 90 * 4096 + 1, 1000, 4096, 4096, 33],
    "one_tile_each": [4096] * 40 + [13],
}


@pytest.mark.parametrize("values", ["spread", "ties"])
@pytest.mark.parametrize("name", sorted(SEGMENTS))
def test_segmented_selection_publishes_lists_offsets_and_shared_bitmap_words(name, values):
    sizes = SEGMENTS[name]
    so, n = offsets(sizes), sum(sizes)
    rng = np.random.default_rng(len(name))
    S_h = np.abs(rng.standard_normal(n)).astype(np.float32)
    if values == "ties":
        S_h = (rng.integers(0, 5, n) / 8.0).astype(np.float32)
    sd = binding.SlimDP(n, 1, seg_off=so)
    ts = sd.tile_starts().astype(np.int64)
    for part in (3, 1, 2):                       # other core sizes on the same context, empty and full cores among them
        ks = [0 if j % 4 == part else (s if j % 7 == part else s * part // 5) for j, s in enumerate(sizes)]
        core_bits = torch.full(((n + 31) // 32,), -1, dtype=torch.int32, device=dev())
        idx, bits, off, _ = sd.select_core(to_dev(S_h), ks, core_bits=core_bits)
        sd.synchronize()
        want = oracle.select_core(S_h, ks, so)
        assert np.array_equal(u32(idx), want)
        assert np.array_equal(u32(bits), oracle.core_bits(n, want))
        assert np.array_equal(u32(off), np.searchsorted(want.astype(np.int64), ts).astype(np.uint32))
    sd.close()


@pytest.mark.parametrize("n", [4096 * 4, 4096 * 5 + 1, 4096 * 16, 300_001])
def test_selection_leaves_clear_counts_whatever_was_counted_before(n):
    """A selection counts from zero: after another one, after a scoring pass whose histogram nobody used, and after one
    that sorted against another bin than its own."""
    wl = workloads.TINY.scaled(n)
    w, g = to_dev(wl.weights()), [to_dev(x) for x in wl.gradients(0)]
    rng = np.random.default_rng(n)
    other = (np.abs(rng.standard_normal(n)) * 1e-3).astype(np.float32)
    S_o = oracle.score(wl.weights(), wl.gradients(0), wl.c)
    sd = binding.SlimDP(n, wl.W)
    k = wl.k
    for _ in range(2):
        S = sd.score(w, g, wl.c)                 # counted twice, used once
        S = sd.score(w, g, wl.c)
        a = sd.select_core(S, [k], reuse_histogram=True)[0]
        S = sd.score(w, g, wl.c)                 # counted, then a selection on another array
        b = sd.select_core(to_dev(other), [k])[0]
        c = sd.select_core(to_dev(S_o), [n - k])[0]
        sd.synchronize()
        assert np.array_equal(u32(a), oracle.select_core(S_o, k))
        assert np.array_equal(u32(b), oracle.select_core(other, k))
        assert np.array_equal(u32(c), oracle.select_core(S_o, n - k))
    sd.close()


@pytest.mark.parametrize("reuse", [False, True])
def test_first_call_of_a_context_on_a_stream_of_its_own_starts_from_clear_counts(reuse):
    """1.3 GB of histograms (20,000 segments) are clear before a stream that does not wait for the default one counts into
    them."""
    sizes = [3] * 20_000
    so, n = offsets(sizes), sum(sizes)
    ks = [1 + j % 2 for j in range(len(sizes))]
    rng = np.random.default_rng(11)
    w_h, g_h = rng.standard_normal(n).astype(np.float32), [rng.standard_normal(n).astype(np.float32)]
    S_h = oracle.score(w_h, g_h, 1.0)
    want = oracle.select_core(S_h, ks, so)
    w, g, S = to_dev(w_h), [to_dev(x) for x in g_h], to_dev(S_h)
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    for _ in range(3):
        sd = binding.SlimDP(n, 1, seg_off=so, stream=st)
        with torch.cuda.stream(st):
            if reuse:
                sd.score(w, g, 1.0, out=S)
            idx = sd.select_core(S, ks, reuse_histogram=reuse)[0]
        sd.synchronize()
        assert np.array_equal(u32(idx), want)
        sd.close()


@pytest.mark.parametrize("n", [5, 4096 * 3 + 1, 4096 * 40 + 4095])
def test_ragged_tile_is_sorted_also_when_tiles_are_dealt_in_ranges_after_the_scoring_pass(n):
    """Whole tiles are sorted by the scoring pass (its prediction holds from the second iteration on), the ragged one by the
    selection, whose blocks take ranges of tiles when "strided_tiles" is switched off in between."""
    W, k = 2, max(1, n // 3)
    rng = np.random.default_rng(n)
    w_h = rng.standard_normal(n).astype(np.float32)
    g_h = [(1e-3 * rng.standard_normal(n)).astype(np.float32) for _ in range(W)]
    sd = binding.SlimDP(n, W)
    w, g = to_dev(w_h), [to_dev(x) for x in g_h]
    for turn in range(4):
        S = sd.score(w, g, 1.0)
        sd.set_option("strided_tiles", 0 if turn else 1)
        idx = sd.select_core(S, [k], reuse_histogram=True)[0]
        sd.set_option("strided_tiles", 1)
        sd.synchronize()
        assert np.array_equal(u32(idx), oracle.select_core(oracle.score(w_h, g_h, 1.0), k)), turn
        tail = n % 4096                          # the next iteration's ragged tile is another one
        w_h[n - tail:] = w_h[n - tail:][::-1].copy()
        w.copy_(to_dev(w_h))
    sd.close()


@pytest.mark.parametrize("segments", [1, 5])
def test_recorded_selection_replays_beside_eager_ones(segments):
    """Score and selection recorded into a graph give the eager result on every replay, whatever eager calls (other core
    sizes, a scoring pass whose histogram nobody used) ran between recording and replay; eager calls stay right after one."""
    n = 5 * 4096 * 3 + 17
    wl = workloads.TINY.scaled(n)
    so = offsets([n]) if segments == 1 else offsets([4096 + 5, 3, 20_000, 30_001, n - 4096 - 5 - 3 - 50_001])
    sizes = np.diff(so)
    ks, other = [int(s) // 7 for s in sizes], [int(s) // 2 for s in sizes]
    w_h, g_h = wl.weights(), wl.gradients(0)
    w, g = to_dev(w_h), [to_dev(x) for x in g_h]
    S_o = oracle.score(w_h, g_h, wl.c)
    want, want_other = oracle.select_core(S_o, ks, so), oracle.select_core(S_o, other, so)
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    sd = binding.SlimDP(n, wl.W, seg_off=so, stream=st)
    S = torch.empty_like(w)
    idx = torch.empty(sum(ks), dtype=torch.int32, device=dev())
    bits = torch.empty((n + 31) // 32, dtype=torch.int32, device=dev())
    off = torch.empty(sd.T + 1, dtype=torch.int32, device=dev())
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        sd.score(w, g, wl.c, out=S)
        sd.select_core(S, ks, reuse_histogram=True, core_idx=idx, core_bits=bits, core_off=off)
    S2 = torch.empty_like(w)
    for turn in range(3):
        with torch.cuda.stream(st):
            if turn != 1:
                got = sd.select_core(to_dev(S_o), other)[0]
                sd.synchronize()
                assert np.array_equal(u32(got), want_other)
            sd.score(w, g, wl.c, out=S2)         # counted, not used
            idx.zero_()
            graph.replay()
        sd.synchronize()
        assert np.array_equal(u32(S), S_o.view(np.uint32))
        assert np.array_equal(u32(idx), want)
        assert np.array_equal(u32(bits), oracle.core_bits(n, want))
    sd.close()


@pytest.mark.parametrize("recorded", ["score and select", "select", "score"])
@pytest.mark.parametrize("segments", [1, 5])
def test_eager_calls_stay_right_after_calls_that_were_only_recorded(segments, recorded):
    """The first recording begins after an eager scoring pass whose counts nobody used; eager passes follow before the first
    replay (which may never come) and between replays."""
    n = 5 * 4096 * 3 + 17
    wl = workloads.TINY.scaled(n)
    so = offsets([n]) if segments == 1 else offsets([4096 + 5, 3, 20_000, 30_001, n - 4096 - 5 - 3 - 50_001])
    ks = [int(s) // 7 for s in np.diff(so)]
    w_h, g_h = wl.weights(), wl.gradients(0)
    w, g = to_dev(w_h), [to_dev(x) for x in g_h]
    want = oracle.select_core(oracle.score(w_h, g_h, wl.c), ks, so)
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    sd = binding.SlimDP(n, wl.W, seg_off=so, stream=st)
    S = torch.empty_like(w)
    idx = torch.empty(sum(ks), dtype=torch.int32, device=dev())
    bits = torch.empty((n + 31) // 32, dtype=torch.int32, device=dev())
    off = torch.empty(sd.T + 1, dtype=torch.int32, device=dev())
    torch.cuda.synchronize()

    def right():
        sd.synchronize()
        return np.array_equal(u32(idx), want) and np.array_equal(u32(bits), oracle.core_bits(n, want)) and int(u32(off)[-1]) == len(want)

    with torch.cuda.stream(st):
        sd.score(w, g, wl.c, out=S)              # counted, not used
    sd.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        if "score" in recorded:
            sd.score(w, g, wl.c, out=S)
        if "select" in recorded:
            sd.select_core(S, ks, reuse_histogram=True, core_idx=idx, core_bits=bits, core_off=off)
    with torch.cuda.stream(st):
        for _ in range(3):
            idx.zero_()
            sd.score(w, g, wl.c, out=S)
            sd.select_core(S, ks, reuse_histogram=True, core_idx=idx, core_bits=bits, core_off=off)
            assert right(), "eager"
            idx.zero_()
            if recorded == "select":
                sd.score(w, g, wl.c, out=S)
            graph.replay()
            if recorded == "score":              # counted by the replay, not used
                sd.score(w, g, wl.c, out=S)
                sd.select_core(S, ks, reuse_histogram=True, core_idx=idx, core_bits=bits, core_off=off)
            assert right(), "replay"
            sd.score(w, g, wl.c, out=S)          # counted, not used
    sd.close()


def test_static_selection_recorded_between_eager_calls():
    n, k = 50_003, 7_000
    rng = np.random.default_rng(5)
    one, two = (np.abs(rng.standard_normal(n)).astype(np.float32) for _ in range(2))
    S = to_dev(one)
    out = [torch.empty(c, dtype=torch.int32, device=dev()) for c in (k, (n + 31) // 32, binding.num_tiles(n) + 1)]
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())

    def check(values):
        st.synchronize()
        assert np.array_equal(u32(out[0]), oracle.select_core(values, k))
        out[0].zero_()
        torch.cuda.synchronize()

    with torch.cuda.stream(st):
        binding.select_core_static(S, k, *out)
        check(one)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            binding.select_core_static(S, k, *out)
        for values in (one, two, one):
            S.copy_(to_dev(values))
            binding.select_core_static(S, k, *out)
            check(values)
            graph.replay()
            check(values)


@pytest.mark.parametrize("draw", ["none", "pairs", "wide"])
@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("W", [6, 7])
def test_numbers_of_workers_with_a_scoring_kernel_of_their_own(W, dense, draw):
    """Six and seven workers in the pipelined scoring kernel: alone, with an announced draw in either format, and after a dense
    update; the second iteration against the first one's threshold.  One size has several tiles to a block."""
    n = 4096 * (520 if draw == "pairs" and not dense else 9) + 77
    wl = workloads.TINY.scaled(n, W=W)
    sd = binding.SlimDP(n, W, seed=workloads.EXPLORE_SEED)
    sd.set_option("explore_per_tile_tail", int(draw == "wide"))
    w_h = wl.weights()
    w = to_dev(w_h)
    for t in range(2):
        g_h = wl.gradients(t)
        g = [to_dev(x) for x in g_h]
        if draw != "none":
            sd.explore_hint([wl.k], t, [wl.m], 0, W)
        if dense:
            S = sd.dense_update_score(w, g, wl.lr, wl.c)
            w_h, S_o = oracle.dense_update_score(w_h, g_h, wl.lr, wl.c)
        else:
            S, S_o = sd.score(w, g, wl.c), oracle.score(w_h, g_h, wl.c)
        core, bits, _, _ = sd.select_core(S, [wl.k], reuse_histogram=True)
        idx, _ = sd.sample_explore(bits, [wl.k], t, [wl.m], 0, W)
        sd.synchronize()
        core_o = oracle.select_core(S_o, wl.k)
        assert np.array_equal(u32(S), S_o.view(np.uint32)) and np.array_equal(u32(w), w_h.view(np.uint32)), t
        assert np.array_equal(u32(core), core_o) and np.array_equal(u32(bits), oracle.core_bits(n, core_o)), t
        for q in (0, W - 1):
            assert np.array_equal(u32(idx[q]), oracle.sample_explore(n, core_o, workloads.EXPLORE_SEED, t, q, wl.m)), (t, q)
    sd.close()


# kept parameters in the four rounds of 256 of a sub-tile.  Its capture holds 256 entries, a round beginning on a line
# (two entries of sixteen workers): the first group fits, the second has entries that the pack must gather
FITS = [(127, 0, 128, 0), (128, 128, 0, 0), (256, 0, 0, 0), (129, 126, 0, 0), (0, 0, 0, 256), (3, 125, 126, 0), (129, 0, 0, 125), (0, 0, 0, 0)]
SPILLS = [(129, 127, 0, 0), (1, 255, 0, 0), (256, 1, 0, 0), (129, 129, 129, 129), (256, 256, 256, 256), (127, 127, 2, 0)]


@pytest.mark.parametrize("spills", [False, True])
@pytest.mark.parametrize("W", [1, 8, 16])
def test_capture_of_clustered_parameters(W, spills):
    """Rounds at the edges of what is staged at a time (128 entries of sixteen workers, 256 of fewer) and of a sub-tile's
    capture.  Where everything fits, the updates are zeroed before the pack: its values can only be those kept."""
    tiles, tail = 7, 50
    n = tiles * 4096 + tail
    rng = np.random.default_rng(W)
    line = 32 // W                               # entries of a line of 128 bytes
    groups = [f for f in FITS if sum((x + line - 1) // line * line for x in f) <= 256] + (SPILLS if spills else [])
    big = np.zeros(n, bool)
    for j in range(tiles * 4):
        for r, count in enumerate(groups[j % len(groups)]):
            big[j * 1024 + r * 256 + rng.choice(256, count, replace=False)] = True
    w_h = np.where(big, 1.0 + rng.random(n), 0.01 * rng.random(n)).astype(np.float32)
    k, m = int(big.sum()), 7
    sd = binding.SlimDP(n, W, seed=workloads.EXPLORE_SEED)
    sd.set_option("speculative_pack", 1)
    w = to_dev(w_h)
    for t in range(3):                           # the first selection sets the bound that the second pass captures under
        g_h = [(1e-3 * rng.standard_normal(n)).astype(np.float32) for _ in range(W)]
        g = [to_dev(x) for x in g_h]
        S = sd.score(w, g, 1.0)
        core, bits, off, epoch = sd.select_core(S, [k], reuse_histogram=True)
        idx, eoff = sd.sample_explore(bits, [k], t, [m], 0, W)
        clobber = t > 0 and not spills
        if clobber:
            for x in g:
                x.zero_()
        core_val, _ = sd.pack(g, core, off, idx, eoff, epoch, updates_as_scored=True)
        sd.synchronize()
        assert np.array_equal(u32(core), np.flatnonzero(big).astype(np.uint32)), t
        for q in range(W):
            assert np.array_equal(u32(core_val[q]), g_h[q][big].view(np.uint32)), (t, q)
    sd.close()


@pytest.mark.parametrize("W,pct", [(1, 2), (2, 1), (4, 5), (8, 2), (16, 2), (16, 5)])
def test_explorer_values_kept_by_the_scoring_pass(W, pct):
    """The draw by rounds and the values it keeps (32 or 48 slots a sub-tile, a ragged tile, more workers announced than scored),
    and packs whose lists are not, or no longer, the ones that were drawn with it."""
    n, more = 4096 * (220 if pct < 5 else 520) + 777, 2          # narrow zones
    wl = workloads.TINY.scaled(n)
    k = n // 10
    m = (n - k) * pct // 100
    rng = np.random.default_rng(W * 10 + pct)
    sd = binding.SlimDP(n, W + more, seed=workloads.EXPLORE_SEED)
    options = [("speculative_pack", 1), ("explore_keep", 2)]          # the later one makes the room
    for name, value in options if W != 2 else options[::-1]:
        sd.set_option(name, value)
    ts = sd.tile_starts().astype(np.int64)
    w = to_dev(wl.weights())
    for t, how in enumerate(["as drawn", "as drawn", "updates gone", "more workers", "another draw between", "other lists"]):
        first, drawn = (3, W + more) if how == "more workers" else (0, W)
        g_h = [(1e-3 * rng.standard_normal(n)).astype(np.float32) for _ in range(W)]
        g = [to_dev(x) for x in g_h]
        sd.explore_hint([k], t, [m], first, drawn)
        S = sd.score(w, g, 1.0)
        core, bits, off, epoch = sd.select_core(S, [k], reuse_histogram=True)
        idx, eoff = sd.sample_explore(bits, [k], t, [m], first, drawn)
        core_h = u32(core)
        for q in {0, drawn - 1}:
            want = oracle.sample_explore(n, core_h, workloads.EXPLORE_SEED, t, first + q, m)
            assert np.array_equal(u32(idx[q]), want), (how, q)
            assert np.array_equal(u32(eoff[q]), np.searchsorted(want.astype(np.int64), ts).astype(np.uint32)), (how, q)
        if how == "another draw between":
            sd.sample_explore(bits, [k], t + 100, [m], 0, W)
        if how == "other lists":
            idx = [to_dev(np.sort(rng.choice(n, m, replace=False)).astype(np.uint32)) for _ in range(W)]
            eoff = [to_dev(np.searchsorted(u32(x).astype(np.int64), ts).astype(np.uint32)) for x in idx]
        if how == "updates gone":                # the pack finds the kept values and, in place of the others, nothing
            for x in g:
                x.zero_()
        _, expl_val = sd.pack(g, core, off, idx[:W], eoff[:W], epoch, updates_as_scored=True)
        sd.synchronize()
        for q in range(W):
            got, want = u32(expl_val[q]), g_h[q][u32(idx[q])].view(np.uint32)
            if how == "updates gone":
                assert np.all((got == want) | (got == 0)) and np.mean(got == want) > 0.8
            else:
                assert np.array_equal(got, want), (how, q)
    sd.close()


@pytest.mark.parametrize("segmented", [False, True])
@pytest.mark.parametrize("W,shift", [(1, 1), (2, 3), (3, 2), (5, 1), (8, 1), (8, 2), (12, 3), (16, 1), (20, 2)])
def test_sixteen_byte_access_from_any_float_address(W, shift, segmented):
    """Model, updates and scores that begin 4, 8 or 12 bytes past a multiple of 16, for every form of the scoring kernels (fixed
    numbers of workers and any), the dense update, selection with and without the pass's histogram, both packs and the merge: the
    same bits as the oracle, and nothing written outside the arrays."""
    sizes = SEGMENTS["words_shared_by_long_tiles"] if segmented else [4096 * 5 + 1234]
    so, n = offsets(sizes), sum(sizes)
    ks, ms = [s // 9 for s in sizes], [s // 30 for s in sizes]
    rng = np.random.default_rng(10 * W + shift + segmented)
    guard = np.float32(123.0)

    def place(a):
        buf = torch.full((shift + n + 5,), float(guard), dtype=torch.float32, device=dev())
        buf[shift:shift + n] = torch.from_numpy(a)
        return buf, buf[shift:shift + n]
    w_h = rng.standard_normal(n).astype(np.float32)
    g_h = [(0.1 * rng.standard_normal(n)).astype(np.float32) for _ in range(W)]
    w_all, w = place(w_h)
    S_all, S = place(np.zeros(n, np.float32))
    g = [place(x)[1] for x in g_h]
    sd = binding.SlimDP(n, W, seg_off=so, seed=workloads.EXPLORE_SEED)
    sd.set_option("speculative_pack", 1)
    for t in range(2):                           # the second pass captures
        sd.score(w, g, 1.0, out=S)
        core, bits, off, epoch = sd.select_core(S, ks, reuse_histogram=True)
        again = sd.select_core(S, ks)[0]
        sd.score(w, g, 1.0, out=S)
        core, bits, off, epoch = sd.select_core(S, ks, reuse_histogram=True)
        idx, eoff = sd.sample_explore(bits, ks, t, ms, 0, W)
        kept = sd.pack(g, core, off, idx, eoff, epoch, updates_as_scored=True)
        plain = sd.pack(g, core, off, idx, eoff, epoch)
        sd.merge(w, 0.1, epoch, core, off, plain[0], idx, eoff, plain[1])
        sd.synchronize()
        S_o = oracle.score(w_h, g_h, 1.0)
        core_o = oracle.select_core(S_o, ks, so)
        assert np.array_equal(u32(S), S_o.view(np.uint32))
        assert np.array_equal(u32(core), core_o) and np.array_equal(u32(again), core_o)
        lists = [oracle.sample_explore(n, core_o, workloads.EXPLORE_SEED, t, q, ms, so) for q in range(W)]
        packs = [oracle.pack(g_h[q], core_o, lists[q]) for q in range(W)]
        for q in range(W):
            for got in (kept, plain):
                assert np.array_equal(u32(got[0][q]), packs[q][0].view(np.uint32)), (t, q)
                assert np.array_equal(u32(got[1][q]), packs[q][1].view(np.uint32)), (t, q)
        w_h = oracle.merge(w_h, 0.1, core_o, [x[0] for x in packs], lists, [x[1] for x in packs])
        assert np.array_equal(u32(w), w_h.view(np.uint32))
    w_h, S_o = oracle.dense_update_score(w_h, g_h, 0.1, 1.0)
    sd.dense_update_score(w, g, 0.1, 1.0, out=S)
    sd.synchronize()
    assert np.array_equal(u32(w), w_h.view(np.uint32)) and np.array_equal(u32(S), S_o.view(np.uint32))
    for buf in (w_all, S_all):
        outside = torch.cat([buf[:shift], buf[shift + n:]]).cpu().numpy()
        assert np.all(outside == guard)
    sd.close()


@pytest.mark.parametrize("n,W,segments,explore_async", [(60_001, 2, 1, 1), (60_001, 3, 5, 1), (60_001, 2, 1, 2), (60_001, 3, 5, 2),
                                                        (4096 * 545 + 3, 16, 1, 1), (4096 * 545 + 3, 16, 3, 1)])
def test_requests_of_changing_sizes_follow_each_other(n, W, segments, explore_async):
    """What one request leaves for the next (zones kept while the sizes stay, counters and the rerun flag cleared by their last
    reader), through changes of size, draws that miss their zones on either side, and announced draws; on the context's own stream
    (few tiles) and on the side stream."""
    so = offsets([n]) if segments == 1 else offsets([n // 3 + 1] + [n // 9] * (segments - 2) + [n - n // 3 - 1 - n // 9 * (segments - 2)])
    sizes = np.diff(so)
    ks = [int(s) // 10 for s in sizes]
    rng = np.random.default_rng(n + W)
    core = oracle.select_core(np.abs(rng.standard_normal(n)).astype(np.float32), ks, so)
    bits = to_dev(oracle.core_bits(n, core))
    sd = binding.SlimDP(n, W, seg_off=so, seed=workloads.EXPLORE_SEED)
    sd.set_option("explore_async", explore_async)
    sd.set_option("explore_hint_mode", 1)
    ts = sd.tile_starts().astype(np.int64)
    small, large = [int(s) // 50 for s in sizes], [int(s) // 9 for s in sizes]
    for it, (ms, miss, hint) in enumerate([(small, 0, 0), (small, 0, 1), (large, 0, 0), (small, 1, 0), (small, 0, 0), (small, 2, 1),
                                           (large, 2, 0), (large, 0, 1), (large, 0, 0)]):
        sd.set_option("explore_force_fallback", miss)
        if hint:
            sd.explore_hint(ks, it, ms, 0, W)
        idx, off = sd.sample_explore(bits, ks, it, ms, 0, W)
        sd.synchronize()
        for q in {0, W - 1}:
            want = oracle.sample_explore(n, core, workloads.EXPLORE_SEED, it, q, ms, so)
            assert np.array_equal(u32(idx[q]), want), (it, q)
            assert np.array_equal(u32(off[q]), np.searchsorted(want.astype(np.int64), ts).astype(np.uint32)), (it, q)
    sd.close()


@pytest.mark.parametrize("n,W,announced", [(64_000_003, 1, True), (64_000_003, 2, True), (16_000_001, 8, True), (30_000_003, 1, True),
                                           (30_000_003, 1, False), (8_000_003, 4, False), (4_500_003, 8, False)])
def test_request_for_a_core_that_stays_leaves_the_own_stream_free(n, W, announced):
    """Cached core keys and "explore_async" on: neither the draw, announced on the side stream or not, nor the request's chain
    stands in the context's own stream, from a moderate number of tiles on.  What stands in it is timed on the device
    (two events around announcement and request, behind a fill that hides the host's part) and compared with the same calls
    without "explore_async", for which the stream waits; the lists are the same."""
    k, m = len(range(5, n, 32)), n // 50
    sd = binding.SlimDP(n, W, seed=workloads.EXPLORE_SEED)
    sd.set_option("explore_hint_mode", 1)
    bits = torch.full(((n + 31) // 32,), 1 << 5, dtype=torch.int32, device=dev())     # every thirty-second parameter is in the core
    blocker = torch.empty(1 << 28, dtype=torch.float32, device=dev())
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    idx, off, took = {}, {}, {0: [], 1: []}
    for turn in range(8):
        for asyn in (0, 1):
            sd.set_option("explore_async", asyn)
            torch.cuda.synchronize()
            blocker.zero_()
            a.record()
            if announced:
                sd.explore_hint([k], turn, [m], 0, W)
            idx[asyn], off[asyn] = sd.sample_explore(bits, [k], turn, [m], 0, W, expl_idx=idx.get(asyn), expl_off=off.get(asyn))
            b.record()
            sd.synchronize()
            torch.cuda.synchronize()
            took[asyn].append(a.elapsed_time(b) * 1e3)
        for q in range(W):
            assert torch.equal(idx[0][q], idx[1][q]) and torch.equal(off[0][q], off[1][q]), (turn, q)
    sd.close()
    waits, free = min(took[0][2:]), min(took[1][2:])
    assert free < 0.5 * waits, "own stream held for %.0f us, %.0f without the option" % (free, waits)


@pytest.mark.parametrize("hint", [0, 1])
@pytest.mark.parametrize("name", ["flat", "words_shared_by_long_tiles", "wide zones"])
def test_more_requests_on_the_side_stream_than_the_context_has_notes_for(name, hint):
    """Seven requests in a row before any list is used (four are noted, the oldest makes room), into arrays of their own, some of
    them missing their zones; then their packs in another order, each right behind a new request into the arrays of the one
    packed before.  Every list and every pack as in the oracle."""
    sizes = SEGMENTS.get(name, [90_001])
    so, n, W, rounds = offsets(sizes), sum(sizes), 3, 7
    part = 2 if name == "wide zones" else 40
    ks, ms = [s // 10 for s in sizes], [s // part for s in sizes]
    rng = np.random.default_rng(len(name) + hint)
    core = oracle.select_core(np.abs(rng.standard_normal(n)).astype(np.float32), ks, so)
    g_h = [rng.standard_normal(n).astype(np.float32) for _ in range(W)]
    g, core_idx = [to_dev(x) for x in g_h], to_dev(core)
    sd = binding.SlimDP(n, W, seg_off=so, seed=workloads.EXPLORE_SEED)
    sd.set_option("explore_async", 2)
    sd.set_option("explore_hint_mode", 1)
    bits, off, epoch = sd.import_core(core_idx, ks)

    def request(it, lists=(None, None)):
        sd.set_option("explore_force_fallback", it % 3 if name != "wide zones" else 0)
        if hint:
            sd.explore_hint(ks, it, ms, 0, W)
        return sd.sample_explore(bits, ks, it, ms, 0, W, expl_idx=lists[0], expl_off=lists[1])

    def check(it, idx, expl_val):
        for q in range(W):
            want = oracle.sample_explore(n, core, workloads.EXPLORE_SEED, it, q, ms, so)
            assert np.array_equal(u32(idx[q]), want), (it, q)
            assert np.array_equal(u32(expl_val[q]), g_h[q][want].view(np.uint32)), (it, q)
    lists = [request(it) for it in range(rounds)]
    order = [6, 1, 4, 0, 5, 2, 3]
    held, kept = [], None
    for j, it in enumerate(order):
        if kept is not None:                     # new entries into the lists of the pack before: they are copied first
            held.append((order[j - 1], [x.clone() for x in lists[order[j - 1]][0]], kept))
            lists[order[j - 1]] = request(100 + order[j - 1], lists[order[j - 1]])
        kept = sd.pack(g, core_idx, off, *lists[it], epoch)[1]
    held.append((order[-1], lists[order[-1]][0], kept))
    sd.synchronize()
    for it, idx, expl_val in held:
        check(it, idx, expl_val)
    for it in order[:-1]:
        expl_val = sd.pack(g, core_idx, off, *lists[it], epoch)[1]
        sd.synchronize()
        check(100 + it, lists[it][0], expl_val)
    sd.close()


@pytest.mark.parametrize("segments,pct", [(1, 2), (3, 2), (1, 60), (5, 60)])
def test_exact_rerun_on_the_side_stream_is_waited_for(segments, pct):
    """A draw that misses its zones (on either side) on the side stream: the emission's small blocks redo the request, and the pack
    enqueued right behind it waits for them.  Ragged tiles and an empty segment's list, demands that most parameters meet, more
    workers than one group of the emission has."""
    W = 5
    n = 4096 * 66 + 77
    so = offsets([n]) if segments == 1 else offsets([4096 * 11 + 5] * (segments - 1) + [n - (4096 * 11 + 5) * (segments - 1)])
    sizes = np.diff(so)
    ks = [int(s) // 10 for s in sizes]
    ms = [(s - k) * pct // 100 if j != 1 else 0 for j, (s, k) in enumerate(zip((int(x) for x in sizes), ks))]
    rng = np.random.default_rng(segments * 100 + pct)
    core = oracle.select_core(np.abs(rng.standard_normal(n)).astype(np.float32), ks, so)
    g_h = [rng.standard_normal(n).astype(np.float32) for _ in range(2)]
    g = [to_dev(g_h[q & 1]) for q in range(W)]
    sd = binding.SlimDP(n, W, seg_off=so, seed=workloads.EXPLORE_SEED)
    sd.set_option("explore_async", 2)
    core_idx = to_dev(core)
    bits, off, epoch = sd.import_core(core_idx, ks)
    ts = sd.tile_starts().astype(np.int64)
    for miss in (1, 2):
        sd.set_option("explore_force_fallback", miss)
        idx, eoff = sd.sample_explore(bits, ks, miss, ms, 0, W)
        core_val, expl_val = sd.pack(g, core_idx, off, idx, eoff, epoch)
        sd.synchronize()
        for q in range(W):
            want = oracle.sample_explore(n, core, workloads.EXPLORE_SEED, miss, q, ms, so)
            assert np.array_equal(u32(idx[q]), want), (miss, q)
            assert np.array_equal(u32(eoff[q]), np.searchsorted(want.astype(np.int64), ts).astype(np.uint32)), (miss, q)
            assert np.array_equal(u32(expl_val[q]), g_h[q & 1][want].view(np.uint32)), (miss, q)
            assert np.array_equal(u32(core_val[q]), g_h[q & 1][core].view(np.uint32)), (miss, q)
    sd.close()


def test_recorded_request_replays_beside_eager_ones():
    """A replay finds counters, zones and the rerun flag as it needs them, whatever eager requests (other sizes, a missed draw)
    ran since it was recorded, and so do eager requests after a replay."""
    n, W = 60_001, 2
    k, m, other = n // 10, n // 50, n // 9
    rng = np.random.default_rng(3)
    core = oracle.select_core(np.abs(rng.standard_normal(n)).astype(np.float32), k)
    bits = to_dev(oracle.core_bits(n, core))
    want = [oracle.sample_explore(n, core, workloads.EXPLORE_SEED, 1, q, m) for q in range(W)]
    want_other = [oracle.sample_explore(n, core, workloads.EXPLORE_SEED, 2, q, other) for q in range(W)]
    st = torch.cuda.Stream()
    sd = binding.SlimDP(n, W, seed=workloads.EXPLORE_SEED, stream=st)
    idx = [torch.empty(m, dtype=torch.int32, device=dev()) for _ in range(W)]
    off = [torch.empty(sd.T + 1, dtype=torch.int32, device=dev()) for _ in range(W)]
    torch.cuda.synchronize()
    with torch.cuda.stream(st):
        sd.sample_explore(bits, [k], 2, [other], 0, W)
    sd.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        sd.sample_explore(bits, [k], 1, [m], 0, W, expl_idx=idx, expl_off=off)
    for turn in range(4):
        with torch.cuda.stream(st):
            if turn:
                sd.set_option("explore_force_fallback", turn - 1)
                got, _ = sd.sample_explore(bits, [k], 2, [other], 0, W)
                sd.synchronize()
                assert all(np.array_equal(u32(got[q]), want_other[q]) for q in range(W)), turn
            for x in idx:
                x.zero_()
            graph.replay()
        sd.synchronize()
        assert all(np.array_equal(u32(idx[q]), want[q]) for q in range(W)), turn
    sd.close()


@pytest.mark.parametrize("per_tile_tail", [0, 1])
@pytest.mark.parametrize("W", [1, 5, 9])
@pytest.mark.parametrize("name", sorted(SEGMENTS) + ["one_segment", "more_blocks_than_run_at_a_time"])
def test_explorer_lists_and_offsets_at_the_edges_of_segments_and_zones(name, W, per_tile_tail):
    """Requests from nothing to everything outside the core (no sure zone, no candidates wanted, every candidate wanted), in both
    formats of the draw, over segments that share waves, blocks and bitmap words."""
    sizes = SEGMENTS.get(name) or ([300_001] if name == "one_segment" else [4096 + 7, 900] * 130)
    so, n = offsets(sizes), sum(sizes)
    rng = np.random.default_rng(len(name))
    ks = [0 if j % 4 == 3 else s // 7 for j, s in enumerate(sizes)]
    core = oracle.select_core(np.abs(rng.standard_normal(n)).astype(np.float32), ks, so)
    bits = to_dev(oracle.core_bits(n, core))
    sd = binding.SlimDP(n, W, seg_off=so, seed=workloads.EXPLORE_SEED)
    sd.set_option("explore_per_tile_tail", per_tile_tail)
    ts = sd.tile_starts().astype(np.int64)
    left = [s - k for s, k in zip(sizes, ks)]
    requests = {
        "few": [a // 50 for a in left],
        "nothing in some": [0 if j % 3 == 1 else a // 3 for j, a in enumerate(left)],
        "all but one": [max(a - 1, 0) for a in left],
        "all": left,
        "most": [a - a // 30 for a in left],
    }
    for it, (what, ms) in enumerate(requests.items()):
        idx, off = sd.sample_explore(bits, ks, it, ms, 3, W)
        sd.synchronize()
        for q in {0, W - 1}:
            want = oracle.sample_explore(n, core, workloads.EXPLORE_SEED, it, 3 + q, ms, so)
            assert np.array_equal(u32(idx[q]), want), what
            assert np.array_equal(u32(off[q]), np.searchsorted(want.astype(np.int64), ts).astype(np.uint32)), what
    sd.close()


@pytest.mark.parametrize("chosen", [1023, 1024, 1025, 2048, 4095, 4096])
def test_emission_of_tiles_that_hold_few_and_many(chosen):
    """Core and explorer lists of tiles at the edge between the two ways of writing them, up to every parameter of a tile, beside
    tiles that hold next to nothing, and a ragged tile that is taken whole."""
    T, tail = 5, 777
    n = T * 4096 + tail
    rng = np.random.default_rng(chosen)
    score = rng.random(n).astype(np.float32) * 0.5
    for t in (0, 3):                             # these tiles hold `chosen` of the core each, the ragged one all it has
        score[t * 4096 + rng.choice(4096, chosen, replace=False)] += 1.0
    score[T * 4096:] += 1.0
    k = 2 * chosen + tail
    sd = binding.SlimDP(n, 2, seed=workloads.EXPLORE_SEED)
    ts = sd.tile_starts().astype(np.int64)
    idx, bits, off, _ = sd.select_core(to_dev(score), [k])
    want = oracle.select_core(score, k)
    m = (n - k) * chosen // 4096                  # about as dense in the tiles without a core, everything at last
    eidx, eoff = sd.sample_explore(bits, [k], 3, [m], 0, 2)
    sd.synchronize()
    assert np.array_equal(u32(idx), want)
    assert np.array_equal(u32(off), np.searchsorted(want.astype(np.int64), ts).astype(np.uint32))
    for q in range(2):
        e = oracle.sample_explore(n, want, workloads.EXPLORE_SEED, 3, q, m)
        assert np.array_equal(u32(eidx[q]), e)
        assert np.array_equal(u32(eoff[q]), np.searchsorted(e.astype(np.int64), ts).astype(np.uint32))
    sd.close()


@pytest.mark.parametrize("overlap", [False, True])
@pytest.mark.parametrize("W,pct", [(1, 2), (3, 17), (8, 6), (8, 11), (9, 10), (16, 17), (32, 3)])
def test_merge_variants_by_explorer_density(W, pct, overlap):
    """Entries per tile for 4, 8 and 16 registers a thread and for the staged path, most positions sent by several workers; with
    overlap the lists also meet the core, whose sum then comes first."""
    check_merge(4096 * 6 + 1111, W, pct, overlap)


@pytest.mark.parametrize("pct", [26, 30])
def test_merge_variants_over_more_tiles_than_run_in_two_turns(pct):
    """About 1,920 and 2,210 entries a tile: tiles on both sides of what eight registers a thread hold, and none of them."""
    check_merge(4096 * 2100 + 5, 2, pct, False)


def check_merge(n, W, pct, overlap):
    rng = np.random.default_rng(W * 100 + pct)
    w_h = rng.standard_normal(n).astype(np.float32)
    core = oracle.select_core(np.abs(rng.standard_normal(n)).astype(np.float32), n // 10)
    sd = binding.SlimDP(n, W)
    ts = sd.tile_starts().astype(np.int64)
    bits, off = torch.empty((n + 31) // 32, dtype=torch.int32, device=dev()), torch.empty(sd.T + 1, dtype=torch.int32, device=dev())
    _, off, epoch = sd.import_core(to_dev(core), [len(core)], bits, off)
    pool = np.arange(n) if overlap else np.setdiff1d(np.arange(n), core)
    m = len(pool) * pct // 100
    idx = [np.sort(rng.choice(pool, m, replace=False)).astype(np.uint32) for _ in range(W)]
    val = [(rng.standard_normal(m) * 10.0 ** rng.integers(-3, 4, m)).astype(np.float32) for _ in range(W)]
    core_val = [(rng.standard_normal(len(core)) * 10.0 ** rng.integers(-3, 4, len(core))).astype(np.float32) for _ in range(W)]
    w = to_dev(w_h)
    sd.merge(w, 0.1, epoch, to_dev(core), off, [to_dev(x) for x in core_val], [to_dev(x) for x in idx],
             [to_dev(np.searchsorted(x.astype(np.int64), ts).astype(np.uint32)) for x in idx], [to_dev(x) for x in val])
    sd.synchronize()
    # the interface's order: +0, the core values in worker order, then the explorer values in worker order, one fused step
    acc, sent = np.zeros(n, np.float32), np.zeros(n, bool)
    for v in core_val:
        acc[core] = acc[core] + v
    sent[core] = True
    for i, v in zip(idx, val):
        acc[i] = acc[i] + v
        sent[i] = True
    exact = w_h.astype(np.longdouble) - np.longdouble(np.float32(0.1)) * acc.astype(np.longdouble)     # 64 bits hold the product; one rounding
    want = np.where(sent, exact.astype(np.float32), w_h)
    assert np.array_equal(u32(w), want.view(np.uint32))
    sd.close()


@pytest.mark.parametrize("exponent", [-140, -126, -81, -80, -79, -41, -40, -39, 0, 39, 40, 41, 120])
def test_quantisation_on_both_sides_of_the_range_of_the_common_reciprocal(exponent):
    """Buckets whose largest, or smallest, magnitude lies at the edges inside which quotients come from the bucket's
    reciprocal; zeros among them, and a ragged last bucket.  Values are finite by the interface: of a bucket that holds an
    infinity the scale alone is compared."""
    n, per = 512 * 24 + 77, 512
    rng = np.random.default_rng(1000 + exponent)
    buckets = []
    for j in range(25):
        x = rng.standard_normal(per) * rng.choice([1.0, 2.0 ** -23, 2.0 ** -60], per)
        top = np.ldexp(1.0 + rng.random(), exponent)
        x = x / np.abs(x).max() * top
        if j % 3 == 1:                           # the other end: a small value in a bucket of usual size
            x = rng.standard_normal(per)
            x[rng.integers(per)] = np.ldexp(1.0 + rng.random(), min(exponent, 0))
        if j % 5 == 2:
            x[rng.integers(per, size=9)] = 0.0
        if j % 8 == 3:
            x[rng.integers(per)] = np.inf
        buckets.append(x)
    with np.errstate(over="ignore"):
        v = np.concatenate(buckets)[:n].astype(np.float32)
    sd = binding.SlimDP(n, 1, seed=5)
    code, scale = sd.quantize([to_dev(v)], 0, 7)
    sd.synchronize()
    code_o, scale_o = oracle.quantize(v, 5, 7, 0, 0)
    assert np.array_equal(u32(scale[0]), scale_o.view(np.uint32))
    finite = np.repeat(np.isfinite(scale_o), per)[:n]
    assert np.array_equal(code[0].cpu().numpy()[finite], code_o[finite])
    sd.close()


@pytest.mark.parametrize("sizes", [[4096 * 3 + 5], [4096 * 256], [4096 + 7, 33, 9000], [4096 * 2, 5]])
@pytest.mark.parametrize("W", [1, 3, 5])
def test_worker_side_with_several_workers_to_a_block_and_few(sizes, W):
    """Local step with extraction, a pull whose values leave with the overwrite (one worker has no local model), and the pull
    with a local step, with one, some and all workers to a block."""
    so, n = offsets(sizes), sum(sizes)
    rng = np.random.default_rng(n + W)
    ks = [s // 9 for s in sizes]
    sd = binding.SlimDP(n, W, seg_off=so, seed=workloads.EXPLORE_SEED)
    core, bits, off, epoch = sd.select_core(to_dev(np.abs(rng.standard_normal(n)).astype(np.float32)), ks)
    for it, pct in enumerate((2, 40)):           # few explorers, and more than a block holds at a time
        ms = [(s - k) * pct // 100 for s, k in zip(sizes, ks)]
        idx, eoff = sd.sample_explore(bits, ks, it, ms, 0, W)
        new = lambda: [rng.standard_normal(n).astype(np.float32) for _ in range(W)]
        w_h, l_h, g_h, d_h = rng.standard_normal(n).astype(np.float32), new(), new(), new()
        w, l, g, d = to_dev(w_h), [to_dev(x) for x in l_h], [to_dev(x) for x in g_h], [to_dev(x) for x in d_h]
        sets = (core, off, idx, eoff)
        cv, ev = sd.local_step_pack(l, g, d, 0.25, False, *sets, epoch)
        c = u32(core)
        for q in range(W):
            l_h[q], d_h[q] = oracle.local_step(l_h[q], d_h[q], g_h[q], 0.25)
            assert np.array_equal(u32(l[q]), l_h[q].view(np.uint32)) and np.array_equal(u32(d[q]), d_h[q].view(np.uint32))
            assert np.array_equal(u32(cv[q]), d_h[q][c].view(np.uint32))
            assert np.array_equal(u32(ev[q]), d_h[q][u32(idx[q])].view(np.uint32))
        co, eo = sd.pull(w, epoch, *sets, w_local=[None if (q == 1) else l[q] for q in range(W)])
        sd.synchronize()
        for q in range(W):
            e = u32(idx[q])
            assert np.array_equal(u32(co[q]), w_h[c].view(np.uint32)) and np.array_equal(u32(eo[q]), w_h[e].view(np.uint32))
            if q != 1:
                l_h[q][c] = w_h[c]
                l_h[q][e] = w_h[e]
            assert np.array_equal(u32(l[q]), l_h[q].view(np.uint32)), q
        sd.pull_local_step(w, epoch, *sets, l, g, d, 0.5, first=True)
        sd.synchronize()
        for q in range(W):
            l_h[q][c] = w_h[c]
            l_h[q][u32(idx[q])] = w_h[u32(idx[q])]
            l_h[q], d_h[q] = oracle.local_step(l_h[q], None, g_h[q], 0.5)
            assert np.array_equal(u32(l[q]), l_h[q].view(np.uint32)) and np.array_equal(u32(d[q]), d_h[q].view(np.uint32))
    sd.close()
