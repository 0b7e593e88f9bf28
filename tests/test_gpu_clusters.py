"""Several workgroups per utterance: the oracle's results whatever their number, on the graphs where
their sharing can go wrong (keys that tie, hub states, closure rounds larger than a table, more
destinations than registers and tables hold, options, boosting), and on one channel that changes hands."""
import numpy as np
import pytest

import test_gpu_parity as parity
from test_gpu_parity import c2_refs, torch_cuda  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.fixture
def cluster(request, monkeypatch):
    """Every decoder made in the test gives each utterance this many workgroups."""
    import paper_2311_04996_amd as package

    class ClusterDecoder(package.Decoder):
        def __init__(self, *a, **kw):
            super().__init__(*a, **kw)
            self.debug_set_cluster_size(request.param)
    monkeypatch.setattr(package, "Decoder", ClusterDecoder)
    return request.param


@pytest.mark.parametrize("cluster", [1, 2, 4, 8], indirect=True)
def test_small_and_tie_heavy_graphs(torch_cuda, cluster):
    parity.test_micro_graphs_with_ties_and_negative_epsilon(torch_cuda)
    parity.test_boost_fst_on_micro_graphs(torch_cuda)
    parity.test_self_loop_candidates_that_tie_exactly_with_candidates_of_other_arcs(torch_cuda)
    parity.test_random_small_configurations(torch_cuda)
    parity.test_dead_and_nonfinal_and_minus_inf(torch_cuda)


@pytest.mark.parametrize("cluster", [1, 2, 4, 8], indirect=True)
def test_hubs_large_closures_and_many_duplicates(torch_cuda, cluster):
    parity.test_more_high_degree_states_than_the_shared_list_holds(torch_cuda)
    parity.test_state_with_more_than_a_million_arcs(torch_cuda)
    parity.test_epsilon_rounds_larger_than_one_chunk_and_one_table(torch_cuda)


@pytest.mark.parametrize("cluster", [2, 8], indirect=True)
def test_options_and_streams(torch_cuda, c1, c2, c2_refs, cluster):
    parity.test_boost_fst_with_frequent_long_matches(torch_cuda, c2)
    parity.test_cost_offsets_match_the_oracle_with_the_same_option(torch_cuda, c1, c2)
    parity.test_advance_and_partial_in_one_launch(torch_cuda, c2)
    parity.test_lattice_arena_overflow_in_a_batch_does_not_touch_the_neighbours(torch_cuda, c2)
    parity.test_recycled_lattice_stream_ten_times_the_window(torch_cuda, c2)


def _same_results(dec, out, refs):
    words, nwords, cost, flags = (t.cpu().numpy() for t in out)
    for b, r in enumerate(refs):
        assert words[b, :nwords[b]].tolist() == r.words.tolist() and int(flags[b]) == r.flags and cost[b] == np.float32(r.cost), b
    assert dec.get_counters()[:7].tolist() == np.sum([r.counters for r in refs], axis=0)[:7].tolist()


def _candidates(g, ll, length, beam, max_active):
    """Per frame, the arcs out of the oracle's token set that end inside the beam, without the usual self-loops: at least
    as many are a workgroup's candidates (while the frame's best cost is not known yet, it lets more in)."""
    from oracle import Oracle
    deg, row = np.diff(g.row_offsets), g.row_offsets
    src = np.repeat(np.arange(g.num_states), deg)
    has_eps = np.zeros(g.num_states, bool)
    has_eps[src[g.ilabel == 0]] = True
    first = np.zeros(len(src), bool)
    first[row[:-1][deg > 0]] = True
    loop = first & (g.next_state == src) & (g.olabel == 0) & ~has_eps[src]
    kinds, which = np.unique(np.stack([g.ilabel[loop], g.weight[loop].view(np.int32)]), axis=1, return_inverse=True)
    usual = np.zeros(len(src), bool)
    usual[np.nonzero(loop)[0]] = which.ravel() == np.argmax(np.bincount(which.ravel()))
    n = []
    frames = Oracle(g).decode(ll, length=length, beam=beam, max_active=max_active, want_frames=True).frames
    for t, (states, costs) in enumerate(frames[:length]):
        d = deg[states]
        arcs = np.repeat(row[states] - np.cumsum(d) + d, d) + np.arange(d.sum())
        emit = g.ilabel[arcs] > 0
        arcs, cost = arcs[emit], np.repeat(costs, d)[emit]
        cost = cost + g.weight[arcs] - ll[t, g.ilabel[arcs] - 1]
        n.append(int(((cost - cost.min() <= beam) & ~usual[arcs]).sum()))
    return n


@pytest.mark.parametrize("cluster", [1], indirect=True)
@pytest.mark.parametrize("ma", [5000, 5001, 12000, 12001])
def test_either_side_of_the_sizes_one_workgroup_of_the_cluster_kernel_takes(torch_cuda, c2, cluster, ma):
    """No option on and no boosting, as the rule asks: results and counters on both sides of its ends, with a workgroup per
    utterance and with fewer, twice on one decoder.  The frames have more candidates than registers hold (3,072) and than
    one pass takes (6,144), and with the larger sets more than four regions' notes hold (11,264 each)."""
    from paper_2311_04996_amd import Decoder
    ll, lengths = np.ascontiguousarray(c2.loglikes[:4, :40]), np.array([40, 33, 40, 1], np.int32)
    refs = parity.oracle_batch(c2.graph, ll, lengths, 20.0, ma)
    n = _candidates(c2.graph, ll[0], 40, 20.0, ma)
    assert min(n) > 6144 and max(n) > (4 * 11264 if ma > 5001 else 2 * 11264)
    dec = Decoder(c2.graph, max_channels=4, max_frames=40, max_active_hint=ma)
    dev = torch_cuda.from_numpy(ll).cuda()
    for n_wg in (0, 2):
        dec.set_launch_workgroups(n_wg)
        dec.get_counters(reset=True)
        out = dec.decode_batch(dev, lengths, 20.0, ma)
        assert dec.debug_last_launch()[1] == 1 and dec.debug_last_kernel() == (2 if ma <= 12000 else 1)
        _same_results(dec, out, refs)
    dec.close()


@pytest.mark.parametrize("cluster", [1], indirect=True)
def test_the_kernel_of_a_launch_with_one_workgroup_per_utterance(torch_cuda, c2, cluster):
    """Up to a max-active of 5,000 the cluster kernel; up to 12,000 whole utterances without boosting and options on graphs
    of which half the states or more have the usual self-loop alone; the first kernel for the rest and for narrow records."""
    from paper_2311_04996_amd import Decoder
    from workloads.boost import boost_fsts
    from workloads.configs import boost_tables
    from workloads.graphs import _csr
    T = 3
    dev = torch_cuda.from_numpy(np.ascontiguousarray(c2.loglikes[:2, :T])).cuda()
    words, fsts = boost_tables(3, 2, 20_000), boost_fsts(3, 2, 20_000, per_utt=20)

    def kernels(g, dev, max_actives, options=None, boost=None, stream=False):
        got = []
        dec = Decoder(g, max_channels=2, max_frames=T, max_active_hint=4000, **(options or {}))
        for ma in max_actives:
            if stream:
                dec.init_channels([0, 1], 17.0, ma)
                dec.advance_chunk_partial([0, 1], dev, [T, T], finalize=True)
            else:
                dec.decode_batch(dev, [T, T], 17.0, ma, **(boost or {}))
            assert dec.debug_last_launch()[1] == 1
            got.append(dec.debug_last_kernel())
        dec.close()
        return got
    assert kernels(c2.graph, dev, (1000, 5000, 5001, 12000, 12001)) == [2, 2, 2, 2, 1]
    for kw in (dict(boost=dict(boosts=words)), dict(boost=dict(boost_fsts=fsts)), dict(stream=True),
               dict(options=dict(record_digests=True)), dict(options=dict(cost_offset=True)),
               dict(options=dict(keep_token_records=True)), dict(options=dict(recycle_lattice=True, lattice_bytes_per_channel=1 << 20))):
        assert kernels(c2.graph, dev, (5000, 5001), **kw) == [2, 1], kw
    assert kernels(c2.graph, dev, (1000, 5001), options=dict(narrow_arcs=True)) == [1, 1]
    for n_simple, want in ((4000, 2), (3999, 1)):          # of 8,000 states
        s = np.arange(8000)
        more = s[n_simple:]
        g = _csr(8000, n_simple, 129, np.concatenate([s, more]), np.concatenate([s, (more + 1) % 8000]),
                 np.concatenate([np.ones(8000, np.int64), 2 + more % 100]), np.zeros(8000 + len(more), np.int64), np.zeros(8000 + len(more)))
        assert kernels(g, dev, (5001,)) == [want]
        assert kernels(g, dev, (5000,)) == [2]


def test_a_stream_whose_chunks_are_decoded_by_different_numbers_of_workgroups(torch_cuda, c2, c2_refs):
    from paper_2311_04996_amd import Decoder
    b = int(np.argmax(c2.lengths))
    n = min(int(c2.lengths[b]), 200)
    dec = Decoder(c2.graph, max_channels=1, max_frames=n, max_active_hint=c2.max_active, record_digests=True)
    ll = torch_cuda.from_numpy(np.ascontiguousarray(c2.loglikes[b:b + 1, :n])).cuda()
    dec.init_channel(0, c2.beam, c2.max_active)
    for k, t in enumerate(range(0, n, 8)):
        dec.debug_set_cluster_size((8, 1, 2, 4, 1, 8)[k % 6])
        dec.advance_chunk([0], ll[:, t:t + 8].contiguous(), [min(8, n - t)])
    cnt, dig = dec.debug_frame_digests(0)
    assert (cnt == c2_refs[b].digest_count[:n + 1]).all() and (dig == c2_refs[b].digest_sum[:n + 1]).all()
    dec.close()


def test_calls_with_many_entries_that_have_nothing_to_do(torch_cuda, c2, c2_refs):
    """Entries without a frame have no exchange but the one that hands them out: the workgroups of
    a cluster go through a row of them, and then decode on as if they had not been there."""
    from paper_2311_04996_amd import Decoder
    n_ch, n = 96, 48
    b = int(np.argmax(c2.lengths))
    dec = Decoder(c2.graph, max_channels=n_ch, max_frames=n, max_active_hint=c2.max_active, record_digests=True)
    dec.debug_set_cluster_size(8)
    dec.set_launch_workgroups(64)                 # eight clusters take them all, a run of empty ones each
    dec.init_channels(list(range(n_ch)), c2.beam, c2.max_active)
    ll = torch_cuda.from_numpy(np.ascontiguousarray(c2.loglikes[b:b + 1, :n])).cuda()
    busy = (0, 41, 95)
    for t in range(0, n, 8):
        rows = ll[:, t:t + 8].expand(n_ch, -1, -1).contiguous()
        dec.advance_chunk(list(range(n_ch)), rows, [8 if ch in busy else 0 for ch in range(n_ch)])
    for ch in busy:
        cnt, dig = dec.debug_frame_digests(ch)
        assert (cnt[:n + 1] == c2_refs[b].digest_count[:n + 1]).all() and (dig[:n + 1] == c2_refs[b].digest_sum[:n + 1]).all()
    dec.close()


def test_memory_of_the_clusters_is_given_back_as_calls_grow(torch_cuda, c2, c2_refs):
    """Calls of growing size: the decoder's memory stays within twice what the largest call alone takes."""
    from paper_2311_04996_amd import Decoder
    b = int(np.argmax(c2.lengths))
    ll = torch_cuda.from_numpy(np.ascontiguousarray(c2.loglikes[b:b + 1, :16])).cuda()
    held = []
    for sizes in ((24,), (1, 2, 3, 5, 8, 12, 16, 20, 24)):
        dec = Decoder(c2.graph, max_channels=24, max_frames=16, max_active_hint=c2.max_active, record_digests=True)
        dec.debug_set_cluster_size(8)
        start = dec.device_bytes()
        for n in sizes:
            dec.init_channels(list(range(n)), c2.beam, c2.max_active)
            dec.advance_chunk(list(range(n)), ll.expand(n, -1, -1).contiguous(), [16] * n)
            cnt, dig = dec.debug_frame_digests(n - 1)
            assert (cnt[:17] == c2_refs[b].digest_count[:17]).all() and (dig[:17] == c2_refs[b].digest_sum[:17]).all()
        held.append(dec.device_bytes() - start)
        dec.close()
    assert 0 < held[0] and held[1] <= 2 * held[0]


def _closure_overflow_graph(middle_first):
    """Start -> 6,000 dead ends and a hub, all over label 1, or one state over label 2.  The hub reaches 4,000
    states over epsilon arcs in one closure round, and 2,000 of them a second time, at the same cost, in the
    next one over eight states in the middle, whose arc ids are lower than the hub's or higher."""
    from workloads.graphs import _csr
    n_dead, n_z, n_mid = 6000, 4000, 8
    mid0 = 1 if middle_first else 2
    hub = 1 + n_mid if middle_first else 1
    one, z0 = 2 + n_mid, 3 + n_mid
    dead0 = z0 + n_z
    S = dead0 + n_dead
    src, dst, il = [], [], []

    def arcs(s, d, label):
        src.extend([s] * len(d)), dst.extend(d), il.extend([label] * len(d))
    arcs(0, list(range(dead0, S)) + [hub], 1)
    arcs(0, [one], 2)
    arcs(hub, list(range(z0, z0 + n_z)) + list(range(mid0, mid0 + n_mid)), 0)
    for k in range(n_mid):
        arcs(mid0 + k, list(range(z0 + 250 * k, z0 + 250 * (k + 1))), 0)
    n = len(src)
    return _csr(S, 0, 2, np.array(src), np.array(dst), np.array(il), np.zeros(n, np.int64), np.zeros(n))


@pytest.mark.parametrize("cluster", [1, 2, 4, 8], indirect=True)
def test_a_closure_that_runs_out_of_room_ends_there(torch_cuda, cluster):
    """10,009 tokens, 8,192 places: the channel is flagged and stops.  What the next closure round would
    compare its exact ties with, the candidates of tokens that found no room, is gone by then."""
    from paper_2311_04996_amd import Decoder, FLAG_CAPACITY, FLAG_DEAD
    for middle_first in (False, True):
        g = _closure_overflow_graph(middle_first)
        dec = Decoder(g, max_channels=2, max_frames=2, max_active_hint=1000, lattice_bytes_per_channel=1 << 18,
                      record_digests=True)
        both = np.zeros((2, 2, 2), np.float32)
        both[1, :, 0] = -1000.0                      # the second utterance keeps to the one state
        lengths = np.array([1, 1], np.int32)
        _, nwords, cost, flags = dec.decode_batch(torch_cuda.from_numpy(both).cuda(), lengths, 5.0, 5000)
        torch_cuda.cuda.synchronize()
        assert flags.tolist()[0] & (FLAG_CAPACITY | FLAG_DEAD) == FLAG_CAPACITY | FLAG_DEAD and int(nwords[0]) == 0
        (ref,) = parity.oracle_batch(g, both[1:], lengths[1:], 5.0, 5000)
        cnt, dig = dec.debug_frame_digests(1)
        assert int(flags[1]) == ref.flags and float(cost[1]) == ref.cost
        assert (cnt == ref.digest_count).all() and (dig == ref.digest_sum).all()
        dec.close()
        # with room for all of them the ties are decided as the oracle decides them
        parity.check_batch(torch_cuda, g, both, lengths, 5.0, 5000, max_active_hint=10000)


def test_clusters_smaller_than_planned(torch_cuda, c1, c2, c2_refs, monkeypatch):
    """The first workgroup of a cluster goes on with those that have started; if it waits for none, clusters of
    every size below the planned one come up."""
    import paper_2311_04996_amd as package

    class Impatient(package.Decoder):
        def __init__(self, *a, **kw):
            super().__init__(*a, **kw)
            self.debug_set_cluster_size(8)
            self.debug_set_cluster_waits(start_ticks=self.ticks)
    monkeypatch.setattr(package, "Decoder", Impatient)
    for Impatient.ticks in (0, 20, 60):                 # 10 ns each
        parity.check_batch(torch_cuda, c2.graph, c2.loglikes, c2.lengths, c2.beam, c2.max_active, refs=c2_refs)
        parity.test_random_small_configurations(torch_cuda)
        parity.test_boost_fst_with_frequent_long_matches(torch_cuda, c2)
    parity.test_candidate_overflow_is_reported_not_fatal(torch_cuda, c2)


@pytest.mark.parametrize("polls", [0, 5, 13, 21, 34, 60, 100, 300])
def test_no_utterance_is_lost_when_clusters_break_up(torch_cuda, c2, polls):
    """Waits that end after a few looks: clusters break up in any of their exchanges.  Every entry of the list
    still has the oracle's result, or is reported as stopped; so is a stream; and the next call is as if
    nothing had been."""
    from paper_2311_04996_amd import Decoder, FLAG_CAPACITY, FLAG_DEAD
    lost = FLAG_CAPACITY | FLAG_DEAD
    B, T = 72, 24                                      # more than the 32 clusters there are of 8
    ll = np.ascontiguousarray(np.concatenate([c2.loglikes[:24, 4 * k:4 * k + T] for k in range(3)]))
    lengths = (T - np.arange(B) % 7).astype(np.int32)
    refs = parity.oracle_batch(c2.graph, ll, lengths, c2.beam, c2.max_active)
    dev = torch_cuda.from_numpy(ll).cuda()
    dec = Decoder(c2.graph, max_channels=B, max_frames=T, max_active_hint=c2.max_active)

    def decode():
        out = dec.decode_batch(dev, lengths, c2.beam, c2.max_active)
        torch_cuda.cuda.synchronize()
        words, nwords, cost, flags = (t.cpu().numpy() for t in out)
        stopped = 0
        for b, r in enumerate(refs):
            if flags[b] & lost:
                assert flags[b] == lost and nwords[b] == 0 and np.isinf(cost[b])
                stopped += 1
            else:
                assert flags[b] == r.flags and cost[b] == np.float32(r.cost) and words[b, :nwords[b]].tolist() == r.words.tolist()
        return stopped

    dec.debug_set_cluster_size(8)
    for size in (8, 2):
        dec.debug_set_cluster_size(size)
        dec.debug_set_cluster_waits(polls=polls)
        stopped = decode()
        print(f"polls {polls}, {size} workgroups: {stopped} of {B} stopped", flush=True)
        assert stopped > 0 or polls > 0                # (a word takes longer than one look)
        dec.debug_set_cluster_waits()
        assert decode() == 0
    dec.init_channels(list(range(B)), c2.beam, c2.max_active)
    dec.debug_set_cluster_waits(polls=polls)
    dec.advance_chunk(list(range(B)), dev, lengths)
    dec.debug_set_cluster_waits()
    for b, r in enumerate(refs):
        words, cost, flags = dec.get_partial(b, finalize=True)
        if flags & lost:
            assert flags == lost and len(words) == 0 and np.isinf(cost)
        else:
            assert flags == r.flags and cost == np.float32(r.cost) and words.tolist() == r.words.tolist()
    assert decode() == 0
    dec.close()


@pytest.mark.parametrize("cluster", [2, 4, 8], indirect=True)
@pytest.mark.parametrize("sample", [0, 4096])
def test_a_sample_of_the_candidates_never_stops_a_channel(torch_cuda, cluster, sample):
    """Some 76,000 candidates per frame: their bins are estimated from a sample, where one run of 64 can stand for
    all of a workgroup's; whether they fit the buffer is counted."""
    from workloads import ctc_loglikes, tlg_shaped_graph
    g = tlg_shaped_graph(31, 200_000, 1_400_000, num_classes=129, alpha=1.8, k_max=5000, p_eps=0.2,
                         num_words=50_000, extra_lo=3, extra_hi=5)
    lengths = np.array([40, 33, 21], np.int32)
    ll = ctc_loglikes(31, lengths, 40, 129, sigma=2.0, p_blank=0.3, blank_boost=6.0, token_boost=4.0)
    refs = parity.check_batch(torch_cuda, g, ll, lengths, 25.0, 10000, max_active_hint=10000, selection_sample=sample,
                              lattice_bytes_per_channel=1 << 23)
    assert sum(int(r.counters[7]) for r in refs) > 6144 * cluster * int(lengths.sum())   # the sample is taken


@pytest.mark.parametrize("cluster", [1, 2, 4, 8], indirect=True)
def test_the_candidate_capacity_is_the_same_for_every_number_of_workgroups(torch_cuda, cluster):
    """Candidates all inside the beam, in four regions by the top bits of the key's hash: 1,024 in the fullest fit a
    capacity of 4,096, one more does not."""
    from paper_2311_04996_amd import Decoder, FLAG_CAPACITY, FLAG_DEAD
    from workloads.graphs import _csr

    def fullest(n):                                    # states 1..n without arcs follow the start state's n arcs
        first = (1 + n + 1) // 2
        key = (first + np.arange(n)).astype(np.uint64)
        return int(np.bincount((key * 0x9E3779B1 & 0xFFFFFFFF).astype(np.int64) >> 30, minlength=4).max())
    fits = max(n for n in range(3800, 4097) if fullest(n) == 1024)
    for n, fit in ((fits, True), (min(k for k in range(fits, 4200) if fullest(k) == 1025), False)):
        g = _csr(n + 1, 0, 2, np.zeros(n), np.arange(1, n + 1), np.ones(n), np.zeros(n), np.zeros(n))
        ll = np.zeros((1, 1, 2), np.float32)
        dec = Decoder(g, max_channels=1, max_frames=1, max_active_hint=1000, candidate_capacity=4096,
                      lattice_bytes_per_channel=1 << 18, record_digests=True)
        _, nwords, cost, flags = dec.decode_batch(torch_cuda.from_numpy(ll).cuda(), np.array([1], np.int32), 5.0, 5000)
        (ref,) = parity.oracle_batch(g, ll, [1], 5.0, 5000)
        if fit:
            cnt, dig = dec.debug_frame_digests(0)
            assert int(flags[0]) == ref.flags and (cnt == ref.digest_count).all() and (dig == ref.digest_sum).all()
        else:
            assert int(flags[0]) == FLAG_CAPACITY | FLAG_DEAD and int(nwords[0]) == 0
        dec.close()


@pytest.mark.parametrize("capacity,size", [(1 << 27, 8), ((1 << 27) + 4, 4)])
def test_clusters_have_as_many_workgroups_as_32_bits_number_candidates_of(torch_cuda, c2, capacity, size):
    """2 * 8 * 8 segments of a quarter of the capacity each are 2^32 records at 2^27, the last of them in the last segment; with
    more, eight workgroups become four."""
    from paper_2311_04996_amd import Decoder
    n = 24
    b = int(np.argmax(c2.lengths))
    rows = np.ascontiguousarray(c2.loglikes[b:b + 1, :n])
    (ref,) = parity.oracle_batch(c2.graph, rows, [n], c2.beam, c2.max_active)
    dec = Decoder(c2.graph, max_channels=1, max_frames=n, max_active_hint=c2.max_active, candidate_capacity=capacity, record_digests=True)
    dec.debug_set_cluster_size(8)
    words, nwords, cost, flags = (t.cpu().numpy() for t in dec.decode_batch(torch_cuda.from_numpy(rows).cuda(), [n], c2.beam, c2.max_active))
    assert dec.debug_last_launch()[1] == size
    cnt, dig = dec.debug_frame_digests(0)
    assert (cnt == ref.digest_count).all() and (dig == ref.digest_sum).all()
    assert words[0, :nwords[0]].tolist() == ref.words.tolist() and cost[0] == np.float32(ref.cost) and flags[0] == ref.flags
    dec.close()


@pytest.mark.parametrize("cluster", [1, 2], indirect=True)
@pytest.mark.parametrize("n_z", [2000, 4000])          # the closure's rounds meet in the kept table, or in one of their own
def test_the_last_token_of_a_full_set_can_still_improve(torch_cuda, cluster, n_z):
    """65,536 tokens, as many as a set holds: the closure makes the last of them in one round and improves all that
    it made in the next."""
    from workloads.graphs import _csr
    hub, mid, z0 = 1, 2, 3
    dead0 = z0 + n_z
    S = 1 + 65536
    n_dead = S - dead0
    src = np.repeat([0, hub, mid], [n_dead + 1, n_z + 1, n_z])
    dst = np.concatenate([[hub], np.arange(dead0, S), [mid], np.arange(z0, dead0), np.arange(z0, dead0)])
    il = np.repeat([1, 0, 0], [n_dead + 1, n_z + 1, n_z])
    w = np.concatenate([np.zeros(n_dead + 1), [0.0], np.full(n_z, 0.01), np.full(n_z, 0.005)])
    g = _csr(S, 0, 2, src, dst, il, np.zeros(len(src)), w)
    ll = np.zeros((1, 1, 2), np.float32)
    (ref,) = parity.check_batch(torch_cuda, g, ll, np.array([1], np.int32), 5.0, 5000, max_active_hint=10000,
                               lattice_bytes_per_channel=1 << 20)
    assert ref.digest_count.tolist() == [1, 65536]


def test_without_memory_for_clusters(torch_cuda, c2, c2_refs):
    """A bound on the clusters' memory: calls that do not get enough decode with one workgroup per utterance, calls that
    can do with what is there keep it, and all of them have the oracle's results."""
    from paper_2311_04996_amd import Decoder
    B, T = 24, int(c2.lengths[:24].max())
    ll = torch_cuda.from_numpy(np.ascontiguousarray(c2.loglikes[:B, :T])).cuda()
    dec = Decoder(c2.graph, max_channels=B, max_frames=T, max_active_hint=c2.max_active)
    own = dec.device_bytes()

    def decode(n, dec=dec):
        words, nwords, cost, flags = (t.cpu().numpy() for t in dec.decode_batch(ll[:n].contiguous(), c2.lengths[:n], c2.beam, c2.max_active))
        for b in range(n):
            r = c2_refs[b]
            assert words[b, :nwords[b]].tolist() == r.words.tolist() and cost[b] == np.float32(r.cost) and flags[b] == r.flags
        return dec.debug_last_launch()[1], dec.device_bytes() - own
    dec.debug_set_cluster_memory(0)
    assert decode(B) == (1, 0)
    dec.debug_set_cluster_memory()
    g, small = decode(2)
    assert g == 8 and small > 0
    dec.debug_set_cluster_memory(small)
    assert decode(B) == (1, small) and decode(2) == (8, small) and decode(B) == (1, small)
    other = Decoder(c2.graph, max_channels=B, max_frames=T, max_active_hint=c2.max_active)
    g, large = decode(B, other)
    other.close()
    dec.debug_set_cluster_memory(large)             # enough for exactly these, not beside the old memory
    assert g == 8 and large > 10 * small and decode(B) == (8, large) and decode(2) == (8, large)
    dec.debug_set_cluster_memory()
    assert decode(B) == (8, large)
    dec.close()


def test_the_first_call_with_clusters_waits_for_no_other_stream(torch_cuda, c2):
    from paper_2311_04996_amd import Decoder
    torch = torch_cuda
    ll = torch.from_numpy(np.ascontiguousarray(c2.loglikes[:4, :40])).cuda()
    dec = Decoder(c2.graph, max_channels=4, max_frames=40, max_active_hint=c2.max_active)
    a, other, done = torch.randn(8192, 8192, device="cuda"), torch.cuda.Stream(), torch.cuda.Event()
    out = tuple(torch.zeros(s, dtype=t, device="cuda") for s, t in (((4, 256), torch.int32), (4, torch.int32), (4, torch.float32), (4, torch.int32)))
    torch.cuda.synchronize()
    with torch.cuda.stream(other):
        for _ in range(60):                          # some 10 ms each
            b = a @ a
        done.record()
    dec.decode_batch(ll, np.full(4, 40, np.int32), c2.beam, c2.max_active, out=out)
    assert not done.query() and dec.debug_last_launch()[1] > 1
    torch.cuda.synchronize()
    del b
    dec.close()


@pytest.mark.parametrize("size", [0, 2, 4, 8])
def test_a_launch_gets_at_most_the_workgroups_it_was_given(torch_cuda, c2, c2_refs, size):
    """Clusters start on all eight XCDs alike, so a launch with few workgroups gets smaller ones, or none."""
    from paper_2311_04996_amd import Decoder
    B, T = 20, 16
    lengths = np.full(B, T, np.int32)
    ll = torch_cuda.from_numpy(np.ascontiguousarray(c2.loglikes[:B, :T])).cuda()
    dec = Decoder(c2.graph, max_channels=B, max_frames=T, max_active_hint=c2.max_active, record_digests=True)
    dec.debug_set_cluster_size(size)
    sizes = {}
    for n in (1, 2, 7, 8, 15, 16, 31, 32, 63, 64, 100, 127, 128, 255, 256, 0):
        dec.set_launch_workgroups(n)
        dec.decode_batch(ll, lengths, c2.beam, c2.max_active)
        wgs, sizes[n] = dec.debug_last_launch()
        assert 0 < wgs <= (n or 256) and (size == 0 or sizes[n] <= size)
        for b in range(B):
            cnt, dig = dec.debug_frame_digests(b)
            assert (cnt == c2_refs[b].digest_count[:T + 1]).all() and (dig == c2_refs[b].digest_sum[:T + 1]).all()
    assert sizes[7] == sizes[8] == sizes[15] == 1 and sizes[0] == sizes[256] == (size or 8)
    if size:
        assert sizes[16] == sizes[31] == 2 and sizes[32] == sizes[63] == min(size, 4) and sizes[64] == size
    dec.close()


def test_launches_in_flight_share_the_compute_units(torch_cuda, c2, c2_refs):
    """Batches on three slots and streams, nothing set: the second and the third launch get a half and a third of the
    compute units while the first runs, the next three a third each, and a batch on its own gets all of them
    again after as many launches as there are slots."""
    from paper_2311_04996_amd import Decoder
    torch = torch_cuda
    B, T = 24, int(c2.lengths[:24].max())
    dec = Decoder(c2.graph, max_channels=3 * B, max_frames=T, max_active_hint=c2.max_active, batch_slots=3)
    ll = torch.from_numpy(np.ascontiguousarray(c2.loglikes[:B, :T])).cuda()
    streams = [torch.cuda.Stream() for _ in range(3)]

    def check(outs):
        torch.cuda.synchronize()
        for out in outs:
            words, nwords, cost, flags = (x.cpu().numpy() for x in out)
            for b, r in enumerate(c2_refs[:B]):
                assert words[b, :nwords[b]].tolist() == r.words.tolist() and cost[b] == np.float32(r.cost) and flags[b] == r.flags
    for rep in range(2):
        torch.cuda.synchronize()
        outs, shapes = [], []
        for k in range(3):
            outs.append(dec.decode_batch(ll, c2.lengths[:B], c2.beam, c2.max_active, slot=k, stream=streams[k]))
            shapes.append(dec.debug_last_launch())
        for most, (wgs, _) in zip((85, 85, 85) if rep else (256, 128, 85), shapes):
            assert 24 <= wgs <= most, shapes
        assert rep or shapes[0] == (192, 8)
        check(outs)
    for k in range(3):
        dec.decode_batch(ll, c2.lengths[:B], c2.beam, c2.max_active, slot=0)
        torch.cuda.synchronize()
    assert dec.debug_last_launch() == (192, 8)
    # with a number of its own a launch keeps it, but when others are in flight it does not spend twice the
    # compute-unit time on an earlier end of its own
    dec.set_launch_workgroups(128)
    outs, shapes = [], []
    for k in range(3):
        outs.append(dec.decode_batch(ll, c2.lengths[:B], c2.beam, c2.max_active, slot=k, stream=streams[k]))
        shapes.append(dec.debug_last_launch())
    assert shapes[0] == (128, 8) and 64 < shapes[2][0] <= 128 and shapes[2][1] < 8, shapes
    check(outs)
    dec.close()


def test_a_captured_call_is_replayed(torch_cuda, c2, c2_refs):
    """A call recorded into a graph (the decoder's very first, which must not allocate) has one workgroup per utterance:
    every replay runs with the arguments of the recording.  Between the replays the inputs change, another
    decoder decodes, and the decoder itself too."""
    from paper_2311_04996_amd import Decoder
    torch = torch_cuda
    B, T = 6, 60
    lengths = np.array([60, 41, 60, 7, 33, 60], np.int32)
    rows = [np.ascontiguousarray(c2.loglikes[k * B:(k + 1) * B, :T]) for k in range(4)]
    refs = [parity.oracle_batch(c2.graph, r, lengths, c2.beam, c2.max_active) for r in rows]
    dec, other = (Decoder(c2.graph, max_channels=B, max_frames=T, max_active_hint=c2.max_active) for _ in range(2))
    ll = torch.from_numpy(rows[0]).cuda()
    out = tuple(torch.zeros(s, dtype=t, device="cuda") for s, t in (((B, 256), torch.int32), (B, torch.int32), (B, torch.float32), (B, torch.int32)))

    def check(out, want):
        torch.cuda.synchronize()
        words, nwords, cost, flags = (t.cpu().numpy() for t in out)
        for b, r in enumerate(want):
            assert words[b, :nwords[b]].tolist() == r.words.tolist() and cost[b] == np.float32(r.cost) and flags[b] == r.flags
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        dec.decode_batch(ll, lengths, c2.beam, c2.max_active, out=out)
    for k in (1, 2, 3, 0):
        ll.copy_(torch.from_numpy(rows[k]))
        for t in out:
            t.zero_()
        graph.replay()
        check(out, refs[k])
        check((dec if k == 3 else other).decode_batch(torch.from_numpy(rows[k]).cuda(), lengths, c2.beam, c2.max_active), refs[k])
    assert dec.debug_last_launch()[1] > 1
    dec.close(), other.close()


def _epsilon_fan_graph(n_items, deg, seed):
    """Start -> n_items states over labels 1 and 2 -> `deg` leaves each over epsilon arcs, out of a few more leaves than
    that; leaves have a self-loop, every eighth an epsilon arc to one more state, and go back to the start."""
    from workloads.graphs import _csr
    rng = np.random.default_rng([seed, n_items, deg])
    n_leaf = deg + 37
    leaf0, deep = 1 + n_items, 1 + n_items + n_leaf
    S = deep + 1
    items, leaves = np.arange(1, 1 + n_items), np.arange(leaf0, deep)
    ends = np.concatenate([leaf0 + rng.permutation(n_leaf)[:deg] for _ in items])
    chain = leaves[::8]
    src = np.concatenate([np.zeros(n_items, np.int64), np.repeat(items, deg), leaves, leaves, chain, [deep]])
    dst = np.concatenate([items, ends, leaves, np.zeros(n_leaf, np.int64), np.full(len(chain), deep), [deep]])
    il = np.concatenate([1 + items % 2, np.zeros(n_items * deg, np.int64), np.full(n_leaf, 1), 1 + leaves % 2,
                         np.zeros(len(chain), np.int64), [1]])
    ol = np.where(rng.random(len(src)) < 0.2, rng.integers(1, 20, len(src)), 0)
    return _csr(S, 0, 2, src, dst, il, ol, rng.choice([0.0, 0.25, 0.5, 1.0], len(src)))


@pytest.mark.parametrize("cluster", [1, 2, 8], indirect=True)
def test_epsilon_arcs_around_the_sizes_of_a_waves_list(torch_cuda, cluster):
    """States with as many epsilon arcs as a wave lists, one more, as many as a segment of the shared list, one more, and
    more segments than that list holds; worklists of one item to more than all waves take at once."""
    rng = np.random.default_rng(5)
    for n_items, deg in ((1, 1), (5, 63), (64, 64), (65, 65), (17, 128), (16, 129), (513, 3), (40, 1000)):
        ll = rng.choice([-0.5, -1.0, -1.5], (2, 5, 2)).astype(np.float32)
        parity.check_batch(torch_cuda, _epsilon_fan_graph(n_items, deg, 3), ll, np.array([5, 3], np.int32), 20.0, 4000,
                           max_active_hint=8000)


@pytest.mark.parametrize("cluster", [2], indirect=True)
@pytest.mark.parametrize("times,n", [(1, 8100), (1, 9000), (1, 10100), (1, 11200), (1, 12600), (1, 21000), (3, 8000)])
def test_candidates_around_what_a_table_and_the_notes_hold(torch_cuda, cluster, times, n):
    """As many candidates for one destination (the start, from every leaf) as slots are noted in LDS and in each of the
    registers behind, and more; closure rounds (hubs that lead to `n` leaves, each leaf `times` over) with fewer and
    more new destinations than the closure's table holds."""
    from workloads.graphs import _csr
    rng = np.random.default_rng([23, n])
    per_hub = 3500
    hubs = np.arange(1, 1 + -(-n * times // per_hub))
    leaves = 1 + len(hubs) + np.arange(n)
    S = 1 + len(hubs) + n
    src = np.concatenate([np.zeros(len(hubs), np.int64), 1 + np.arange(n * times) // per_hub, leaves, leaves])
    dst = np.concatenate([hubs, np.concatenate([rng.permutation(leaves) for _ in range(times)]), leaves, np.zeros(n, np.int64)])
    il = np.concatenate([1 + hubs % 2, np.zeros(n * times, np.int64), np.ones(n, np.int64), 1 + leaves % 2])
    g = _csr(S, 0, 2, src, dst, il, np.where(rng.random(len(src)) < 0.2, 7, 0), rng.choice([0.0, 0.25, 0.5, 1.0], len(src)))
    ll = rng.choice([-0.5, -1.0, -1.5], (2, 5, 2)).astype(np.float32)
    parity.check_batch(torch_cuda, g, ll, np.array([5, 3], np.int32), 20.0, 30000, max_active_hint=60000)


@pytest.mark.parametrize("cluster", [1], indirect=True)
@pytest.mark.parametrize("n", [3072, 3073, 6144, 6145, 8192, 8193, 9216, 9217, 10240, 10241, 11264, 11265, 15000, 21000])
def test_candidates_around_what_one_workgroup_notes(torch_cuda, cluster, n):
    """One workgroup of the cluster kernel: `n` tokens have an arc each, all to one state, or each to a state of its own.  Sizes
    around what the registers, one pass, the notes in LDS and each of the registers behind them hold, for the fullest
    of its regions; twice as many candidates from tokens with two arcs."""
    from paper_2311_04996_amd import Decoder
    from workloads.graphs import _csr
    rng = np.random.default_rng([37, n])
    hubs = 1 + np.arange(-(-n // 3500))
    leaves = 1 + len(hubs) + np.arange(n)
    ends = 1 + len(hubs) + n + np.arange(n + len(hubs) + 1)        # with the usual self-loop alone: half of the states
    S = int(ends[-1]) + 1
    ll = rng.choice([-0.5, -1.0, -1.5], (2, 4, 2)).astype(np.float32)
    lengths = np.array([4, 2], np.int32)
    for dst in (np.zeros(n, np.int64), ends[:n], np.concatenate([np.zeros(n, np.int64), rng.permutation(ends[:n])])):
        src = np.resize(leaves, len(dst))
        a_src = np.concatenate([np.zeros(len(hubs), np.int64), 1 + np.arange(n) // 3500, src, ends])
        a_dst = np.concatenate([hubs, rng.permutation(leaves), dst, ends])
        il = np.concatenate([1 + hubs % 2, np.zeros(n, np.int64), 1 + src % 2, np.ones(len(ends), np.int64)])
        g = _csr(S, 0, 2, a_src, a_dst, il, np.where(a_src == a_dst, 0, rng.integers(1, 1000, len(a_src))),
                 np.where(a_src == a_dst, 0.0, rng.choice([0.0, 0.25, 0.5, 1.0], len(a_src))))
        refs = parity.oracle_batch(g, ll, lengths, 20.0, 12000)
        assert _candidates(g, ll[0], 2, 20.0, 12000)[1] == len(dst)
        dec = Decoder(g, max_channels=2, max_frames=4, max_active_hint=60000)
        out = dec.decode_batch(torch_cuda.from_numpy(ll).cuda(), lengths, 20.0, 12000)
        assert dec.debug_last_launch()[1] == 1 and dec.debug_last_kernel() == 2
        _same_results(dec, out, refs)
        dec.close()


@pytest.mark.parametrize("cluster,n,ma", [(1, 6144, 5000), (2, 11000, 5000), (2, 12288, 5000), (1, 6144, 6000), (1, 12000, 6000)], indirect=["cluster"])
def test_a_closure_whose_destinations_lie_at_regular_distances(torch_cuda, cluster, n, ma):
    """`n` states of three blocks each one behind the other, all reached over epsilon arcs in one round: as many as a closure's
    table (8,192 slots) takes, or nearly, but with probe sequences so alike that in four of five orders one of 6,144 finds no
    slot in the number of probes there are.  It is not lost, nor the channel stopped: sets, words, counters of the oracle.
    (With digests one workgroup takes another kernel beyond a max-active of 5,000.)"""
    from workloads.graphs import _csr
    rng = np.random.default_rng([41, n])
    per_hub = 3500
    hubs = 1 + np.arange(-(-n // per_hub))
    leaves = 1 + len(hubs) + np.arange(n)
    src = np.concatenate([np.zeros(len(hubs), np.int64), 1 + np.arange(n) // per_hub, np.repeat(leaves, 5)])
    dst = np.concatenate([hubs, rng.permutation(leaves), np.zeros(5 * n, np.int64)])
    il = np.concatenate([1 + hubs % 2, np.zeros(n, np.int64), np.tile([1, 2, 1, 2, 1], n)])
    g = _csr(1 + len(hubs) + n, 0, 2, src, dst, il, rng.integers(1, 1000, len(src)), rng.choice([0.0, 0.25, 0.5, 1.0], len(src)))
    ll = rng.choice([-0.5, -1.0, -1.5], (8, 5, 2)).astype(np.float32)
    refs = parity.check_batch(torch_cuda, g, ll, np.full(8, 5, np.int32), 20.0, ma, max_active_hint=20000)
    assert all(r.digest_count.tolist() == [1, len(hubs) + n] * 3 for r in refs)


def _probe(taken, key):
    """Probes of a key in a table of 8,192 slots until it comes to a free one, and that slot."""
    h, n = int(key) * 0x9E3779B1 & 0xFFFFFFFF, 0
    at, step = h >> 6 & 8191, (h >> 19 | 1) & 8191
    while taken[at]:
        at, n = (at + step) & 8191, n + 1
    return n, at


@pytest.mark.parametrize("cluster", [1], indirect=True)
@pytest.mark.parametrize("ma,narrow", [(5000, False), (500, False), (5000, True)])
def test_few_candidates_whose_destinations_lie_at_regular_distances(torch_cuda, cluster, ma, narrow):
    """3,000 states of three blocks each, a third of a table, but the probe sequence of the one that comes last runs through more
    than 257 others: with one that finds no slot the candidates, as many as registers hold, are recombined in more passes, and
    no channel stops.  (Narrow records: the other kernel.)"""
    from workloads.graphs import _csr
    n, rng = 3000, np.random.default_rng(43)
    leaves = 1 + np.arange(n)
    key = (n + 2) // 2 + 3 * np.arange(n)              # behind the start: a header and n arcs, two to a block
    taken = np.zeros(8192, bool)
    for k in key:
        taken[_probe(taken, k)[1]] = True
    last = int(np.argmax([_probe(taken, k)[0] for k in key]))
    order = np.concatenate([np.delete(leaves, last), [leaves[last]]])
    taken[:] = False
    for k in key[order[:-1] - 1]:
        taken[_probe(taken, k)[1]] = True
    assert _probe(taken, key[last])[0] > 300
    src = np.concatenate([np.zeros(n, np.int64), np.repeat(leaves, 5)])
    dst = np.concatenate([order, np.zeros(5 * n, np.int64)])
    il = np.concatenate([np.ones(n, np.int64), np.tile([1, 2, 1, 2, 1], n)])
    g = _csr(1 + n, 0, 2, src, dst, il, rng.integers(1, 1000, len(src)), np.concatenate([rng.choice([0.0, 0.015625], n), rng.choice([0.0, 0.25], 5 * n)]))
    ll = rng.choice([-0.5, -1.0, -1.5], (4, 5, 2)).astype(np.float32)
    parity.check_batch(torch_cuda, g, ll, np.full(4, 5, np.int32), 20.0, ma, max_active_hint=20000, narrow_arcs=narrow)


@pytest.mark.parametrize("cluster", [1, 2, 4, 8], indirect=True)
def test_an_overflow_in_a_frames_last_closure_round_stops_the_channel(torch_cuda, cluster):
    """10,002 tokens, 8,192 places, and no round and several frames after the one that finds no room: the channel is flagged
    all the same, whether another workgroup learns of it in this frame or in the next, and for every number of workgroups
    the frame has no digest and none of its tokens are expanded."""
    from paper_2311_04996_amd import Decoder, FLAG_CAPACITY, FLAG_DEAD
    from workloads.graphs import _csr
    n_dead, n_z = 6000, 4000
    hub, one, z0, dead0 = 1, 2, 3, 3 + n_z
    S = dead0 + n_dead
    dead, z = np.arange(dead0, S), np.arange(z0, dead0)
    src = np.concatenate([np.zeros(n_dead + 2, np.int64), np.full(n_z, hub), z, [one]])
    dst = np.concatenate([dead, [hub, one], z, z, [one]])
    il = np.concatenate([np.ones(n_dead + 1, np.int64), [2], np.zeros(n_z, np.int64), np.ones(n_z, np.int64), [2]])
    g = _csr(S, 0, 2, src, dst, il, np.zeros(len(src), np.int64), np.zeros(len(src)))
    ll = np.zeros((2, 4, 2), np.float32)
    ll[1, :, 0] = -1000.0                            # the second utterance keeps to the one state
    lengths = np.array([4, 4], np.int32)
    dec = Decoder(g, max_channels=2, max_frames=4, max_active_hint=1000, lattice_bytes_per_channel=1 << 18, record_digests=True,
                  keep_token_records=True)
    _, nwords, cost, flags = dec.decode_batch(torch_cuda.from_numpy(ll).cuda(), lengths, 5.0, 5000)
    torch_cuda.cuda.synchronize()
    assert flags.tolist()[0] & (FLAG_CAPACITY | FLAG_DEAD) == FLAG_CAPACITY | FLAG_DEAD and int(nwords[0]) == 0
    first, ref = parity.oracle_batch(g, ll, [1, 4], 5.0, 5000)
    cnt, dig = dec.debug_frame_digests(1)
    assert int(flags[1]) == ref.flags and float(cost[1]) == ref.cost
    assert (cnt == ref.digest_count).all() and (dig == ref.digest_sum).all()
    cnt, dig = dec.debug_frame_digests(0)
    assert len(dig) == 2 and cnt[0] == first.digest_count[0] and dig[0] == first.digest_sum[0] and dig[1] == 0
    # tokens expanded, arcs out of them, frames: of the stopped channel its one frame's
    assert dec.get_counters()[[0, 1, 7]].tolist() == [int(first.counters[k] + ref.counters[k]) for k in (0, 1)] + [1 + 4]
    dec.close()
    parity.check_batch(torch_cuda, g, ll, lengths, 5.0, 5000, max_active_hint=10000)


@pytest.mark.parametrize("cluster", [1, 2, 8], indirect=True)
def test_survivors_around_the_number_a_wave_collects(torch_cuda, cluster):
    """Sets of as many tokens as a wave, or all waves of a workgroup, make at a time, one fewer and one more: from candidates
    in the first frame, and from candidates and tokens that stay where they are in the next ones."""
    from workloads.graphs import _csr
    rng = np.random.default_rng(11)
    for n in (1, 63, 64, 65, 1023, 1025, 2049, 4000):
        leaves = np.arange(1, n + 1)
        back = leaves[::3]                           # the others have the self-loop alone
        src = np.concatenate([np.zeros(n, np.int64), leaves, back])
        dst = np.concatenate([leaves, leaves, np.zeros(len(back), np.int64)])
        il = np.concatenate([2 + leaves % 2, np.ones(n, np.int64), np.full(len(back), 2)])
        w = np.concatenate([rng.choice([0.0, 0.5, 1.0], n), np.zeros(n), np.full(len(back), 0.25)])
        g = _csr(n + 1, 0, 3, src, dst, il, np.where(rng.random(len(src)) < 0.1, 7, 0), w)
        ll = rng.choice([-0.5, -1.0, -2.0], (2, 4, 3)).astype(np.float32)
        parity.check_batch(torch_cuda, g, ll, np.array([4, 2], np.int32), 20.0, 5000, max_active_hint=5000)


@pytest.mark.parametrize("cluster", [1, 2, 4, 8], indirect=True)
@pytest.mark.parametrize("n", [3, 700])
def test_frames_whose_last_closure_round_is_any_of_the_first_five(torch_cuda, cluster, n):
    """Label k leads to n chains of k - 1 epsilon arcs, and one label is ahead of the beam in every frame: the frame's number of
    closure rounds is that label's, and whatever the round it ends with, the next frame's candidates do not meet the ones of
    that round."""
    from workloads.graphs import _csr
    rng = np.random.default_rng(17)
    arcs, first = [], 1
    for k in range(1, 6):
        at = first + np.arange(n * k).reshape(n, k)      # chain by chain
        first += n * k
        arcs += [(0, s, k, 0) for s in at[:, 0]] + [(s, d, 0, 0) for s, d in zip(at[:, :-1].ravel(), at[:, 1:].ravel())]
        arcs += [(s, 0, 1 + (k + j) % 5, 3 + k) for s in at[:, -1] for j in (0, 2)] + [(s, s, k, 0) for s in at[:, -1]]
    arcs += [(0, 0, k, 0) for k in range(1, 6)]
    src, dst, il, ol = (np.array(v, np.int64) for v in zip(*arcs))
    g = _csr(first, 0, 5, src, dst, il, ol, rng.choice([0.0, 0.25, 0.5], len(src)))
    label = np.array([[0, 1, 2, 3, 4, 1, 1, 3, 3, 0, 2, 4], [4, 3, 2, 1, 0, 0, 2, 2, 4, 4, 1, 3]])
    ll = np.where(np.arange(5) == label[..., None], -0.25, -100.0).astype(np.float32)
    parity.check_batch(torch_cuda, g, ll, np.array([12, 11], np.int32), 20.0, 5000, max_active_hint=5000)


@pytest.mark.parametrize("cluster", [2, 4, 8], indirect=True)
def test_closure_rounds_in_which_most_workgroups_get_nothing(torch_cuda, cluster):
    """Chains of 40 and 23 epsilon arcs, so a round has one or two candidates and most workgroups of a cluster go from one
    exchange to the next with nothing to expand and nothing to recombine, some forty times a frame: all waves of all of them
    leave the closure in the same round, with the oracle's sets, links and words (one per arc of the chains)."""
    import test_gpu_lattice as lattice
    from workloads.graphs import _csr
    rng = np.random.default_rng(29)
    arcs = [(0, 0, 2, 0)]
    for first, n, label in ((1, 40, 1), (42, 23, 2)):
        chain = first + np.arange(n + 1)
        arcs += [(0, first, label, 0)] + [(int(s), int(s) + 1, 0, int(s)) for s in chain[:-1]]
        arcs += [(int(chain[-1]), 0, 1, 70 + label), (int(chain[-1]), int(chain[-1]), 2, 0), (int(chain[n // 2]), 0, 2, 0)]
    src, dst, il, ol = (np.array(v, np.int64) for v in zip(*arcs))
    final = np.full(66, np.inf)
    final[41] = 0.0                                    # the longer chain's end
    g = _csr(66, 0, 2, src, dst, il, ol, rng.choice([0.0, 0.25, 0.5], len(src)), final)
    B, T = 40, 6                                       # more than the 32 clusters there are of 8
    ll = rng.choice([-0.25, -0.5, -1.0], (B, T, 2)).astype(np.float32)
    refs = parity.check_batch(torch_cuda, g, ll, (T - np.arange(B) % 5).astype(np.int32), 40.0, 5000, max_active_hint=5000)
    assert min(len(r.words) for r in refs) >= 40
    lattice.check_lattice(torch_cuda, g, ll[0], T, 40.0, 5000, 20.0)


@pytest.mark.parametrize("cluster", [2, 4, 8], indirect=True)
def test_token_numbers_where_the_first_workgroup_has_no_epsilon_arcs_to_expand(torch_cuda, cluster):
    """Label k leads to 200 dead ends and one hub, of 24 states between the workgroups, whose 300 epsilon arcs make the frame's other
    tokens: in many frames the first workgroup, which stores the number of tokens the closure starts from, has nothing to
    expand, and the others' tokens still get numbers, places in the lattice and backpointers of their own."""
    import test_gpu_lattice as lattice
    from workloads.graphs import _csr
    rng = np.random.default_rng(31)
    n_hub, n_dead, n_leaf = 24, 200, 300
    hubs, dead = np.arange(1, 1 + n_hub), 1 + n_hub + np.arange(n_dead)
    leaves = 1 + n_hub + n_dead + np.arange(n_leaf)
    src = np.concatenate([np.zeros(n_hub * (1 + n_dead), np.int64), np.repeat(hubs, n_leaf), np.repeat(leaves, n_hub)])
    dst = np.concatenate([hubs, np.tile(dead, n_hub), np.tile(leaves, n_hub), np.zeros(n_leaf * n_hub, np.int64)])
    il = np.concatenate([hubs, np.repeat(hubs, n_dead), np.zeros(n_hub * n_leaf, np.int64), np.tile(hubs, n_leaf)])
    ol = np.concatenate([hubs, np.zeros(n_dead * n_hub, np.int64), np.tile(100 + leaves, n_hub), np.zeros(n_leaf * n_hub, np.int64)])
    g = _csr(1 + n_hub + n_dead + n_leaf, 0, n_hub, src, dst, il, ol, rng.choice([0.0, 0.25, 0.5, 1.0], len(src)),
             np.where(np.arange(1 + n_hub + n_dead + n_leaf) < 1 + n_hub + n_dead, np.inf, 0.0))
    B, T = 12, 24
    label = rng.integers(0, n_hub, (B, T))
    ll = np.where(np.arange(n_hub) == label[..., None], -0.25, -100.0).astype(np.float32)
    refs = parity.check_batch(torch_cuda, g, ll, np.full(B, T - 1, np.int32), 20.0, 5000, max_active_hint=5000)
    assert min(len(r.words) for r in refs) == T and refs[0].digest_count[1] == 1 + n_dead + n_leaf
    lattice.check_lattice(torch_cuda, g, ll[0], T - 1, 20.0, 5000, 10.0)


def _late_fan_graph(n_dead, n_z, n_few=20):
    """Start -> a state with a loop over label 2, from where label 1 leads to `n_dead` dead ends and, over a hub's epsilon arcs,
    to `n_z` states with a self-loop, and label 3 to a few states and back over label 2."""
    from workloads.graphs import _csr
    one, hub, few0 = 1, 2, 3
    z0 = few0 + n_few
    dead0 = z0 + n_z
    S = dead0 + n_dead
    few, z, dead = np.arange(few0, z0), np.arange(z0, dead0), np.arange(dead0, S)
    src = np.concatenate([[0], np.full(2 + n_few + n_dead, one), np.full(n_z, hub), few, few, z])
    dst = np.concatenate([[one], [one, hub], few, dead, z, np.full(n_few, one), np.roll(few, 1), z])
    il = np.concatenate([[2], [2, 1], np.full(n_few, 3), np.full(n_dead, 1), np.zeros(n_z), np.full(n_few, 2), np.full(n_few, 3),
                         np.ones(n_z)]).astype(np.int64)
    w = np.concatenate([np.zeros(3), 0.125 * np.arange(n_few), np.zeros(n_dead + n_z), np.full(2 * n_few, 0.5), np.zeros(n_z)])
    return _csr(S, 0, 3, src, dst, il, np.where(il == 3, 7, 0), w)


@pytest.mark.parametrize("cluster,ma", [(1, 5000), (1, 6000), (2, 5000), (4, 5000), (8, 5000)], indirect=["cluster"])
def test_an_arena_that_ends_in_a_frames_only_closure_round_keeps_the_neighbours_records(torch_cuda, cluster, ma):
    """The 13th frame's 3,001 emitted tokens fit the arena of 4,096, the 3,000 its closure adds do not, and more frames
    follow: the channel is flagged and its lattice refused, and the digests and lattices of the channels whose arenas lie
    between and behind are the oracle's, every token and link.  (With digests one workgroup takes another kernel beyond a
    max-active of 5,000.)"""
    from oracle import Oracle
    from paper_2311_04996_amd import Decoder, FLAG_DEAD, FLAG_LATTICE_OVERFLOW, WfstError
    from test_gpu_lattice import gpu_rows, oracle_rows
    g = _late_fan_graph(3000, 3000)
    B, T, beam = 5, 16, 5.0
    over = (0, 2, 4)
    ll = np.full((B, T, 3), -1000.0, np.float32)
    rng = np.random.default_rng(17)
    ll[:, :, 1:] = rng.choice([-0.25, -0.5, -1.0], (B, T, 2))     # labels 2 and 3
    for b in over:
        ll[b] = -1000.0
        ll[b, :12, 1] = ll[b, 12:, 0] = 0.0
    dec = Decoder(g, max_channels=B, max_frames=T, max_active_hint=1000, lattice_bytes_per_channel=8 * 4096, keep_token_records=True,
                  record_digests=True)
    dev = torch_cuda.from_numpy(ll).cuda()
    lengths = np.full(B, T, np.int32)
    _, nwords, _, flags = (t.cpu().numpy() for t in dec.decode_batch(dev, lengths, beam, ma))
    o = Oracle(g)
    for b in range(B):
        if b in over:
            assert flags[b] & (FLAG_LATTICE_OVERFLOW | FLAG_DEAD) == FLAG_LATTICE_OVERFLOW | FLAG_DEAD and nwords[b] == 0
            with pytest.raises(WfstError):
                dec.get_lattice(b, dev[b], 4.0)
            continue
        (ref,), (cnt, dig) = parity.oracle_batch(g, ll[b:b + 1], lengths[:1], beam, ma), dec.debug_frame_digests(b)
        assert (cnt == ref.digest_count).all() and (dig == ref.digest_sum).all()
        L = o.lattice(ll[b], T, beam=beam, max_active=ma, lattice_beam=4.0)
        lat = dec.get_lattice(b, dev[b], 4.0)
        assert lat.frame_off.tolist() == L.set_off.tolist()
        for t in range(T + 1):
            a, e = int(L.set_off[t]), int(L.set_off[t + 1])
            assert sorted(zip(lat.state[a:e].tolist(), lat.cost[a:e].tolist())) == sorted(zip(L.states[a:e].tolist(), L.costs[a:e].tolist()))
        want, got = oracle_rows(o, g, L), gpu_rows(lat)
        assert got.shape == want.shape and (got == want).all()
    dec.close()
