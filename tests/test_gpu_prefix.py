"""GPU parity of the prefix-hit index and lookup (Section 4.4, prefix hit
detection) against the oracle, bit-exact: matched prefix length and tier of
every request, from seeded block-hash workloads with shared prefix families,
shallower duplicates, cached blocks past a gap and unrelated entries."""
import numpy as np
import pytest
import torch  # noqa: F401  (imported at collection: the first import is slow)

from oracle import ref

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    from paper_2608_06557_amd import cascade, device
    assert torch.cuda.is_available()
    cascade.load()
    return device


def run_both(dev, pw, capacity=None):
    d = dev.DevicePrefix(pw, capacity=capacity)
    assert d.build() == 0
    assert d.probe() == 0
    g = d.fetch()
    o = ref.prefix_probe(pw["index_hashes"], pw["index_tiers"], pw["block_offsets"],
                         pw["block_hashes"], pw["n_in"], pw["block_tokens"])
    return g, o, d


def assert_same(g, o, label=""):
    assert g["status"] == o["rc"], (label, g["status"], o["rc"])
    if o["rc"] != 0:
        return
    for k in ["n_prefix", "prefix_tier"]:
        if not np.array_equal(g[k], o[k]):
            bad = np.flatnonzero(g[k] != o[k])
            raise AssertionError(f"{label} {k}: {len(bad)} differ, first {bad[:5]}: "
                                 f"gpu {g[k][bad[:5]]} oracle {o[k][bad[:5]]}")


@pytest.mark.parametrize("cfg,shared", [(0, 0.0), (0, 0.3), (1, 0.3), (2, 0.3), (3, 0.5),
                                        (4, 0.2)])
def test_workloads(dev, cfg, shared):
    import paper_2608_06557_amd.synth as synth
    pw = synth.make_prefix_workload(cfg, shared_frac=shared, noise=5000)
    print(f"config {cfg}: {len(pw['n_in'])} requests, {len(pw['block_hashes'])} blocks, "
          f"{len(pw['index_hashes'])} index facts", flush=True)
    g, o, _ = run_both(dev, pw)
    assert_same(g, o, f"config {cfg}")
    assert (o["n_prefix"] > 0).sum() > len(o["n_prefix"]) // 4


def _pw(entries, reqs, bt=16):
    return {"index_hashes": np.array([e[0] for e in entries], np.uint64),
            "index_tiers": np.array([e[1] for e in entries], np.uint8),
            "block_offsets": np.cumsum([0] + [len(r[1]) for r in reqs]).astype(np.int32),
            "block_hashes": np.array([h for r in reqs for h in r[1]], np.uint64),
            "n_in": np.array([r[0] for r in reqs], np.int32), "block_tokens": bt}


def test_hand_example_and_long_runs(dev):
    # request 4 has 300 cached blocks (several 64-block rounds of one wave)
    # and request 5 misses at block 130
    long_run = list(range(1000, 1300))
    miss_130 = list(range(2000, 2200))
    entries = [(11, 0), (12, 0), (21, 2), (12, 1), (32, 1), (41, 0), (42, 0), (43, 0)]
    entries += [(h, h % 3) for h in long_run] + [(h, 1) for h in miss_130 if h != 2130]
    reqs = [(64, [11, 12, 13]), (40, [21, 22]), (64, [31, 32]), (40, [41, 42, 43]),
            (16 * 400, long_run), (16 * 400, miss_130)]
    g, o, _ = run_both(dev, _pw(entries, reqs))
    assert_same(g, o, "hand")
    assert list(g["n_prefix"][:4]) == [32, 16, 0, 32]
    assert g["n_prefix"][4] == 16 * 300 and g["n_prefix"][5] == 16 * 130


def test_duplicates_keep_the_deepest_tier(dev):
    rng = np.random.default_rng(4)
    hashes = np.arange(1, 201, dtype=np.uint64)
    entries = [(int(h), int(t)) for h in hashes for t in rng.integers(0, 3, 7)]
    rng.shuffle(entries)
    reqs = [(16 * 300, [int(h) for h in hashes])] + [(64, [int(h)]) for h in hashes]
    g, o, _ = run_both(dev, _pw(entries, reqs))
    assert_same(g, o, "duplicates")


def test_full_table_reports_enospc(dev):
    entries = [(h, 0) for h in range(1, 101)]      # 100 keys, 64 slots
    g, o, d = run_both(dev, _pw(entries, [(64, [1, 2])]), capacity=64)
    assert g["status"] == -2


@pytest.mark.parametrize("case", ["hash0_request", "hash0_index", "tier3", "n_in0", "offsets"])
def test_einval(dev, case):
    entries, reqs = [(7, 0)], [(64, [7, 8])]
    if case == "hash0_request":
        reqs = [(64, [0, 8])]
    elif case == "hash0_index":
        entries = [(0, 0)]
    elif case == "tier3":
        entries = [(7, 3)]
    elif case == "n_in0":
        reqs = [(0, [7])]
    pw = _pw(entries, reqs)
    if case == "offsets":
        pw = _pw(entries, [(64, [7]), (64, [8])])
        pw["block_offsets"] = np.array([0, 2, 1], np.int32)
    g, o, _ = run_both(dev, pw)
    assert o["rc"] == ref.EINVAL and g["status"] == ref.EINVAL


def test_clear_and_rebuild(dev):
    import paper_2608_06557_amd.synth as synth
    a = synth.make_prefix_workload(0, seed=11)
    b = synth.make_prefix_workload(0, seed=12)
    d = dev.DevicePrefix(a, capacity=1 << 16)
    assert d.build() == 0 and d.probe() == 0
    ga = d.fetch()
    db = dev.DevicePrefix(b, capacity=1 << 16)
    db.index = d.index                      # same index memory, cleared and refilled
    assert db.build() == 0 and db.probe() == 0
    gb = db.fetch()
    for pw, g in [(a, ga), (b, gb)]:
        o = ref.prefix_probe(pw["index_hashes"], pw["index_tiers"], pw["block_offsets"],
                             pw["block_hashes"], pw["n_in"], pw["block_tokens"])
        assert_same(g, o, "rebuild")


def test_empty(dev):
    g, o, _ = run_both(dev, _pw([], [(64, [5])]))
    assert_same(g, o, "empty index")
    g, o, _ = run_both(dev, _pw([(5, 1)], []))
    assert g["status"] == 0


def test_runs_ending_at_window_edges(dev):
    # A wave looks up 64, 128, 256, 256, ... blocks per window, so windows
    # start at blocks 0, 64, 192, 448, 704, 960, ...  Request j owns a
    # sequence whose first miss is at block m_j; the blocks past the miss are
    # cached in the deepest tier, and only the last block before the miss
    # reaches tier 1, so a window that let a block past the miss into the run
    # or its tier would show.
    edges = [0, 1, 2, 63, 64, 65, 127, 191, 192, 193, 447, 448, 449, 703, 704, 705, 959,
             960, 1215, 1216]
    entries, reqs = [], []
    for j, m in enumerate(edges):
        seq = [(j + 1) * 10_000 + b for b in range(1400)]
        entries += [(h, 0) for h in seq[:max(m - 1, 0)]]
        if m >= 1:
            entries.append((seq[m - 1], 1))
        entries += [(h, 2) for h in seq[m + 1:]]
        reqs.append((16 * 1400 + 5, seq))
    # runs capped by the prompt length at a window edge, with every block cached
    for j, lim in enumerate([64, 192, 448, 704]):
        seq = [900_000 + j * 10_000 + b for b in range(lim + 40)]
        entries += [(h, 1) for h in seq]
        reqs.append((16 * lim + 1, seq))
    g, o, _ = run_both(dev, _pw(entries, reqs))
    assert_same(g, o, "window edges")
    assert list(g["n_prefix"][:len(edges)] // 16) == edges
    assert list(g["n_prefix"][len(edges):] // 16) == [64, 192, 448, 704]


@pytest.mark.parametrize("seed", [1, 2])
def test_crowded_table(dev, seed):
    # 3700 keys in 4096 slots: long probe sequences, sequences that wrap past
    # the table's last slot, and keys one past a home slot at the end of a line
    rng = np.random.default_rng(seed)
    keys = np.unique(rng.integers(1, 1 << 40, 4000, dtype=np.uint64))[:3700]
    assert len(keys) == 3700
    tiers = rng.integers(0, 3, len(keys))
    entries = [(int(k), int(t)) for k, t in zip(keys, tiers)]
    absent = rng.integers(1 << 40, 1 << 41, 300, dtype=np.uint64)  # never a key
    reqs = []
    for _ in range(400):
        run = int(rng.integers(0, 600))
        seq = [int(k) for k in rng.choice(keys, run)] + [int(absent[rng.integers(0, 300)])]
        seq += [int(k) for k in rng.choice(keys, int(rng.integers(0, 50)))]
        reqs.append((16 * len(seq) + 1, seq))
    g, o, _ = run_both(dev, _pw(entries, reqs), capacity=4096)
    assert_same(g, o, f"crowded {seed}")


def test_null_status_and_a_single_long_request(dev):
    # status_dev may be NULL: the lookup then reports nothing, also on a zero
    # hash, and still writes every request's result.  One request in a
    # workgroup of four waves, its run of 700 blocks over five windows.
    import paper_2608_06557_amd.cascade as cx
    from paper_2608_06557_amd.device import stream_handle
    seq = [50_000 + b for b in range(900)]
    entries = [(h, 1) for h in seq[:700]]
    for reqs, want in [([(16 * 900 + 1, seq)], 700), ([(16 * 4 + 1, [7, 0, 8, 9])], None)]:
        pw = _pw(entries + [(7, 2)], reqs)
        d = dev.DevicePrefix(pw)
        assert d.build() == 0
        d.n_prefix.fill_(-1)
        assert cx.cascade_prefix_probe(d.index.data_ptr(), d.capacity, d.n, d.off.data_ptr(),
                                       d.bh.data_ptr(), d.n_in.data_ptr(), d.bt,
                                       d.n_prefix.data_ptr(), d.tier.data_ptr(), None,
                                       stream_handle(None)) == 0
        g = d.fetch()
        o = ref.prefix_probe(pw["index_hashes"], pw["index_tiers"], pw["block_offsets"],
                             pw["block_hashes"], pw["n_in"], pw["block_tokens"])
        assert g["status"] == 0  # the status word was left alone
        if want is None:  # invalid input (hash 0): the result is written, its value unspecified
            assert o["rc"] == ref.EINVAL and int(g["n_prefix"][0]) >= 0
        else:
            assert_same(g, o, "null status")
            assert int(g["n_prefix"][0]) == 16 * want


def _edge_requests(edges, length, first_key):
    """One request per edge m: its first miss is at block m, the last block
    before it is in tier 1, the earlier ones in tier 0 and those past it in
    tier 2, so a block counted past the miss would show in the tier."""
    entries, reqs = [], []
    for j, m in enumerate(edges):
        seq = [first_key + j * 10_000 + b for b in range(length)]
        entries += [(h, 0) for h in seq[:max(m - 1, 0)]]
        if m >= 1:
            entries.append((seq[m - 1], 1))
        entries += [(h, 2) for h in seq[m + 1:]]
        reqs.append((16 * length + 5, seq))
    return entries, reqs


@pytest.mark.parametrize("n", [32, 2048, 2049, 3001])
def test_long_runs_shared_by_waves(dev, n):
    # up to 2048 requests a workgroup looks up one request in rounds of 1024
    # blocks; above, it shares the runs that reach block 1984 among its four
    # waves, whether one, two, three or all four of its requests do (rounds of
    # 1024, 512, 512 and 256, or 256 blocks)
    edges = [1983, 1984, 1985, 2239, 2240, 2241, 2495, 2496, 2497, 3007, 3008, 3009,
             4031, 4032, 0, 255, 256, 1023, 1024, 1025, 2047, 2048]
    entries, longs = _edge_requests(edges, 4100, 1_000_000)
    short, shorts = _edge_requests([0, 1, 40], 50, 9_000_000)
    at = {}
    pos = 4
    for k, r in enumerate(longs):           # workgroups of 1, 2, 3 and 4 long runs
        if k in (1, 3, 6):
            pos = (pos + 7) // 4 * 4
        at[min(pos, n - len(longs) + k)] = r
        pos += 1
    reqs = [at.get(i, shorts[i % 3]) for i in range(n)]
    pw = _pw(entries + short, reqs)
    g, o, _ = run_both(dev, pw)
    assert_same(g, o, f"shared runs {n}")
    assert sorted(g["n_prefix"][sorted(at)] // 16)[-1] == 4032


@pytest.mark.parametrize("n", [1, 2500])
@pytest.mark.parametrize("miss,zero,bad", [
    (10, 60, True), (10, 64, False), (100, 191, True), (100, 192, False), (500, 703, True),
    (500, 704, False), (1000, 1215, True), (1000, 1216, False), (2000, 2239, True),
    (2000, 2240, False), (2100, 2300, False)])
def test_zero_hash_past_the_miss(dev, n, miss, zero, bad):
    # a hash 0 is reported when it lies in the window (0, 64, 192, 448, 704, 960,
    # ...) that holds the first miss, or before it, however many waves look
    entries, reqs = _edge_requests([miss], 2400, 1_000_000)
    reqs[0][1][zero] = 0
    reqs += [(64, [5, 6])] * (n - 1)
    d = dev.DevicePrefix(_pw(entries, reqs))
    assert d.build() == 0 and d.probe() == 0
    g = d.fetch()
    assert g["status"] == (ref.EINVAL if bad else 0)
    assert g["n_prefix"][0] == 16 * miss and g["prefix_tier"][0] == 1


def test_insert_contended_and_repeated(dev):
    # many facts on few keys, in one wave and across workgroups, then the same
    # facts again, then one more tier for keys whose slots are there
    rng = np.random.default_rng(9)
    hashes = rng.integers(1, 1 << 60, 500, dtype=np.uint64)
    entries = [(int(hashes[k]), int(t)) for k, t in
               zip(rng.integers(0, 500, 60_000) // rng.integers(1, 60, 60_000),
                   rng.integers(0, 2, 60_000))]
    entries += [(int(h), 0) for h in hashes]
    reqs = [(16 * 501, [int(h) for h in hashes])] + [(64, [int(h)]) for h in hashes]
    pw = _pw(entries, reqs)
    d = dev.DevicePrefix(pw, capacity=1024)
    o = ref.prefix_probe(pw["index_hashes"], pw["index_tiers"], pw["block_offsets"],
                         pw["block_hashes"], pw["n_in"], pw["block_tokens"])
    assert d.build() == 0
    words = []
    for _ in range(2):
        assert d.probe() == 0
        assert_same(d.fetch(), o, "contended")
        words.append(d.index.clone())
        import paper_2608_06557_amd.cascade as cx
        from paper_2608_06557_amd.device import stream_handle
        assert cx.cascade_prefix_index_insert(
            d.index.data_ptr(), d.capacity, d.ih.data_ptr(), d.it.data_ptr(), d.n_entries,
            d.status.data_ptr(), stream_handle(None)) == 0
    assert torch.equal(words[0], words[1])  # facts already there change nothing
    slots = d.index.cpu().numpy().view(np.uint64).reshape(-1, 2)
    keys = slots[:, 0][slots[:, 0] != 0]
    assert len(keys) == len(np.unique(keys)) == len(np.unique(hashes))
    sets = dict(zip(slots[:, 0].tolist(), slots[:, 1].tolist()))
    want = {}
    for h, t in entries:
        want[h] = want.get(h, 0) | 1 << t
    assert all(sets[h] == w for h, w in want.items())
    assert (slots[:, 1][slots[:, 0] == 0] == 0).all()


# facts from which on an insert reads a slot before it claims it (half as many
# in an index of less than four slots a fact)
LOOK_FACTS = 1 << 19


def _insert(dev, index, capacity, hashes, tiers, status, stream=None):
    import paper_2608_06557_amd.cascade as cx
    assert cx.cascade_prefix_index_insert(index.data_ptr(), capacity, hashes.data_ptr(),
                                          tiers.data_ptr(), len(tiers), status.data_ptr(),
                                          dev.stream_handle(stream)) == 0


def _facts(rng, keys, n):
    """n facts on the keys, every key among them, and each key's tier set."""
    k = np.concatenate([np.arange(len(keys)), rng.integers(0, len(keys), n - len(keys))])
    t = rng.integers(0, 3, n).astype(np.uint8)
    order = rng.permutation(n)
    want = np.zeros(len(keys), np.uint32)
    np.bitwise_or.at(want, k, np.uint32(1) << t)
    return (torch.from_numpy(keys[k][order].view(np.int64)).cuda(),
            torch.from_numpy(t[order]).cuda(), want)


def _assert_contents(dev, index, keys, want):
    got_keys, got_sets = dev.index_contents(index.cpu().numpy())
    order = np.argsort(keys)
    assert np.array_equal(got_keys, keys[order])
    assert np.array_equal(got_sets, want[order])


@pytest.mark.parametrize("n,cap", [
    (200, 128), (5000, 2048), (LOOK_FACTS // 2 - 1, 1 << 17), (LOOK_FACTS // 2, 1 << 17),
    (LOOK_FACTS // 2, 1 << 20), (LOOK_FACTS // 2 + 1, 1 << 20), (LOOK_FACTS - 1, 1 << 21),
    (LOOK_FACTS, 1 << 21)])
def test_insert_both_ways(dev, n, cap):
    """Several facts per key, most of them on their way at the same time, into
    a table filled to 9/10 or a large one, then all of them again."""
    rng = np.random.default_rng(n + cap)
    keys = np.unique(rng.integers(1, 1 << 63, min(int(cap * 0.9), n // 2), dtype=np.uint64))
    h, t, want = _facts(rng, keys, n)
    index = torch.zeros(cap * 16, dtype=torch.uint8, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    for _ in range(2):
        _insert(dev, index, cap, h, t, status)
        assert int(status.item()) == 0
        _assert_contents(dev, index, keys, want)
    assert (index.view(torch.int32)[3::4] == 0).all()     # nothing was reclaimed


def test_inserts_of_both_ways_at_once(dev):
    """One long insert and many short ones on other streams, which share keys
    and slots with it: the union of their facts."""
    rng = np.random.default_rng(5)
    cap = 1 << 19
    keys = np.unique(rng.integers(1, 1 << 63, 400_000, dtype=np.uint64))
    h, t, want = _facts(rng, keys, LOOK_FACTS + 77)
    short = [_facts(rng, keys[rng.permutation(len(keys))[:3000]], 4000) for _ in range(24)]
    by_key = dict(zip(keys.tolist(), range(len(keys))))
    for sh, st, _ in short:
        at = [by_key[k] for k in sh.cpu().numpy().view(np.uint64).tolist()]
        np.bitwise_or.at(want, at, np.uint32(1) << st.cpu().numpy())
    index = torch.zeros(cap * 16, dtype=torch.uint8, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    streams = [torch.cuda.Stream() for _ in range(3)]
    torch.cuda.synchronize()
    _insert(dev, index, cap, h, t, status, streams[0])
    for k, (sh, st, _) in enumerate(short):
        _insert(dev, index, cap, sh, st, status, streams[1 + k % 2])
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    _assert_contents(dev, index, keys, want)


def test_insert_into_emptied_slots_without_a_mark(dev):
    """Index memory whose emptied slots carry no mark (as a copy of one made
    otherwise may): the wait for a first tier that will not come ends, and the
    facts are there all the same."""
    rng = np.random.default_rng(8)
    keys = np.unique(rng.integers(1, 1 << 63, 300, dtype=np.uint64))
    h, t, want = _facts(rng, keys, 900)
    index = torch.zeros(1024 * 16, dtype=torch.uint8, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    _insert(dev, index, 1024, h, t, status)
    index.view(torch.int32)[2::4] = 0                     # every set emptied
    _insert(dev, index, 1024, h, t, status)
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    _assert_contents(dev, index, keys, want)


@pytest.mark.parametrize("per_key,capacity", [(3, 1 << 16), (60, 1 << 20)])
def test_insert_into_reclaimed_sets(dev, per_key, capacity):
    """Blocks whose last copy a reclamation took come back, beside new blocks
    that probe past their slots.  The reclamation marks every slot it took a
    tier from, so that an insert knows an empty set from one whose first tier
    is on its way."""
    import paper_2608_06557_amd.synth as synth
    w = synth.make_tier_workload(2, seed=21, sizes=(2000, 9000, 30_000), needs=(700, 400, 3000))
    d = dev.DeviceTiers(w["tables"], w["needs"], w["index_keys"], w["index_masks"],
                        capacity=capacity)
    assert d.run_chain() == 0
    torch.cuda.synchronize()
    keys, sets = dev.index_contents(d.index.cpu().numpy())
    gone = keys[sets == 0]
    assert len(gone) > 1000
    words = d.index.cpu().numpy().view(np.uint32).reshape(-1, 4)
    occupied = (words[:, 0] | words[:, 1]) != 0
    assert (words[occupied & (words[:, 2] == 0), 3] == 1).all()
    rng = np.random.default_rng(per_key)
    new = np.setdiff1d(rng.integers(1, 1 << 63, 9000, dtype=np.uint64), keys)
    back = np.concatenate([gone, new])
    n = per_key * len(back)
    assert (n >= LOOK_FACTS // 2) == (per_key > 3)
    h, t, want = _facts(rng, back, n)
    _insert(dev, d.index, d.capacity, h, t, d.status)
    torch.cuda.synchronize()
    assert int(d.status.item()) == 0
    old = dict(zip(keys.tolist(), sets.tolist()))
    old.update(zip(back.tolist(), want.tolist()))
    all_keys = np.array(sorted(old), np.uint64)
    _assert_contents(dev, d.index, all_keys,
                     np.array([old[k] for k in all_keys.tolist()], np.uint32))


@pytest.mark.parametrize("n", [18, 2048, 2049])
def test_short_prompts(dev, n):
    """Prompts around 256 and 512 blocks, up to which a workgroup looks at
    4 x 64 and 4 x 128 blocks at once, and runs that end at the edges of the
    windows."""
    edges = [0, 1, 63, 64, 65, 127, 128, 191, 192, 193, 255, 256, 257, 447, 448, 510, 511, 512]
    for length in (70, 255, 256, 257, 511, 512, 513):
        entries, reqs = _edge_requests([min(e, length) for e in edges], length, 1_000_000)
        reqs = [reqs[i % len(reqs)] for i in range(n)]
        g, o, _ = run_both(dev, _pw(entries, reqs))
        assert_same(g, o, f"{length} blocks")
        assert int(g["n_prefix"].max()) == 16 * min(length, 512)


@pytest.mark.parametrize("n", [1, 2500])
@pytest.mark.parametrize("length,miss,zero,bad", [
    (500, 10, 60, True), (500, 10, 64, False), (500, 63, 64, False), (500, 64, 191, True),
    (500, 191, 192, False), (500, 192, 447, True), (500, 200, 448, False), (500, 255, 447, True),
    (500, 256, 447, True), (500, 447, 448, False), (500, 448, 499, True), (500, 300, 200, True),
    (250, 63, 64, False), (250, 64, 191, True), (250, 191, 192, False), (250, 192, 249, True),
    (900, 200, 447, True), (900, 200, 448, False), (900, 500, 703, True), (900, 500, 704, False)])
def test_zero_hash_past_the_miss_of_a_short_prompt(dev, n, length, miss, zero, bad):
    # as for the long prompts above, where other windows than those that decide
    # it are looked up
    entries, reqs = _edge_requests([miss], length, 1_000_000)
    reqs[0][1][zero] = 0
    reqs += [(64, [5, 6])] * (n - 1)
    d = dev.DevicePrefix(_pw(entries, reqs))
    assert d.build() == 0 and d.probe() == 0
    g = d.fetch()
    assert g["status"] == (ref.EINVAL if bad else 0)
    assert g["n_prefix"][0] == 16 * min(miss, zero) and g["prefix_tier"][0] == (zero > miss)
