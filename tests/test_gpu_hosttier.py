"""GPU tests of the DRAM-tier side of restores and spills: pinned host blocks
-> staging -> pool (restore) and pool -> staging -> host (spill), pipelined
in batches over two streams, byte-exact against the oracle's per-chunk
memcpy."""
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


def _geom(layout, nb, L, chunk):
    if layout == "layer_major":
        g = dict(slot_stride=chunk, kv_stride=nb * chunk, layer_stride=2 * nb * chunk)
    else:
        g = dict(slot_stride=2 * L * chunk, kv_stride=chunk, layer_stride=2 * chunk)
    g.update(num_layers=L, chunk_bytes=chunk, num_blocks=nb)
    return g


def _case(seed, layout, chunk, nm, nb=70, L=3):
    rng = np.random.default_rng(seed)
    g = _geom(layout, nb, L, chunk)
    blk = 2 * L * chunk
    mv = np.zeros(nm, ref.MOVE_DTYPE)
    mv["pool_slot"] = rng.permutation(nb)[:nm]
    mv["staging_slot"] = np.arange(nm)
    # distinct host places in [0, 3*nm] (the buffer holds 3*nm + 1 blocks),
    # about 40 % of them right after the
    # previous move's place (runs that travel as one copy)
    host_off = np.zeros(nm, np.int64)
    used = set()
    for m in range(nm):
        p = int(rng.integers(0, 3 * nm))
        nxt = int(host_off[m - 1] // blk + 1) if m > 0 else -1
        if m > 0 and rng.random() < 0.4 and nxt <= 3 * nm and nxt not in used:
            p = nxt
        while p in used:
            p = (p + 1) % (3 * nm + 1)
        used.add(p)
        host_off[m] = p * blk
    host_len = (3 * nm + 1) * blk
    return rng, g, blk, mv, host_off, host_len


def _restore_spill(dev, layout, chunk, batch, nm=25, nb=70, L=3, n_dev=None, seed=0):
    """Restore nm moves from pinned host blocks into the pool and spill the
    same slots back out, checked byte for byte against the oracle.  Only
    the first n_dev moves (the device count) are unpacked and packed; the
    host link carries all nm.  Every buffer is written on the compute stream
    just before the call, so the copies rely on the entry points' own
    ordering against earlier compute-stream work."""
    import torch
    from paper_2608_06557_amd import cascade
    n_dev = nm if n_dev is None else n_dev
    rng, g, blk, mv, host_off, host_len = _case(seed, layout, chunk, nm, nb=nb, L=L)
    pool_h = rng.integers(0, 256, 2 * g["num_layers"] * g["num_blocks"] * chunk, dtype=np.uint8)
    host = torch.from_numpy(rng.integers(0, 256, host_len, dtype=np.uint8)).pin_memory()
    host_h = host.numpy().copy()
    # restore: staging slot m gets host block host_off[m], then the oracle
    # unpacks the moves the device count covers
    st_h = np.concatenate([host_h[o:o + blk] for o in host_off])
    exp_pool = pool_h.copy()
    ref.unpack(exp_pool, g, st_h, mv[:n_dev])
    comp_s = torch.cuda.current_stream()
    pool = torch.from_numpy(pool_h.copy()).cuda()
    st = torch.full((nm * blk,), 7, dtype=torch.uint8, device="cuda")
    mv_d = torch.from_numpy(mv.view(np.int32).copy()).cuda()
    n_d = torch.tensor([n_dev], dtype=torch.int32, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    copy_s = torch.cuda.Stream()
    evs, handles = dev.event_handles(2)
    pl = dev.kv_pool_struct(pool.data_ptr(), g)
    rc = cascade.cascade_restore_from_host(pl, st.data_ptr(), nm, host.data_ptr(), host_off,
                                           mv_d.data_ptr(), n_d.data_ptr(), nm, batch,
                                           status.data_ptr(), copy_s.cuda_stream,
                                           comp_s.cuda_stream, handles)
    assert rc == 0
    comp_s.synchronize()
    assert int(status.item()) == 0
    assert np.array_equal(pool.cpu().numpy(), exp_pool)
    # spill the same slots back out to other host places: the oracle packs
    # the moves the device count covers; the staging slots past it keep
    # their old bytes, which the host link still carries
    host2 = torch.zeros(host_len, dtype=torch.uint8).pin_memory()
    st2 = torch.full((nm * blk,), 9, dtype=torch.uint8, device="cuda")
    exp_st = np.full(nm * blk, 9, np.uint8)
    ref.pack(exp_pool, g, exp_st, mv[:n_dev])
    exp_host = np.zeros(host_len, np.uint8)
    for m in range(nm):
        exp_host[host_off[m]:host_off[m] + blk] = exp_st[m * blk:(m + 1) * blk]
    rc = cascade.cascade_spill_to_host(pl, st2.data_ptr(), nm, host2.data_ptr(), host_off,
                                       mv_d.data_ptr(), n_d.data_ptr(), nm, batch,
                                       status.data_ptr(), copy_s.cuda_stream,
                                       comp_s.cuda_stream, handles)
    assert rc == 0
    copy_s.synchronize()
    assert np.array_equal(host2.numpy(), exp_host)
    torch.cuda.synchronize()


@pytest.mark.parametrize("layout", ["layer_major", "block_major"])
@pytest.mark.parametrize("chunk", [64, 4096])
@pytest.mark.parametrize("batch", [1, 3, 7, 100])
def test_restore_and_spill(dev, layout, chunk, batch):
    _restore_spill(dev, layout, chunk, batch, seed=batch * 7 + chunk)


@pytest.mark.parametrize("n_dev", [0, 1, 13, 24])
def test_device_count_short_of_the_host_count(dev, n_dev):
    """Batches past the device count copy nothing on the GPU."""
    _restore_spill(dev, "layer_major", 256, 4, nm=25, n_dev=n_dev, seed=40 + n_dev)


@pytest.mark.parametrize("layout", ["layer_major", "block_major"])
def test_real_2mib_blocks(dev, layout):
    """Blocks of the 8B-class geometry: 32 layers x K/V x 32 KiB = 2 MiB."""
    print(f"host tier 2 MiB blocks {layout}", flush=True)
    _restore_spill(dev, layout, 32768, 5, nm=24, nb=48, L=32, seed=3)


def test_host_checks(dev):
    import torch
    from paper_2608_06557_amd import cascade
    g = _geom("layer_major", 8, 2, 64)
    pl = dev.kv_pool_struct(4096, g)
    _, handles = dev.event_handles(1)
    args = dict(staging=4096, staging_slots=4, host_blocks=4096, host_offsets=np.zeros(4),
                moves_dev=4096, n_moves_dev=4096, n_moves=4, batch_moves=2, status_dev=0,
                copy_stream=0, compute_stream=0, events=handles)
    f = cascade.cascade_restore_from_host
    assert f(pl, **dict(args, batch_moves=0)) == cascade.EINVAL
    assert f(pl, **dict(args, n_moves=5)) == cascade.ENOSPC
    assert f(pl, **dict(args, events=[])) == cascade.EINVAL
    assert f(pl, **dict(args, n_moves=0, events=[])) == cascade.OK


@pytest.mark.parametrize("how", ["pinned", "pageable", "odd_offset", "same_place", "many"])
@pytest.mark.parametrize("chunk", [16, 4112])
def test_link_routes(dev, how, chunk):
    """Pinned and pageable host memory, offsets off 16 bytes, two spills to one
    place (the later move's block stays) and more moves than a batch: the same
    bytes whatever route the host link's copies take."""
    import torch
    from paper_2608_06557_amd import cascade
    nm = 300 if how == "many" else 20
    rng, g, blk, mv, host_off, host_len = _case(chunk, "layer_major", chunk, nm, nb=nm + 9)
    if how == "odd_offset":
        host_off = host_off + 8
        host_len += 16
    if how == "same_place":
        host_off[7] = host_off[3]
    pool_h = rng.integers(0, 256, 2 * g["num_layers"] * g["num_blocks"] * chunk, dtype=np.uint8)
    host_h = rng.integers(0, 256, host_len, dtype=np.uint8)
    pin = (lambda t: t) if how == "pageable" else (lambda t: t.pin_memory())
    host, back = pin(torch.from_numpy(host_h.copy())), pin(torch.zeros(host_len, dtype=torch.uint8))
    exp_pool = pool_h.copy()
    ref.unpack(exp_pool, g, np.concatenate([host_h[o:o + blk] for o in host_off]), mv)
    exp_st = np.zeros(nm * blk, np.uint8)
    ref.pack(exp_pool, g, exp_st, mv)
    exp_back = np.zeros(host_len, np.uint8)
    for m in range(nm):
        exp_back[host_off[m]:host_off[m] + blk] = exp_st[m * blk:(m + 1) * blk]
    pool = torch.from_numpy(pool_h.copy()).cuda()
    st = torch.zeros(nm * blk, dtype=torch.uint8, device="cuda")
    mv_d = torch.from_numpy(mv.view(np.int32).copy()).cuda()
    n_d = torch.tensor([nm], dtype=torch.int32, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    copy_s, comp_s = torch.cuda.Stream(), torch.cuda.current_stream()
    _, handles = dev.event_handles(2)
    pl = dev.kv_pool_struct(pool.data_ptr(), g)
    for f, h in [(cascade.cascade_restore_from_host, host), (cascade.cascade_spill_to_host, back)]:
        print(how, chunk, f.__name__, flush=True)
        assert f(pl, st.data_ptr(), nm, h.data_ptr(), host_off, mv_d.data_ptr(), n_d.data_ptr(),
                 nm, 150, status.data_ptr(), copy_s.cuda_stream, comp_s.cuda_stream,
                 handles) == 0
        torch.cuda.synchronize()
    assert int(status.item()) == 0
    assert np.array_equal(pool.cpu().numpy(), exp_pool)
    assert np.array_equal(back.numpy(), exp_back)


@pytest.mark.parametrize("way", ["spill", "restore"])
def test_the_link_leaves_the_gpu_to_others(dev, way):
    """Kernels of another stream run at their usual pace while the host link
    moves blocks: each launch boundary on the GPU waits for the requests in
    flight before it, so a copy over the link that keeps many of them in
    flight from the compute units slows every other stream (a step 28 times).
    The bound of 4 leaves room for the copies' own share of HBM and for a
    cold clock; the copy engines measure 1.0 to 1.3."""
    import torch
    import paper_2608_06557_amd.synth as synth
    from paper_2608_06557_amd import cascade
    nm, chunk, layers = 160, 32768, 32
    g = _geom("layer_major", nm, layers, chunk)
    blk = 2 * layers * chunk
    mv = np.zeros(nm, ref.MOVE_DTYPE)
    mv["pool_slot"], mv["staging_slot"] = np.arange(nm), np.arange(nm)
    host_off = np.random.default_rng(4).permutation(nm).astype(np.int64) * blk
    pool = torch.zeros(nm * blk, dtype=torch.uint8, device="cuda")
    st = torch.zeros(nm * blk, dtype=torch.uint8, device="cuda")
    host = torch.zeros(nm * blk, dtype=torch.uint8, pin_memory=True)
    mv_d = torch.from_numpy(mv.view(np.int32).copy()).cuda()
    n_d = torch.tensor([nm], dtype=torch.int32, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    pl = dev.kv_pool_struct(pool.data_ptr(), g)
    f = cascade.cascade_spill_to_host if way == "spill" else cascade.cascade_restore_from_host
    copy_s, comp_s = torch.cuda.Stream(), torch.cuda.current_stream()
    # streams share a few hardware queues: one of these has a queue that waits
    # for neither of the call's streams
    sides = [torch.cuda.Stream() for _ in range(4)]
    _, handles = dev.event_handles(2)
    d = dev.DeviceStep(synth.make_workload(1, seed=2, n=8192))
    stamp = lambda: torch.cuda.Event(enable_timing=True)
    runs = 150

    def steps(side):
        with torch.cuda.stream(side):
            at = [stamp() for _ in range(runs + 1)]
            at[0].record()
            for e in at[1:]:
                assert d.run() == 0
                e.record()
        return at

    def link():
        assert f(pl, st.data_ptr(), nm, host.data_ptr(), host_off, mv_d.data_ptr(),
                 n_d.data_ptr(), nm, 16, status.data_ptr(), copy_s.cuda_stream,
                 comp_s.cuda_stream, handles) == 0

    link()
    steps(sides[0])
    torch.cuda.synchronize()                 # both paths are warm
    t = steps(sides[0])
    torch.cuda.synchronize()
    alone = sorted(a.elapsed_time(b) for a, b in zip(t, t[1:]))[runs // 2]
    best = []
    for side in sides:
        begin, end = stamp(), stamp()
        begin.record(comp_s)
        link()
        end.record(copy_s)
        t = steps(side)
        torch.cuda.synchronize()
        link_ms = begin.elapsed_time(end)
        beside = [a.elapsed_time(b) for a, b in zip(t, t[1:])
                  if begin.elapsed_time(a) < link_ms]
        print(f"{way}: link {link_ms:.2f} ms, {len(beside)} steps beside it, alone "
              f"{alone:.4f} ms", flush=True)
        best = max(best, beside, key=len)
    assert len(best) >= 4
    assert sorted(best)[len(best) // 2] < 4 * alone


def test_captured_restore_and_spill(dev):
    """Both calls in one captured graph, the copy stream forked and joined by
    their events: every replay moves the bytes that the buffers hold then, as
    an eager call does."""
    import torch
    from paper_2608_06557_amd import cascade
    nm, chunk = 25, 4096
    rng, g, blk, mv, host_off, host_len = _case(77, "layer_major", chunk, nm)
    pool_len = 2 * g["num_layers"] * g["num_blocks"] * chunk
    host = torch.zeros(host_len, dtype=torch.uint8).pin_memory()
    back = torch.zeros(host_len, dtype=torch.uint8).pin_memory()
    pool = torch.zeros(pool_len, dtype=torch.uint8, device="cuda")
    st_in = torch.zeros(nm * blk, dtype=torch.uint8, device="cuda")
    st_out = torch.zeros(nm * blk, dtype=torch.uint8, device="cuda")
    mv_d = torch.from_numpy(mv.view(np.int32).copy()).cuda()
    n_d = torch.tensor([nm], dtype=torch.int32, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    copy_s = torch.cuda.Stream()
    _, handles = dev.event_handles(3)
    pl = dev.kv_pool_struct(pool.data_ptr(), g)

    def both():
        comp_s = torch.cuda.current_stream()
        for f, st, h in [(cascade.cascade_restore_from_host, st_in, host),
                         (cascade.cascade_spill_to_host, st_out, back)]:
            assert f(pl, st.data_ptr(), nm, h.data_ptr(), host_off, mv_d.data_ptr(),
                     n_d.data_ptr(), nm, 7, status.data_ptr(), copy_s.cuda_stream,
                     comp_s.cuda_stream, handles) == 0
        comp_s.wait_stream(copy_s)

    both()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        both()
    for k in range(4):
        pool_h = rng.integers(0, 256, pool_len, dtype=np.uint8)
        host_h = rng.integers(0, 256, host_len, dtype=np.uint8)
        host.copy_(torch.from_numpy(host_h))
        pool.copy_(torch.from_numpy(pool_h))
        back.zero_()
        torch.cuda.synchronize()
        graph.replay() if k != 2 else both()      # an eager call between the replays
        torch.cuda.synchronize()
        want = pool_h.copy()
        ref.unpack(want, g, np.concatenate([host_h[o:o + blk] for o in host_off]), mv)
        assert np.array_equal(pool.cpu().numpy(), want), k
        for m in range(nm):
            o = host_off[m]
            assert np.array_equal(back.numpy()[o:o + blk], host_h[o:o + blk]), (k, m)
    assert int(status.item()) == 0
