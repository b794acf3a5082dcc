"""The lean walk kernels (one Philox block per lane and iteration; several lanes per walk for small
queries) against the per-step form, which draws word by word, and the oracle."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _graph(mode, **kw):
    """A graph whose vertices hold groups of every type and of ranks past the ten and twenty highest:
    a few heavy edges over many light ones, degrees 0 to 3000."""
    import torch
    from paper_2504_10233_amd import Graph, quantize_biases
    n, m = 600, 30000
    src = (synth.below(1, 1, m, n) * synth.below(1, 2, m, n)) // n
    src[:3000] = 5
    dst = synth.below(1, 3, m, n)
    w = torch.where(synth.below(1, 4, m, 50) == 0, synth.weights_uniform(m, 1 << 20, 1 << 23, 2),
                    synth.weights_zipf(m, 1.3, (1 << 18) - 1, 3))
    if mode == "float":
        bias = (w.double() + synth.uniform_f64(4, 1, m)).float().cuda()
        return n, Graph(n, src, dst, quantize_biases(bias, 1.0, 8), frac_bits=8)
    return n, Graph(n, src, dst, w, alias_table=mode == "alias", adaptive=mode != "plain")


# one lane group each up to a few thousand walks (64, 16, then 8 lanes a walk), the persistent kernel above
@pytest.mark.parametrize("mode", ["int", "plain", "float", "alias"])
def test_walks_equal_the_per_step_form(mode):
    import torch
    from paper_2504_10233_amd import MODE_PER_STEP
    n, g = _graph(mode)
    for nw in (1, 3, 257, 1999, 2049, 7001, 8200, 30001, 70003):
        starts = synth.below(9, nw, nw, n).to(torch.int32)
        a, sa = g.walk(starts, 17, 77, base=nw)
        b, sb = g.walk(starts, 17, 77, base=nw, mode=MODE_PER_STEP)
        assert torch.equal(a, b) and int(sa) == int(sb), nw
    g.close()


@pytest.mark.parametrize("mode", ["int", "float", "alias"])
@pytest.mark.parametrize("sources,per_source,stop", [(1, 1, 0.15), (3, 700, 0.15), (7, 1001, 0.02), (50, 999, 0.15),
                                                     (300, 301, 0.15), (40, 40, 1.0)])
def test_ppr_equals_the_per_step_form(mode, sources, per_source, stop):
    import torch
    from paper_2504_10233_amd import MODE_PER_STEP
    n, g = _graph(mode)
    src = synth.below(8, 1, sources, n).to(torch.int32)
    thr = min(int(stop * 2**32), 2**32 - 1)
    a = g.ppr(src, per_source, thr, 200, 5, base=1 << 33)
    b = g.ppr(src, per_source, thr, 200, 5, base=1 << 33, mode=MODE_PER_STEP)
    assert all(torch.equal(x, y) for x, y in zip(a[:3], b[:3])) and a[3] == b[3]
    g.close()


def test_a_vertex_past_the_32_bit_sums():
    """2^21 + 5 edges: the sums of its groups take the 64-bit path."""
    import torch
    import oracle as O
    from paper_2504_10233_amd import Graph
    n, hub = 64, (1 << 21) + 5
    src = torch.cat([torch.zeros(hub, dtype=torch.int64), synth.below(3, 1, 500, n)])
    dst = torch.cat([synth.below(3, 2, hub, n), torch.zeros(500, dtype=torch.int64)])
    w = synth.weights_uniform(src.numel(), 1, 1 << 24, 4)
    g = Graph(n, src, dst, w)
    og = O.Graph(n, src.numpy(), dst.numpy(), w.numpy())
    starts = torch.zeros(300, dtype=torch.int32)
    p, _ = g.walk(starts, 12, 3)
    q, _ = og.deepwalk(starts.numpy(), 12, seed=3)
    assert np.array_equal(p.cpu().numpy().view(np.uint32), q)
    g.close()


@pytest.mark.parametrize("p,q", [(0.5, 2.0), (4.0, 0.5), (1.0, 1.0), (0.25, 1.0)])
def test_node2vec_lanes_per_walk(p, q):
    """16, 8, 4, 2 lanes per walk and one: the first and last 600 walks of each size equal the oracle's."""
    import torch
    import oracle as O
    from paper_2504_10233_amd import Graph
    n, m = 500, 9000
    src = (synth.below(1, 1, m, n) * synth.below(1, 2, m, n)) // n
    dst = (synth.below(1, 3, m, n) * synth.below(1, 5, m, n)) // n
    w = synth.weights_uniform(m, 1, 1 << 16, 2)
    g = Graph(n, src, dst, w)
    og = O.Graph(n, src.numpy(), dst.numpy(), w.numpy())
    for nw in (1, 600, 20481, 41001, 90000, 170003, 340000):
        starts = synth.below(9, 1, nw, n).to(torch.int32)
        a, c = g.node2vec(starts, 9, 77, p, q, base=5)
        k = min(nw, 600)
        for lo in (0, nw - k):
            b = og.node2vec(starts[lo:lo + k].numpy(), 9, 77, p, q, base=5 + lo)[0]
            assert np.array_equal(a[lo:lo + k].cpu().numpy().view(np.uint32), b), (nw, lo)
        if nw == 600:
            assert c.tolist() == list(og.node2vec(starts.numpy(), 9, 77, p, q, base=5, with_proposals=True)[1:])
    g.close()


@pytest.mark.parametrize("degree", [2047, 2048, 2049, 2112, 16385, 40001])
@pytest.mark.parametrize("frac", [0, 8])
def test_build_around_the_hub_threshold(degree, frac):
    """A vertex at the edges of the block-per-hub construction, with groups of every type, beside others."""
    import oracle as O
    import torch
    from paper_2504_10233_amd import Graph
    n = 40
    src = torch.cat([torch.full((degree,), 7), synth.below(1, 1, 3000, n), torch.full((2500,), 39)])
    dst = synth.below(1, 2, src.numel(), n)
    w = synth.weights_zipf(src.numel(), 1.2, (1 << 30) - 1, 5)
    perm = torch.argsort(synth.uniform_u32(6, 1, src.numel()), stable=True)
    src, dst, w = src[perm], dst[perm], w[perm]
    g = Graph(n, src, dst, w, frac_bits=frac)
    og = O.Graph(n, src.numpy(), dst.numpy(), w.numpy(), frac_bits=frac)
    assert np.array_equal(g.export(), og.dump())
    assert np.array_equal(g.export_index(), og.index_dump())
    g.close()


@pytest.mark.parametrize("m", [4095, 4097, 256 * 4096 - 1, 256 * 4096, 256 * 4096 + 1])
def test_build_around_the_fused_sort_passes(m):
    """The records' sort around one tile and around the largest sort whose scatter adds up the counts itself."""
    import oracle as O
    from paper_2504_10233_amd import Graph
    n = 70000
    src, dst = synth.below(1, 1, m, n), synth.below(1, 2, m, n)
    w = synth.weights_uniform(m, 1, 1 << 16, 3)
    g = Graph(n, src, dst, w)
    og = O.Graph(n, src.numpy(), dst.numpy(), w.numpy())
    assert np.array_equal(g.export(), og.dump())
    g.close()


@pytest.mark.parametrize("degrees", [(1023, 1024, 1025), (2048, 2049, 40001), (1, 63, 64), (5000,) * 64])
@pytest.mark.parametrize("spread", [1, 3, 1 << 20])
def test_locator_build_around_its_chunks(degrees, spread):
    """Vertices at the edges of the chunks that building the locator splits hubs into, with many copies of an edge."""
    import torch
    from paper_2504_10233_amd import Graph
    n = 70000
    src = torch.cat([torch.full((d,), 60 + i) for i, d in enumerate(degrees)] + [synth.below(1, 1, 5000, n)])
    dst = synth.below(1, 2, src.numel(), min(n, spread))
    g = Graph(n, src, dst, synth.weights_uniform(src.numel(), 1, 1 << 12, 5))
    st = g.update(src[:3], dst[:3], torch.tensor([1, 2, 3]), src[1:70], dst[1:70])
    assert st["deleted"] == 69 and st["inserted"] == 3
    assert g.check_locator() == (0, src.numel() + 3 - 69)
    g.close()


@pytest.mark.parametrize("k", [3, 4, 5, 8, 9, 31, 32, 33, 64, 65])
@pytest.mark.parametrize("frac", [0, 8])
def test_batches_around_the_small_set_sizes(k, frac):
    """k inserts and k deletes on one vertex (low and high in its adjacency), on others one of the two."""
    import oracle as O
    import torch
    from paper_2504_10233_amd import Graph
    n, d, hot = 1200, 150, 12
    src = torch.arange(hot).repeat_interleave(d)
    dst = torch.arange(hot * d) % d  # no copies: a record names its edge
    w = synth.weights_zipf(hot * d, 1.2, (1 << 30) - 1, 5)
    g = Graph(n, src, dst, w, frac_bits=frac)
    og = O.Graph(n, src.numpy(), dst.numpy(), w.numpy(), frac_bits=frac)
    new = torch.arange(k) + 1000
    at = [torch.arange(k), d - 1 - torch.arange(k), (torch.arange(k) * 37) % d]
    ins = torch.cat([torch.full((k,), u) for u in (0, 1, 2, 3)])
    iw = synth.weights_zipf(4 * k, 1.2, (1 << 30) - 1, 6)
    dels = torch.cat([torch.full((k,), u) for u in (0, 1, 2, 4)])
    dd = torch.cat(at + [at[1]])
    for _ in range(2):
        g.update(ins, new.repeat(4), iw, dels, dd)
        og.update(ins.numpy(), new.repeat(4).numpy(), iw.numpy(), dels.numpy(), dd.numpy())
        assert np.array_equal(g.export(), og.dump())
        assert np.array_equal(g.export_index(), og.index_dump())
    g.close()


@pytest.mark.parametrize("ni,nd", [(1, 0), (0, 1), (1, 1), (63, 1), (0, 65), (500, 523), (1023, 0), (0, 1024), (512, 512),
                                   (512, 513), (700, 1348), (1025, 1024)])
@pytest.mark.parametrize("locate,split", [(1, 4096), (0, 0), (1, 100)])
def test_batches_around_the_one_block_steps(ni, nd, locate, split):
    """Batches up to, at and past the size whose steps run in one block: equal to the oracle's, records
    in random order, copies of edges, deletes of the batch's own inserts and of edges that are not there."""
    import oracle as O
    import torch
    from paper_2504_10233_amd import Graph
    n, m = 300, 9000
    src, dst = (synth.below(1, 1, m, n) * synth.below(1, 2, m, n)) // n, synth.below(1, 3, m, 40)
    w = synth.weights_zipf(m, 1.2, (1 << 30) - 1, 5)
    g = Graph(n, src, dst, w)
    g.set_tuning(update_locate=locate, update_split=split)
    og = O.Graph(n, src.numpy(), dst.numpy(), w.numpy())
    for b in range(3):
        isrc, idst = synth.below(20 + b, 1, ni, n) // 2, synth.below(20 + b, 2, ni, 60)
        iw = synth.weights_zipf(ni, 1.2, (1 << 30) - 1, 60 + b)
        pick = synth.below(20 + b, 3, nd, m) if nd else torch.zeros(0, dtype=torch.int64)
        ds, dd = src[pick], dst[pick] + (synth.below(20 + b, 4, nd, 10) == 0) * 20
        k = min(ni, nd) // 4
        ds[:k], dd[:k] = isrc[:k], idst[:k]
        s1 = g.update(isrc, idst, iw, ds, dd)
        s2 = og.update(isrc.numpy(), idst.numpy(), iw.numpy(), ds.numpy(), dd.numpy())
        for key in ("inserted", "deleted", "not_found"):
            assert s1[key] == s2[key], (b, key)
        assert np.array_equal(s1["transitions"], s2["transitions"])
        assert np.array_equal(g.export(), og.dump()) and np.array_equal(g.export_index(), og.index_dump())
        if locate:
            assert g.check_locator()[0] == 0
    # nothing of a rejected batch is applied
    with pytest.raises(Exception):
        g.update(torch.tensor([1, n]), torch.tensor([1, 1]), torch.tensor([1, 1]), torch.tensor([0]), torch.tensor([0]))
    assert np.array_equal(g.export(), og.dump())
    g.close()


@pytest.mark.parametrize("degree", [4095, 4096, 16384, 40001])
@pytest.mark.parametrize("values", [30, 3000, 1 << 17])
def test_streams_on_hubs(degree, values):
    """A hub's chain of records, deletes located for 64 at a time (few destinations: more candidates than
    the table holds; many: deletes that find nothing), inserts deleted again, the last edges deleted."""
    import oracle as O
    import torch
    from paper_2504_10233_amd import Graph
    n = 1 << 17
    src = torch.cat([torch.full((degree,), 9), synth.below(1, 1, 2000, n)])
    dst = synth.below(1, 2, src.numel(), values)
    w = synth.weights_zipf(src.numel(), 1.2, (1 << 30) - 1, 5)
    g = Graph(n, src, dst, w)
    og = O.Graph(n, src.numpy(), dst.numpy(), w.numpy())
    m = 323  # five windows and three records, the hub's records among others
    op = (synth.below(4, 1, m, 5) < 3).to(torch.int64)
    u = torch.where(synth.below(4, 2, m, 8) == 0, synth.below(4, 3, m, n), torch.full((m,), 9))
    v = torch.where(synth.below(4, 4, m, 4) == 0, synth.below(4, 5, m, values), dst[synth.below(4, 6, m, degree)])
    v[:20] = dst[degree - 20:degree].flip(0)
    op[:20], u[:20] = 1, 9
    op[40:80], u[40:80] = torch.arange(40) % 2, 9
    v[41:80:2] = v[40:80:2]  # each insert deleted by the next record, or an older copy is
    ww = synth.weights_zipf(m, 1.2, (1 << 30) - 1, 7)
    s1 = g.update_stream(op, u, v, ww)
    s2 = og.update_stream(op.numpy(), u.numpy(), v.numpy(), ww.numpy())
    for key in ("inserted", "deleted", "not_found"):
        assert s1[key] == s2[key]
    assert np.array_equal(s1["transitions"], s2["transitions"])
    assert np.array_equal(g.export(), og.dump()) and np.array_equal(g.export_index(), og.index_dump())
    g.close()


@pytest.mark.parametrize("degree", [1023, 1024, 1025, 8190, 8191, 8192, 16384, 24577])
def test_sparse_rebuild_around_its_classes(degree):
    """S(u) and the sparse indexes after batches, around the degrees that one wave, one block and chunks rebuild."""
    import oracle as O
    import torch
    from paper_2504_10233_amd import Graph
    n = 50
    src = torch.cat([torch.full((degree,), 7), torch.full((degree // 2,), 8), synth.below(1, 1, 2000, n)])
    dst = synth.below(1, 2, src.numel(), n)
    w = synth.weights_zipf(src.numel(), 1.2, (1 << 30) - 1, 5)
    g = Graph(n, src, dst, w)
    og = O.Graph(n, src.numpy(), dst.numpy(), w.numpy())
    for b in range(3):
        k = 2 + b  # the degree crosses a line by one either way
        ins = (torch.full((k,), 7), synth.below(3 + b, 1, k, n), synth.weights_zipf(k, 1.2, (1 << 30) - 1, 9 + b))
        dels = (torch.full((3,), 7), dst[100 * b:100 * b + 3])
        g.update(*ins, *dels)
        og.update(*(x.numpy() for x in ins + dels))
        assert np.array_equal(g.export(), og.dump()) and np.array_equal(g.export_index(), og.index_dump())
    g.close()


def _philox(ids, step, blk, seed):
    """Words of the streams (seed, ids, step) at block blk; ids and blk broadcast (uint64 arrays)."""
    m32 = np.uint64(0xFFFFFFFF)
    ids, blk = np.broadcast_arrays(np.asarray(ids, np.uint64), np.asarray(blk, np.uint64))
    c = [ids & m32, ids >> np.uint64(32), np.full(ids.shape, step, np.uint64), blk.copy()]
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for _ in range(10):
        a, b = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
        c = [(b >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), b & m32, (a >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), a & m32]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return np.stack(c, -1)


@pytest.mark.parametrize("head", [2, 3])  # words before the first attempt: walk, personalized PageRank
def test_the_last_attempts_of_a_dense_step(head):
    """A dense step ends after 2^16 attempts, in every form alike.  With alpha = 0 a group of two members is
    dense in a vertex of 2^17 edges; walks whose first acceptance is among the last attempts find it."""
    import torch
    from paper_2504_10233_amd import MODE_PER_STEP, Graph
    d, seed = 1 << 17, 91
    dst = torch.full((d,), 2, dtype=torch.int64)
    w = torch.ones(d, dtype=torch.int64)
    hits = (70001, 70002)
    for i in hits:
        w[i], dst[i] = 1 << 20, 1
    # d is a power of two: a word w names the edge w >> 15, and none is drawn again
    accepts = lambda words: ((words >> np.uint64(15)) == hits[0]) | ((words >> np.uint64(15)) == hits[1])
    ids = np.arange(1 << 20, dtype=np.uint64)
    late = accepts(_philox(ids, 0, 1 << 14, seed)[:, :head]).any(1)  # words 2^16 .. of the stream
    W = (1 << 21) + d - 2
    picked = []
    for j in ids[late]:
        words = _philox(j, 0, np.arange(1 << 14, dtype=np.uint64), seed).reshape(-1)
        x = (int(words[head - 2]) << 32) | int(words[head - 1])
        if (x * W) >> 64 >= d - 2 and not accepts(words[head:]).any():
            picked.append(int(j))
    assert len(picked) >= 3
    g = Graph(3, torch.zeros(d, dtype=torch.int64), dst, w, alpha=0)
    for wave in (0, 1, 1 << 31):  # several lanes per walk; wave-served steps; a lane per walk
        g.set_tuning(wave_degree=wave)
        for j in picked[:4]:
            for mode in (0, MODE_PER_STEP):
                if head == 2:
                    assert g.walk(torch.zeros(1, dtype=torch.int32), 1, seed, base=j, mode=mode)[0][0].tolist() == [0, 1]
                else:
                    assert g.ppr(torch.zeros(1, dtype=torch.int32), 1, 0, 1, seed, base=j, mode=mode)[1].tolist() == [0, 1]
    g.close()


def test_the_longest_rows():
    """Walks of 2^32 - 2 steps that end at once: the rest of each row, up to entry 2^32 - 2, is padding."""
    import torch
    from paper_2504_10233_amd import Graph
    L = (1 << 32) - 2
    g = Graph(2, torch.tensor([0]), torch.tensor([1]), torch.tensor([5]))
    out = torch.empty((1, L + 1), dtype=torch.int32, device="cuda")
    for form in ("lanes", "lane", "node2vec", "bad start"):
        out.zero_()
        g.set_tuning(wave_degree=(1 << 31) if form == "lane" else 0)
        start = torch.tensor([2 if form == "bad start" else 0], dtype=torch.int32)
        if form == "node2vec":
            g.node2vec(start, L, 3, 0.5, 2.0, out=out)
        else:
            g.walk(start, L, 3, out=out)
        if form != "bad start":
            assert out[0, :2].tolist() == [0, 1], form
        assert bool((out[0, 2:] == -1).all()), form
    g.close()


@pytest.mark.parametrize("mode", ["int", "plain", "float", "decimal", "alias"])
def test_a_large_hub_equals_the_per_step_form(mode):
    """2^21 + 77 edges at one vertex, whose group choice takes 64-bit sums: groups of every type on ranks past the
    ten and twenty highest, one member or two in some, most of the weight in the decimal group or next to none."""
    import torch
    from paper_2504_10233_amd import MODE_PER_STEP, Graph, quantize_biases
    d, n = (1 << 21) + 77, 5000
    src = torch.cat([torch.zeros(d, dtype=torch.int64), torch.arange(1, n)])
    dst = torch.cat([synth.below(31, 1, d, n), torch.zeros(n - 1, dtype=torch.int64)])
    w = synth.weights_zipf(d + n - 1, 1.5, (1 << 18) - 1, 32)
    w[5], w[9], w[11] = (1 << 31) + 3, 1 << 27, 3 << 26
    kw = {"alias_table": mode == "alias", "adaptive": mode != "plain"}
    if mode in ("float", "decimal"):
        b = synth.uniform_f64(33, 1, d + n - 1) * 0.98 + 0.01
        if mode == "float":
            b += w.clamp(max=1 << 22)
        w = quantize_biases(b.float().cuda(), 1.0, 8)
        kw = {"frac_bits": 8}
    g = Graph(n, src, dst, w, **kw)
    for nw in (3, 3000, 90001):
        starts = synth.below(9, nw, nw, n).to(torch.int32)
        a, sa = g.walk(starts, 7, 77, base=nw)
        b, sb = g.walk(starts, 7, 77, base=nw, mode=MODE_PER_STEP)
        assert torch.equal(a, b) and int(sa) == int(sb), nw
    for ns in (2, 100, 200):  # the last on a lane each, the others on several lanes per walk
        s = synth.below(8, 1, ns, n).to(torch.int32)
        a, b = (g.ppr(s, 1000, int(0.15 * 2**32), 200, 5, mode=m) for m in (0, MODE_PER_STEP))
        assert all(torch.equal(x, y) for x, y in zip(a[:3], b[:3])) and a[3] == b[3]
    a, _ = g.node2vec(starts, 7, 77, 1.0, 1.0, base=nw)
    assert torch.equal(a, g.walk(starts, 7, 77, base=nw)[0])
    g.close()


@pytest.mark.parametrize("mode", ["int", "plain", "float", "alias"])
def test_ppr_around_the_end_of_the_forms_with_several_lanes(mode):
    """163,000 walks on eight lanes each, 165,000 on one (327,680 lanes are resident), equal the per-step form."""
    import torch
    from paper_2504_10233_amd import MODE_PER_STEP
    n, g = _graph(mode)
    for ns in (163, 165, 240):
        src = synth.below(8, ns, ns, n).to(torch.int32)
        a, b = (g.ppr(src, 1000, int(0.15 * 2**32), 200, 5, base=1 << 33, mode=m) for m in (0, MODE_PER_STEP))
        assert all(torch.equal(x, y) for x, y in zip(a[:3], b[:3])) and a[3] == b[3]
    g.close()
