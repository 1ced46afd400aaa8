"""The prefix sum over a count pass's tile counts, which also yields the total
and the list of overflowed tiles: one block, blocks that add up the counts
before them, blocks that read per-block sums, and sums scanned by a block of
their own; parts of several geometries with slabs of different size."""
import json

import numpy as np
import pytest

import oracle
import rkgen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1810_01051_amd as rk
    return rk


# blocks of 4,096 tiles with 2,304-byte (9,216 from 36 MiB on) tiles
@pytest.mark.parametrize("n,blocks", [(0, 0), (100, 1), (2304 * 4096, 1), (2304 * 4096 + 1, 2), (80 << 20, 3),
                                      (1 << 30, 29), (10 << 30, 285)])
@pytest.mark.parametrize("k", [1, 2])
def test_totals_and_overflow_at_every_block_count(rk, n, blocks, k):
    """One byte repeated with plants whose positions are known: with one slab
    slot per tile, tiles of two plants overflow and tiles of one do not; first
    without any overflowed tile."""
    sub = 2304 if (n + 2303) // 2304 < 8192 else 9216 if (n + 2303) // 2304 >= 16384 else 4608
    assert -(-(-(-n // sub)) // 4096) == blocks
    pats = [b"xyzzy", b"qqq"][:k]
    g = rkgen.rng(91, k)
    ctx = rk.Context(0)
    ctx.set_option(rk._lib.RK_OPT_TILE_CFG, 3)
    ctx.set_option(rk._lib.RK_OPT_SLAB_CAP, 1)
    text = torch.full((n,), ord("a"), dtype=torch.uint8, device="cuda:0")
    plan = rk.Plan(ctx, pats, "screen")
    try:
        want = [np.zeros(0, np.int64) for _ in range(k)]
        for rnd in range(2):
            for j, p in enumerate(pats):
                if n < 10000:
                    new = np.array([0, 50] if rnd and n else [], np.int64) + 20 * j
                elif rnd == 0:  # one plant in a tile at most
                    new = np.unique(g.integers(0, n // (2 * 9216) - 1, size=500)) * 2 * 9216 + 9216 * j + 700
                else:           # and some 40 more in tiles from the first to the last
                    at = np.concatenate([g.integers(0, n - 9300, size=5), [0, n - 9216]])
                    new = np.unique(np.concatenate([a + 16 + 64 * np.arange(40) for a in at // 64 * 64]) + 16 * j)
                    new = new[~np.isin(new // 64, np.concatenate(want) // 64)]
                idx = torch.from_numpy(new).to("cuda:0")
                for i, c in enumerate(p):
                    text[idx + i] = c
                want[j] = np.unique(np.concatenate([want[j], new]))
            total = plan.count(text)
            assert total == sum(len(w) for w in want)
            for _ in range(2):  # a second collect after one count
                off, got = plan.collect(text, total)
                off, got = off.cpu().numpy(), got.cpu().numpy()
                for j in range(k):
                    assert got[off[j]:off[j + 1]].tolist() == want[j].tolist(), (rnd, j)
    finally:
        plan.close()
        ctx.close()
        del text
        torch.cuda.empty_cache()


@pytest.mark.parametrize("cap", [0, 1, 3])
@pytest.mark.parametrize("queue", [-1, 0])
def test_batch_of_two_geometries(rk, tmp_path, cap, queue):
    """A table by which one-pattern and 40-pattern instances want different
    geometries: two parts, each with its slabs and overflowed tiles."""
    rows = [{"mode": 2, "mclass": mc, "kclass": kc, "k": 1, "n": 1 << 20, "cfg": c,
             "ms": 1.0 if c == (1 if kc == 0 else 3) else 5.0, "hits": 0, "digest": 0}
            for mc in range(5) for kc in range(4) for c in range(4)]
    path = str(tmp_path / "t.json")
    base = json.load(open(rk.__path__[0] + "/autotune_gfx950.json"))
    with open(path, "w") as f:
        f.write('{"arch": "%s", "n": 1, "timings": [\n], "bucket_timings": [\n' % base["arch"])
        f.write(",\n".join(json.dumps(r) for r in rows))
        f.write('\n], "buckets": [\n], "choice": [\n]}\n')
    g = rkgen.rng(92, cap)
    ctx = rk.Context(0)
    ctx.autotune_load(path)
    ctx.set_option(rk._lib.RK_OPT_QUEUE, queue)
    if cap:
        ctx.set_option(rk._lib.RK_OPT_SLAB_CAP, cap)
    texts, sets = [], []
    for i in range(24):
        n = int(g.integers(1, 200000))
        t = rkgen.iid_text(g, n, rkgen.ACGT)
        texts.append(t)
        sets.append([rkgen.ACGT[g.integers(0, 4, size=int(g.integers(8, 12)))].tobytes()
                     for _ in range(1 if i % 2 else 40)])
    ctx.set_option(rk._lib.RK_OPT_PROFILE, 1)
    plan = rk.BatchPlan(ctx, [torch.from_numpy(t).to("cuda:0") for t in texts], sets, "screen")
    off, pos = plan.search()
    torch.cuda.synchronize()
    assert ctx.profile(0)[0] == 2  # a scan per part
    off, pos = off.cpu().numpy(), pos.cpu().numpy()
    p = 0
    for t, s in zip(texts, sets):
        ro, rp = oracle.search(t, s)
        for j in range(len(s)):
            assert pos[off[p]:off[p + 1]].tolist() == rp[ro[j]:ro[j + 1]].tolist()
            p += 1
    plan.close()
    ctx.close()


@pytest.mark.parametrize("mode", ["screen", "exact"])
@pytest.mark.parametrize("k", [6000, 150000])
@pytest.mark.parametrize("cap", [1, 40])
def test_rescan_of_a_dictionary_of_several_images(rk, mode, k, cap):
    """Dictionaries whose patterns take several images (some few, and more
    than are rescanned image by image), with tiles of every image overflowing
    their slabs and tiles that do not."""
    g = rkgen.rng(93, k % 97)
    text = rkgen.iid_text(g, 60011, rkgen.LOWER)
    text[20000:20200] = ord("q")
    pats = [b"q" * m for m in (1, 5, 9, 14, 17, 33)]
    lens = g.integers(1, 41, size=k)
    at = g.integers(0, len(text) - 41, size=k)
    for j in range(k - len(pats)):
        m = max(4, int(lens[j]))
        pats.append(text[at[j]:at[j] + m].tobytes() if j % 3 else rkgen.LOWER[g.integers(0, 26, size=m)].tobytes())
    ref = oracle.search(text, pats, threads=8)
    ctx = rk.Context(0)
    ctx.set_option(rk._lib.RK_OPT_SLAB_CAP, cap)
    plan = rk.Plan(ctx, pats, mode)
    off, pos = plan.search(torch.from_numpy(text).to("cuda:0"))
    torch.cuda.synchronize()
    assert off.cpu().numpy().astype(np.uint64).tolist() == ref[0].tolist()
    assert (pos.cpu().numpy().astype(np.uint64) == ref[1]).all()
    plan.close()
    ctx.close()


def test_counts_leave_their_stream_idle(rk):
    """Calls that return a value synchronise the stream they are given."""
    ctx = rk.Context(0)
    g = rkgen.rng(87, 0)
    text = torch.from_numpy(rkgen.iid_text(g, 1 << 20, rkgen.LOWER)).to("cuda:0")
    flags = torch.zeros(1 << 20, dtype=torch.uint8, device="cuda:0")
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    for pats in ([b"abcd"], [b"abc", b"de", b"fghijklm"]):
        plan = rk.Plan(ctx, pats, "screen")
        for _ in range(20):
            plan.count(text, stream=stream)
            assert stream.query()
            assert ctx.paper_positions(flags, stream=stream).numel() == 0
            assert stream.query()
        plan.close()
    ctx.close()
