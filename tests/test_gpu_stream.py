"""Streamed searches of texts in host memory and in files (rk_search_host,
rk_search_file) against the oracle: occurrences planted across piece
boundaries, short and long patterns, both modes, piece sizes down to the
minimum, and the degenerate texts."""
import numpy as np
import pytest

import oracle
import rkgen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

MODES = ["screen", "exact"]


@pytest.fixture(scope="module")
def rk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1810_01051_amd as rk
    return rk


@pytest.fixture(scope="module")
def ctx(rk):
    c = rk.Context(0)
    yield c
    c.close()


def planted_text(seed, n, pats, piece):
    g = rkgen.rng(90, seed)
    text = rkgen.iid_text(g, n, rkgen.ACGT)
    mmax = max(len(p) for p in pats)
    L = ((piece + 15) // 16 * 16) - (mmax - 1)
    for p in pats:
        m = len(p)
        for b in range(L, n, L):
            for d in (-m, -m + 1, -1, 0, 1):
                x = b + d
                if 0 <= x <= n - m:
                    text[x:x + m] = np.frombuffer(p, np.uint8)
    return text


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("piece", [1 << 16, (1 << 18) + 5, 1 << 20])
def test_host_text_pieces(ctx, rk, mode, piece):
    g = rkgen.rng(91, piece)
    pats = [rkgen.ACGT[g.integers(0, 4, size=m)].tobytes() for m in (1, 7, 32, 64, 65, 300, 1024)]
    n = 6 * (1 << 20) + 123
    text = planted_text(piece, n, pats, piece)
    pats.append(text[5000:5016].tobytes())
    plan = rk.Plan(ctx, pats, mode)
    off, pos = plan.search_host(text, piece)
    plan.close()
    ro, rp = oracle.search(text, pats, threads=4)
    assert int(ro[-1]) > 100
    assert off.tolist() == ro.tolist()
    assert pos.tolist() == rp.tolist()


@pytest.mark.parametrize("mode", MODES)
def test_file_text(ctx, rk, mode, tmp_path):
    g = rkgen.rng(92, 0)
    pats = [b"ACGTACGTAC", rkgen.ACGT[g.integers(0, 4, size=200)].tobytes(), b"A"]
    text = planted_text(7, 3 * (1 << 20) + 17, pats, 1 << 18)
    path = tmp_path / "text.bin"
    path.write_bytes(text.tobytes())
    plan = rk.Plan(ctx, pats, mode)
    off, pos = plan.search_host(str(path), 1 << 18)
    plan.close()
    ro, rp = oracle.search(text, pats, threads=4)
    assert off.tolist() == ro.tolist() and pos.tolist() == rp.tolist()


def test_stream_edges(ctx, rk):
    plan = rk.Plan(ctx, [b"abc", b"b"], "screen")
    for text in (b"", b"ab", b"abc", b"xabcabc" * 20000):
        off, pos = plan.search_host(np.frombuffer(text, np.uint8), 1 << 16)
        ro, rp = oracle.search(text, [b"abc", b"b"])
        assert off.tolist() == ro.tolist() and pos.tolist() == rp.tolist(), len(text)
    with pytest.raises(rk._lib.RkError) as e:
        plan.search_host(np.zeros(10, np.uint8), 1000)
    assert e.value.status == rk._lib.RK_EINVAL
    plan.close()


@pytest.mark.parametrize("n,piece", [((2 << 20) - 1, 256 << 20), (2 << 20, 256 << 20), ((2 << 20) + 1, 1 << 30),
                                     ((70 << 20) + 11, 3 << 20), ((70 << 20) + 11, 128 << 20),
                                     (2 * (3 << 20) - 30, 3 << 20), (5 << 20, 1 << 16)])
def test_staging_ring_chunk_edges(ctx, rk, n, piece):
    """Texts of one chunk of the staging ring, of just more, of more chunks
    than the ring has slots, pieces of a broken number of chunks, and a last
    piece that lies in its predecessor's overlap but for some bytes; twice,
    as the ring outlives a call."""
    pats = [b"ACGTTGCAACGGTACC", b"TTTTTTTTTTTT", rkgen.ACGT[rkgen.rng(93, 0).integers(0, 4, size=64)].tobytes()]
    if piece < n:
        text = planted_text(n % 97, n, pats, piece)
    else:
        text = rkgen.iid_text(rkgen.rng(93, 1), n, rkgen.ACGT)
        for x in (0, (2 << 20) - 20, n - 64):
            text[x:x + len(pats[x % 2])] = np.frombuffer(pats[x % 2], np.uint8)[:n - x]
    ro, rp = oracle.search(text, pats, threads=8)
    plan = rk.Plan(ctx, pats, "screen")
    for _ in range(2):
        off, pos = plan.search_host(text, piece)
        assert off.tolist() == ro.tolist() and pos.tolist() == rp.tolist()
    plan.close()


def test_streamed_searches_of_two_threads(rk):
    """A context, and so a ring, per thread."""
    import threading
    pats = [b"ACGTACGTAC", b"GGGGGGGG"]
    texts = [rkgen.iid_text(rkgen.rng(94, i), (9 << 20) + i, rkgen.ACGT) for i in range(2)]
    want = [oracle.search(t, pats, threads=4) for t in texts]
    bad = []

    def work(i):
        c = rk.Context(0)
        plan = rk.Plan(c, pats, "screen")
        for _ in range(4):
            off, pos = plan.search_host(texts[i], 4 << 20)
            if off.tolist() != want[i][0].tolist() or pos.tolist() != want[i][1].tolist():
                bad.append(i)
        plan.close()
        c.close()

    th = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert not bad


@pytest.mark.parametrize("source", ["memory", "file"])
@pytest.mark.parametrize("n,piece", [
    ((8 << 20) - 1, 256 << 20), (8 << 20, 256 << 20), ((8 << 20) + 1, 256 << 20),
    # three and more pieces of three chunks, the last of 4 MiB and 16 bytes
    ((70 << 20) + 11, (20 << 20) + 16),
    # a whole number of chunks per piece
    (3 * (16 << 20) + 5, 16 << 20),
    # the piece before the last one is cut by the text's end: its last chunk of 16 bytes is empty
    ((16 << 20) + 16 - 63 + (16 << 20) - 10, (16 << 20) + 16),
    # and a first piece that is
    ((16 << 20) - 20, (16 << 20) + 16)])
def test_staging_ring_pieces_of_several_chunks(ctx, rk, tmp_path, source, n, piece):
    """Chunks of 8 MiB: texts at a chunk's edges, pieces of several chunks and
    texts of several such pieces, hits at the seams of chunks and pieces; twice,
    as the ring outlives a call."""
    pats = [b"ACGTTGCAACGGTACC", b"TTTTTTTTTTTT", rkgen.ACGT[rkgen.rng(95, 0).integers(0, 4, size=64)].tobytes()]
    text = rkgen.iid_text(rkgen.rng(95, n % 97), n, rkgen.ACGT)
    L = piece - 63
    seams = [b + c for b in range(0, n, L) for c in range(0, piece, 8 << 20)] + list(range(L, n, L)) + [n]
    for i, s in enumerate(seams):
        for j, d in enumerate((-130, -20, 40)):
            p = pats[(i + j) % 3]
            if 0 <= s + d <= n - len(p):
                text[s + d:s + d + len(p)] = np.frombuffer(p, np.uint8)
    ro, rp = oracle.search(text, pats, threads=8)
    if source == "file":
        path = tmp_path / "text.bin"
        path.write_bytes(text.tobytes())
        text = str(path)
    plan = rk.Plan(ctx, pats, "screen")
    for _ in range(2):
        off, pos = plan.search_host(text, piece)
        assert off.tolist() == ro.tolist() and pos.tolist() == rp.tolist()
    plan.close()
