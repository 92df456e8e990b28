"""GPU decode of archives above 8 MiB by what their ratio comes from: the entropy
coder (few bytes copied, the blocks are walked), matches (marked), or repeats of
a block's own bytes (walked again), and on either side of the share of copied
bytes at which the decoder changes from one to the other.  Each as a whole
archive, as a range of it, and in a batch with archives of every kind.  The bytes
must be the input's (the oracle's decode of every archive is), and archives that
the ratio alone gets wrong must not take longer than the level-synchronous
schedule takes over them."""
import numpy as np
import pytest

import oracle
import shaped_archive
import synth

torch = pytest.importorskip("torch")
import paper_2608_10188_amd as ax  # noqa: E402

pytestmark = pytest.mark.gpu
N = 9 << 20
ACGT = np.frombuffer(b"ACGT", np.uint8)


def _say(*a):
    print("[gpu case]", *a, flush=True)


def _uniform(n, seed):
    return ACGT[np.random.default_rng(seed).integers(0, 4, n)]


def _with_text(share):
    """uniform ACGT with a share of 64 KiB pieces of text, whose bytes are nearly all copies"""
    rng = np.random.default_rng(5)
    pick = np.zeros(N >> 16, bool)
    pick[: int(share * pick.size)] = True
    rng.shuffle(pick)
    return np.where(np.repeat(pick, 1 << 16), synth.text(N, 6), _uniform(N, 7))


def _noisy(n):
    """text with every twentieth byte replaced: chains at a ratio below three"""
    rng = np.random.default_rng(11)
    x, k = synth.text(n, 12), rng.random(n) < 0.05
    x[k] = rng.integers(0, 256, int(k.sum()), dtype=np.uint8)
    return ax.encode(x, threads=8)


def _pages(block):
    x = np.random.default_rng(8).integers(0, 256, N, dtype=np.uint8).reshape(-1, 4096)
    x[np.random.default_rng(9).random(x.shape[0]) < 0.75] = 0
    return ax.encode(x.reshape(-1)[:-5], threads=8, block_size=block)


def _literals_only(n):
    """zeros as literals but for a few matches"""
    return ax.encode(np.zeros(n, np.uint8), threads=8, depth_cap=1)


def _shaped(every):
    x, cmds = shaped_archive.build(N + 77, 10, every=every)
    return oracle.assemble(x, cmds)


KINDS = {
    "uniform": lambda: ax.encode(_uniform(N + 3, 1), threads=8),
    "copies_18": lambda: ax.encode(_with_text(0.12), threads=8),
    "copies_30": lambda: ax.encode(_with_text(0.28), threads=8),
    "copies_34": lambda: ax.encode(_with_text(0.34), threads=8),
    "copies_47": lambda: ax.encode(_with_text(0.5), threads=8),
    "pages": lambda: _pages(16384),
    "pages_4k": lambda: _pages(4096),
    "zeros": lambda: ax.encode(np.zeros(N + 1, np.uint8), threads=8),
    "literals": lambda: _literals_only(N - 1),
    "constant_blocks": lambda: _shaped(1 << 30),
    "shaped": lambda: _shaped(32),
    "noisy": lambda: _noisy(N + 5),
    "text": lambda: ax.encode(synth.text(N - 9, 2), threads=8),
    "dna": lambda: ax.encode(synth.dna(2 << 20, 3), threads=8),
}
_made = {}


def _archive(kind):
    if kind not in _made:
        arc = KINDS[kind]()
        _made[kind] = (arc, oracle.decode(arc))
    return _made[kind]


def _same(got, x):
    assert np.array_equal(got[: x.size], x), int(np.nonzero(got[: x.size] != x)[0][0])
    assert (got[x.size:] == 0xCC).all(), "bytes past the archive's end were written"


@pytest.mark.parametrize("kind", [k for k in KINDS if k != "dna"])
def test_whole_and_range(kind):
    arc, x = _archive(kind)
    dec = ax.Decoder(arc, torch.from_numpy(arc).cuda())
    assert x.size > 8 << 20 and (dec.info.payload_bytes < x.size // 3) == (kind != "noisy")
    out = torch.full((x.size + 64,), 0xCC, dtype=torch.uint8, device="cuda")
    work = torch.full((dec.workspace_bytes,), 0x5A, dtype=torch.uint8, device="cuda")
    for k in range(2):
        _say(kind, "decode", k)
        dec.decode_all(out=out, work=work)
        assert dec.status(work=work)[0] == 0
        _same(out.cpu().numpy(), x)
    dec.build_index()
    for off, ln in ((0, x.size), (x.size // 2 - 5, 70001)):
        _say(kind, "range", off, ln)
        work = torch.full((dec.range_workspace(off, ln),), 0x5A, dtype=torch.uint8, device="cuda")
        r = torch.full((ln,), 0xCC, dtype=torch.uint8, device="cuda")
        dec.decode_range(off, ln, r, work)
        assert ax.workspace_status(work)[0] == 0
        assert np.array_equal(r.cpu().numpy(), x[off: off + ln]), (off, ln)


@pytest.mark.parametrize("kinds", [("uniform", "dna"), ("zeros", "dna"), ("uniform", "zeros", "text", "dna"),
                                   ("text", "uniform"), tuple(KINDS)])
def test_batches_of_kinds(kinds):
    """deep, undecided and other archives in one window, replayed from a graph
    with other work and a synchronization between the replays"""
    made = [_archive(k) for k in kinds]
    decs = [ax.Decoder(arc, torch.from_numpy(arc).cuda()) for arc, _ in made]
    outs = [torch.full((x.size + 16,), 0xCC, dtype=torch.uint8, device="cuda") for _, x in made]
    batch = ax.Batch(decs, outs)
    for graph in (0, 1):
        batch.set_option(ax.OPT_GRAPH, graph)
        for k in range(3):
            for o in outs:
                o.fill_(0xCC)
            torch.cuda.synchronize()
            _say("batch", kinds, "graph", graph, k)
            batch.decode()
            assert batch.status()[0] == 0
            for (_, x), o in zip(made, outs):
                _same(o.cpu().numpy(), x)


@pytest.mark.parametrize("sizes", [(17 << 20, 100000), (17 << 20, 17 << 20), (17 << 20, 8 << 20, 8 << 20),
                                   (17 << 20, 9 << 20, 9 << 20)])
def test_finish_of_a_batch(sizes):
    """One archive with more than half of the marked blocks, with half of them
    and with fewer: finished in eight launches and in one."""
    xs = [synth.text(n, 40 + i) for i, n in enumerate(sizes)]
    arcs = [ax.encode(x, threads=8) for x in xs]
    assert all(np.array_equal(oracle.decode(a), x) for a, x in zip(arcs, xs))
    decs = [ax.Decoder(a, torch.from_numpy(a).cuda()) for a in arcs]
    outs = [torch.full((x.size + 16,), 0xCC, dtype=torch.uint8, device="cuda") for x in xs]
    batch = ax.Batch(decs, outs)
    _say("finish of a batch", sizes)
    batch.decode()
    assert batch.status()[0] == 0
    for x, o in zip(xs, outs):
        _same(o.cpu().numpy(), x)


def _fastest(dec, out, n=8):
    ms = []
    for _ in range(n):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        a.record()
        dec.decode_all(out=out)
        b.record()
        torch.cuda.synchronize()
        ms.append(a.elapsed_time(b))
    return min(ms)


@pytest.mark.parametrize("kind", ["uniform", "literals", "noisy"])
def test_ratio_is_not_depth(kind):
    n = 64 << 20
    arc = {"uniform": lambda: ax.encode(_uniform(n, 4), threads=16), "literals": lambda: _literals_only(n),
           "noisy": lambda: _noisy(n)}[kind]()
    x = oracle.decode(arc)
    out = torch.full((n,), 0xCC, dtype=torch.uint8, device="cuda")
    ms = []
    for rounds in (0, 1, 5):  # 0: the default schedule
        d = ax.Decoder(arc, torch.from_numpy(arc).cuda())
        if rounds:
            d.set_option(ax.OPT_BULK_ROUNDS, rounds)
        for _ in range(4):
            out.fill_(0xCC)
            d.decode_all(out=out)
            assert d.status()[0] == 0
        assert np.array_equal(out.cpu().numpy(), x)
        ms.append(_fastest(d, out))
    _say(kind, "ms", ms)
    assert ms[0] <= 1.1 * min(ms[1:])  # runs of one build differ by a few percent
