"""GPU parity of the default match layer at the sizes where it can go wrong:
match lengths around its 16-byte items, periods around 16 bytes, sources that
end at or cross a block's or a 32-position record's edge, sources inside
self-overlapping matches, long chains, ragged ends — for archives taken to be
deep (compressed three times and better, or at most 8 MiB) and for others,
each as a whole archive, as a range of it, and in a batch of both.  The bytes
must be the input's (the oracle assembles the containers from the commands)."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
import paper_2608_10188_amd as ax  # noqa: E402

pytestmark = pytest.mark.gpu
LENS = [4, 5, 8, 12, 15, 16, 17, 20, 31, 32, 33, 47, 48, 49, 63, 64, 65, 129, 300, 1500]
PERIODS = [1, 2, 3, 5, 7, 8, 9, 13, 15, 16, 17, 23, 31, 32, 33, 40]


def _say(*a):
    print("[gpu case]", *a, flush=True)


def _archive(n, B, seed, alphabet, content_every):
    """Input and commands: blocks of literals, and every content_every blocks
    one of short literal runs and matches."""
    rng = np.random.default_rng(seed)
    x = alphabet[rng.integers(0, alphabet.size, n)]
    rows, recent = [], []
    for b in range((n + B - 1) // B):
        p, end = b * B, min((b + 1) * B, n)
        if b % content_every or b == 0:
            rows.append((0, p, end - p, 0, 0))
            continue
        while p < end:
            room = end - p
            if room < 4 or rng.random() < 0.25:
                ln = int(min(room, rng.integers(1, 20)))
                rows.append((0, p, ln, 0, 0))
                p += ln
                continue
            ln = int(min(room, LENS[rng.integers(0, len(LENS))]))
            u = rng.random()
            if u < 0.3:  # self-overlapping or close
                src = p - min(p, PERIODS[rng.integers(0, len(PERIODS))])
            elif u < 0.65 and recent:  # at the edges and inside of an earlier match, chains of them
                s, l = recent[-1 - int(rng.integers(0, min(len(recent), 40)))]
                src = s + int(rng.integers(-9, l))
            elif u < 0.85:  # around a block's or a record's edge
                src = int(rng.integers(1, p // 32 + 1)) * 32 if u < 0.75 else int(rng.integers(1, p // B + 1)) * B
                src -= int(rng.integers(1, 40))
            else:
                src = int(rng.integers(0, p))
            src = min(max(src, 0), p - 1)
            per = p - src
            x[p: p + ln] = x[src: src + ln] if per >= ln else np.resize(x[src:p], ln)
            rows.append((1, p, ln, src, 0))
            recent.append((p, ln))
            p += ln
    cmds = np.zeros(len(rows), oracle.CMD_DTYPE)
    r = np.array(rows, np.uint64)
    for k, name in enumerate(("kind", "dst", "len", "src", "rep")):
        cmds[name] = r[:, k]
    arc = oracle.assemble(x, cmds, block_size=B)
    assert np.array_equal(oracle.decode(arc), x)
    return x, arc


BYTES, ONE = np.arange(256, dtype=np.uint8), np.frombuffer(b"AC", np.uint8)
SHAPES = {  # n, block size, alphabet, content blocks' spacing, compressed three times and better
    "small": (40 * 16384 + 77, 16384, BYTES, 2, False),
    "small_4k": (90 * 4096 + 3, 4096, ONE, 2, True),
    "shallow": ((9 << 20) + 5, 16384, BYTES, 12, False),
    "shallow_4k": ((9 << 20) - 4093, 4096, BYTES, 40, False),
    "deep": ((9 << 20) + 13, 16384, ONE, 12, True),
}


@pytest.fixture(scope="module")
def archives():
    return {k: _archive(n, B, 11 + i, al, every) for i, (k, (n, B, al, every, _)) in enumerate(SHAPES.items())}


@pytest.mark.parametrize("shape", list(SHAPES))
def test_whole_and_range(shape, archives):
    x, arc = archives[shape]
    dec = ax.Decoder(arc, torch.from_numpy(arc).cuda())
    assert (dec.info.payload_bytes < x.size // 3) == SHAPES[shape][4]
    out = torch.full((x.size + 64,), 0xCC, dtype=torch.uint8, device="cuda")
    for k in range(2):
        _say(shape, "decode", k)
        dec.decode_all(out=out)
        assert dec.status()[0] == 0
        got = out.cpu().numpy()
        assert np.array_equal(got[: x.size], x), int(np.nonzero(got[: x.size] != x)[0][0])
        assert (got[x.size:] == 0xCC).all(), "bytes past the archive's end were written"
    dec.build_index()
    for off, ln in ((0, x.size), (x.size // 2 - 5, 4099), (x.size - 1, 1)):
        _say(shape, "range", off, ln)
        work = torch.full((dec.range_workspace(off, ln),), 0x5A, dtype=torch.uint8, device="cuda")
        r = torch.full((ln,), 0xCC, dtype=torch.uint8, device="cuda")
        dec.decode_range(off, ln, r, work)
        assert ax.workspace_status(work)[0] == 0
        assert np.array_equal(r.cpu().numpy(), x[off: off + ln]), (off, ln)


def test_batch_of_all(archives):
    xs, decs = [], []
    for name in SHAPES:
        x, arc = archives[name]
        xs.append(x)
        decs.append(ax.Decoder(arc, torch.from_numpy(arc).cuda()))
    outs = [torch.full((x.size,), 0xCC, dtype=torch.uint8, device="cuda") for x in xs]
    batch = ax.Batch(decs, outs)
    _say("batch of", len(xs))
    batch.decode()
    assert batch.status()[0] == 0
    for name, x, o in zip(SHAPES, xs, outs):
        assert np.array_equal(o.cpu().numpy(), x), name


@pytest.mark.parametrize("n_off", [15, 16, 17, 3071, 3072, 3073])
@pytest.mark.parametrize("wide", [False, True])
def test_offset_streams_around_the_stage(n_off, wide):
    """A block whose offset stream has n_off bytes, of one-byte values or (wide)
    of one- and two-byte ones, around a 16-byte piece and around what the parse
    keeps in LDS; decoded matches against the oracle's parse."""
    B = 16384
    rng = np.random.default_rng(n_off)
    x = rng.integers(0, 256, 2 * B).astype(np.uint8)
    rows, p, used = [(0, 0, B, 0, 0)], B, 0
    while used < n_off:
        two = wide and n_off - used >= 2 and rng.random() < 0.5
        src = int(rng.integers(128, B - 8)) if two else int(rng.integers(0, 120))
        x[p: p + 4] = x[src: src + 4]
        rows.append((1, p, 4, src, 0))
        p, used = p + 4, used + (2 if two else 1)
    rows.append((0, p, 2 * B - p, 0, 0))
    arc = oracle.assemble(x, rows)
    assert np.array_equal(oracle.decode(arc), x)
    assert oracle.block_streams(arc, 1)["off"].size == n_off
    dec = ax.Decoder(arc, torch.from_numpy(arc).cuda())
    _say("offset stream", n_off, wide)
    out = dec.decode_all()
    assert dec.status()[0] == 0
    assert np.array_equal(out.cpu().numpy(), x)
    dec.build_index()
    src, dst, ln = dec.tokens(0, len(rows) - 2)
    assert [(int(a), int(b), int(c)) for a, b, c in zip(src, dst, ln)] == [(r[3], r[1], r[2]) for r in rows[1:-1]]


@pytest.mark.parametrize("blocks", [4095, 4096, 5001])
def test_finish_in_one_launch_and_in_eight(blocks):
    """Deep archives around the 16 MiB of positions that are finished run by run."""
    x, arc = _archive(blocks * 4096 - 9, 4096, blocks, ONE, 12)
    dec = ax.Decoder(arc, torch.from_numpy(arc).cuda())
    assert dec.info.payload_bytes < x.size // 3
    _say("finish", blocks)
    out = dec.decode_all()
    assert dec.status()[0] == 0 and np.array_equal(out.cpu().numpy()[: x.size], x)
