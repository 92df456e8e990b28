"""GPU parity of the command parse where its forms change: windows of up to
256, up to 768 and more blocks (1024, 512 and 256 commands at a time), blocks
whose command counts lie around those, all four history slots, escaped lengths
and offset streams too long to be staged."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
import paper_2608_10188_amd as ax  # noqa: E402

pytestmark = pytest.mark.gpu
B = 16384
COUNTS = (1, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2048, 2600)


def _block(x, at, count, rng, rows):
    """`count` commands that fill the block at `at`, decoded into x."""
    lens = 4 + rng.multinomial(B - 4 * count, rng.dirichlet(np.full(count, 0.3)))
    kinds = rng.choice(3, count, p=[0.3, 0.45, 0.25])
    hist, p = [1, 2, 3, 4], at
    for ln, kind in zip(lens.tolist(), kinds.tolist()):
        rep = int(rng.integers(0, 4))
        if kind == 2 and hist[rep] <= p:
            hist.insert(0, hist.pop(rep))
            src = p - hist[0]
        elif kind and p:
            kind, rep, src = 1, 0, int(rng.integers(0, p))
            hist = [p - src] + hist[:3]
        else:
            kind, rep, src = 0, 0, 0
            x[p: p + ln] = rng.integers(0, 256, ln)
        if kind:
            x[p: p + ln] = np.resize(x[src: min(p, src + ln)], ln)
        rows.append((kind, p, ln, src, rep))
        p += ln


@pytest.mark.parametrize("blocks", [len(COUNTS), 256, 257, 768, 769])
def test_command_counts_around_the_chunk(blocks):
    print("[gpu case] parse", blocks, flush=True)
    rng = np.random.default_rng(blocks)
    x, rows = np.zeros(blocks * B, np.uint8), []
    for b in range(blocks):
        _block(x, b * B, COUNTS[b] if b < len(COUNTS) else int(rng.integers(2, 20)), rng, rows)
    cmds = np.zeros(len(rows), oracle.CMD_DTYPE)
    for k, name in enumerate(("kind", "dst", "len", "src", "rep")):
        cmds[name] = np.array(rows, np.uint64)[:, k]
    arc = oracle.assemble(x, cmds, block_size=B)
    assert np.array_equal(oracle.decode(arc), x)
    dec = ax.Decoder(arc, torch.from_numpy(arc).cuda())
    for _ in range(2):
        out = dec.decode_all()
        assert dec.status()[0] == 0 and np.array_equal(out.cpu().numpy()[: x.size], x)
