"""GPU decode of archives whose matches copy from just behind: rows of a few
bytes, each a copy of the row before but for its first bytes, so that a byte's
chain is as long as the archive and its hops as short as a row.  The bytes must
be the input's (the oracle assembles the containers from the commands), and the
default match layer must not take longer over the short hops than the
level-synchronous schedule does, whose pointer jumping needs a number of passes
that is logarithmic in the chain's length."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
import paper_2608_10188_amd as ax  # noqa: E402

pytestmark = pytest.mark.gpu


def _say(*a):
    print("[gpu case]", *a, flush=True)


def _rows(n, w, lit, seed):
    """n bytes in rows of w: lit literal bytes, then the row before's."""
    rng = np.random.default_rng(seed)
    nr = n // w
    x = np.empty((nr, w), np.uint8)
    x[:] = rng.integers(0, 256, w).astype(np.uint8)
    x[:, :lit] = rng.integers(0, 256, (nr, lit))
    cmds = np.zeros(2 * nr, oracle.CMD_DTYPE)
    p = np.arange(nr, dtype=np.uint64) * w
    cmds["dst"][0::2], cmds["len"][0::2] = p, lit
    cmds["dst"][1::2], cmds["len"][1::2], cmds["kind"][1::2] = p + lit, w - lit, 1
    cmds["src"][1::2] = p + lit - np.uint64(w)
    cmds["kind"][1], cmds["src"][1] = 0, 0  # the first row has none before it
    arc = oracle.assemble(x.reshape(-1), cmds)
    assert np.array_equal(oracle.decode(arc), x.reshape(-1))
    return x.reshape(-1), arc


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


# every byte has an entry (at most 8 MiB; larger with long matches), or those of unfinished walks have
@pytest.mark.parametrize("n,w,lit,timed", [((4 << 20) - 48, 16, 4, True), ((4 << 20) - 8, 8, 4, True),
                                           ((12 << 20) + 64, 64, 4, False), ((12 << 20) - 64, 64, 24, False),
                                           ((32 << 20) - 16, 16, 4, True)])
def test_chains_of_short_hops(n, w, lit, timed):
    x, arc = _rows(n, w, lit, 31)
    dec = ax.Decoder(arc, torch.from_numpy(arc).cuda())
    out = torch.full((x.size + 64,), 0xCC, dtype=torch.uint8, device="cuda")
    for k in range(3):
        _say("rows", n, w, lit, "decode", k)
        dec.decode_all(out=out)
        assert dec.status()[0] == 0
        got = out.cpu().numpy()
        assert np.array_equal(got[: x.size], x), int(np.nonzero(got[: x.size] != x)[0][0])
        assert (got[x.size:] == 0xCC).all(), "bytes past the archive's end were written"
    if not timed:
        return
    ms = _fastest(dec, out)
    rounds = ax.Decoder(arc, torch.from_numpy(arc).cuda())
    rounds.set_option(ax.OPT_BULK_ROUNDS, 1)  # straight to pointer jumping
    for _ in range(4):  # it learns its pass count
        rounds.decode_all(out=out)
        assert rounds.status()[0] == 0
    assert np.array_equal(out.cpu().numpy()[: x.size], x)
    ref = _fastest(rounds, out)
    _say("rows", n, w, lit, "ms", ms, "rounds", ref)
    assert ms <= 1.1 * ref  # runs of one build differ by a few percent
