"""GPU parity of the entropy stage where its forms change: alphabets around 64
present symbols (entries addressed by rank or by byte offset) and up to 256,
stream lengths around whole groups of four steps for one to 64 lanes."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
import paper_2608_10188_amd as ax  # noqa: E402

pytestmark = pytest.mark.gpu
B = 16384


@pytest.mark.parametrize("spread", [32, 128])
@pytest.mark.parametrize("symbols", [2, 3, 33, 63, 64, 65, 255, 256])
def test_literal_streams(symbols, spread):
    """One block per length, a single literal run each: the decoded literal
    stream is the block."""
    print("[gpu case] entropy", symbols, spread, flush=True)
    rng = np.random.default_rng(symbols * 1000 + spread)
    alphabet = np.sort(rng.permutation(256)[:symbols]).astype(np.uint8)
    p = 0.9 ** np.arange(symbols) + 1e-3  # skewed, every symbol present in a long stream
    p /= p.sum()
    x = alphabet[rng.choice(symbols, 40 * B, p=p)]
    x[: symbols] = alphabet
    arc, _ = oracle.encode(x, min_match=255, rans_min_syms_per_lane=spread)
    dec = ax.Decoder(arc, torch.from_numpy(arc).cuda())
    for b, got in enumerate(dec.streams(0, int(dec.info.n_blocks))):
        want = oracle.block_streams(arc, b)
        for k in ("lit", "len", "off", "cmd"):
            assert np.array_equal(got[k], want[k]), (symbols, spread, b, k)


@pytest.mark.parametrize("spread", [32, 128])
def test_stream_lengths(spread):
    """A ragged last block of every length in turn, so that the literal stream
    runs with 1 to 64 lanes and ends anywhere in a group of four steps."""
    rng = np.random.default_rng(spread)
    lens = sorted({k * spread * (1 << j) // 4 + d for j in range(7) for k in (4, 5, 7) for d in (-1, 0, 1, 5)} |
                  {1, 2, 3, 31, 33, 16383, 16384})
    for n in (v for v in lens if 1 <= v <= B):
        x = (rng.integers(0, 6, n) * rng.integers(0, 2, n) + 65).astype(np.uint8)
        arc = oracle.assemble(x, [(0, 0, n, 0, 0)], rans_min_syms_per_lane=spread)
        print("[gpu case] entropy length", n, spread, flush=True)
        dec = ax.Decoder(arc, torch.from_numpy(arc).cuda())
        assert np.array_equal(dec.streams(0, 1)[0]["lit"], x), n
        out = dec.decode_all()
        assert dec.status()[0] == 0 and np.array_equal(out.cpu().numpy()[:n], x), n


@pytest.mark.parametrize("blocks", [512, 513])
@pytest.mark.parametrize("symbols", [64, 65, 256])
def test_windows_around_the_wide_tables(symbols, blocks):
    """Windows of up to 512 blocks decode from per-slot entries, larger ones by rank."""
    print("[gpu case] entropy window", symbols, blocks, flush=True)
    rng = np.random.default_rng(symbols + blocks)
    p = 0.95 ** np.arange(symbols) + 1e-3
    x = rng.permutation(256)[:symbols].astype(np.uint8)[rng.choice(symbols, blocks * 4096 - 7, p=p / p.sum())]
    arc, _ = oracle.encode(x, block_size=4096, min_match=255)
    dec = ax.Decoder(arc, torch.from_numpy(arc).cuda())
    assert int(dec.info.n_blocks) == blocks
    out = dec.decode_all()
    assert dec.status()[0] == 0 and np.array_equal(out.cpu().numpy()[: x.size], x)
    for b, got in zip((0, blocks - 1), (dec.streams(0, 1)[0], dec.streams(blocks - 1, 1)[0])):
        assert np.array_equal(got["lit"], oracle.block_streams(arc, b)["lit"])
