"""GPU decodes by the match layer's two schedules: which one the options select,
and the level-synchronous one wherever a decode can run it, with parity against
the input (every archive's oracle decode is)."""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
import paper_2608_10188_amd as ax  # noqa: E402

pytestmark = pytest.mark.gpu


def _say(*a):
    print("[gpu case]", *a, flush=True)


def _make(kind, n, seed, **kw):
    arc = ax.encode(synth.GENERATORS[kind](n, seed), threads=8, **kw)
    return arc, oracle.decode(arc)


@pytest.fixture(scope="module")
def text():
    return _make("text", 3 << 20, 81)


def _decoder(arc, opts=()):
    d = ax.Decoder(arc, torch.from_numpy(arc).cuda())
    for k, v in opts:
        d.set_option(k, v)
    return d


POISON = 0x5A


def _whole(text, opts, mode=ax.COPY_PERIODIC):
    """The bytes of the workspace that a decode with these options wrote."""
    arc, x = text
    d = _decoder(arc, opts)
    work = torch.full((d.workspace_bytes,), POISON, dtype=torch.uint8, device="cuda")
    out = torch.full((x.size,), 0xCC, dtype=torch.uint8, device="cuda")
    d.decode_all(out=out, work=work, copy_mode=mode)
    assert d.status(work=work)[0] == 0
    assert np.array_equal(out.cpu().numpy(), x), opts
    return work != POISON


def _range(text, opts):
    arc, x = text
    d = _decoder(arc, opts)
    d.build_index()
    off, ln = x.size // 2, 300000
    work = torch.full((d.range_workspace(off, ln),), POISON, dtype=torch.uint8, device="cuda")
    out = torch.full((ln,), 0xCC, dtype=torch.uint8, device="cuda")
    d.decode_range(off, ln, out, work)
    assert ax.workspace_status(work)[0] == 0
    assert np.array_equal(out.cpu().numpy(), x[off: off + ln]), opts
    return work != POISON


class _Rounds:
    """Tells the schedules apart: the rounds keep state of every match (a block
    index and a state byte at least) where the other schedule writes nothing."""

    def __init__(self, decode):
        self.decode = decode
        self.only = decode([(ax.OPT_BULK_ROUNDS, 5)]) & ~decode([])
        self.bytes = int(self.only.sum())

    def __call__(self, opts, **kw):
        share = int((self.decode(opts, **kw) & self.only).sum()) / self.bytes
        assert share < 0.05 or share > 0.25, (opts, share)
        return share > 0.25


KNOBS = [(ax.OPT_BULK_ROUNDS, 4), (ax.OPT_FILL_ROUNDS, 0), (ax.OPT_FILL_TAIL, 0), (ax.OPT_TAIL_CHUNKS, 1),
         (ax.OPT_ROUND0_TILE, 1), (ax.OPT_TAIL_MODE, ax.TAIL_JUMP), (ax.OPT_JUMP_PASSES, 0)]
ROOTS, ROUNDS = (ax.OPT_SCHEDULE, ax.SCHEDULE_ROOTS), (ax.OPT_SCHEDULE, ax.SCHEDULE_ROUNDS)


def test_knobs_select_the_rounds_whatever_their_value(text):
    _say("schedules of whole decodes")
    rounds = _Rounds(lambda opts, **kw: _whole(text, opts, **kw))
    assert rounds.bytes > 5 * int(ax.read_info(text[0]).n_matches)
    assert not rounds([(ax.OPT_GRAPH, 0)])
    assert rounds([], mode=ax.COPY_SERIAL) and rounds([ROOTS], mode=ax.COPY_SERIAL)
    for k in KNOBS:
        assert rounds([k]), k
        assert not rounds([k, ROOTS]), k
    assert not rounds([(ax.OPT_RANGE_JUMP_TOKENS, 4096)])  # a knob of range decodes
    assert rounds([ROUNDS])
    with pytest.raises(ax.AceapexError):
        _decoder(text[0], [(ax.OPT_SCHEDULE, 3)])


def test_knobs_select_the_rounds_of_range_decodes(text):
    _say("schedules of range decodes")
    rounds = _Rounds(lambda opts: _range(text, opts))
    for k in KNOBS + [(ax.OPT_RANGE_JUMP_TOKENS, 4096), ROUNDS]:
        assert rounds([k]), k
    assert not rounds([(ax.OPT_RANGE_JUMP_TOKENS, 0), ROOTS])


# ------------------------------------------------- the rounds, everywhere --

CONFIGS = {
    "learned": [ROUNDS],
    "learned-waves": [ROUNDS, (ax.OPT_ROUND0_TILE, 0)],
    "one": [(ax.OPT_BULK_ROUNDS, 1)],
    "four": [(ax.OPT_BULK_ROUNDS, 4)],
    "five-waves-fill": [(ax.OPT_BULK_ROUNDS, 5), (ax.OPT_ROUND0_TILE, 0), (ax.OPT_FILL_ROUNDS, 1)],
    "chase": [(ax.OPT_TAIL_MODE, ax.TAIL_CHASE), (ax.OPT_TAIL_CHUNKS, 2), (ax.OPT_FILL_TAIL, 1)],
    "two-passes": [(ax.OPT_BULK_ROUNDS, 2), (ax.OPT_JUMP_PASSES, 2)],
}


def _long_chains():
    """Blocks of a 300-byte match of the block before's and a long periodic
    fill: long tokens in the remainder, whatever the number of rounds."""
    rng, B, nb = np.random.default_rng(82), 16384, 40
    data = rng.integers(0, 256, nb * B, dtype=np.uint8)
    cmds, prev = [(0, 0, B, 0, 0)], 0
    for b in range(1, nb):
        s, h, p = b * B, 5 + 3 * b, (1, 7, 64, 255, 256, 300)[b % 6]
        a, f, ln = s + h, s + h + 300, 2000 + 37 * b
        data[a: f] = data[prev: prev + 300]
        data[f: f + ln] = np.resize(data[f - p: f], ln)
        cmds += [(0, s, h, 0, 0), (1, a, 300, prev, 0), (1, f, ln, f - p, 0), (0, f + ln, s + B - f - ln, 0, 0)]
        prev = a
    arc = oracle.assemble(data, cmds)
    return arc, oracle.decode(arc)


@pytest.fixture(scope="module")
def archives(text):
    return {"text": text, "dna": _make("dna", (2 << 20) + 77, 83), "chains": _long_chains(),
            "dna_4k": _make("dna", 700001, 84, block_size=4096), "empty": _make("dna", 0, 85),
            "one": _make("text", 1, 86)}


@pytest.mark.parametrize("config", list(CONFIGS))
def test_rounds_of_repeated_decodes(archives, config):
    """Decodes after the first run the round and pass counts it reported."""
    for name, (arc, x) in archives.items():
        d = _decoder(arc, CONFIGS[config])
        out = torch.empty((x.size + 16,), dtype=torch.uint8, device="cuda")
        for k in range(4):
            out.fill_(0xCC)
            _say(name, config, "decode", k)
            d.decode_all(out=out)
            assert d.status()[0] == 0
            got = out.cpu().numpy()
            assert np.array_equal(got[: x.size], x) and (got[x.size:] == 0xCC).all(), (name, k)


RANGES = [(0, 1), (16384 - 3, 6), (300001, 70001), (1 << 20, 5), (1234567, 16384), (5, 40000), (1 << 19, 2 << 14),
          (2000000, 3), (77, 1000)]


@pytest.mark.parametrize("config", list(CONFIGS) + ["jump-all", "jump-none", "serial"])
def test_rounds_of_range_decodes(archives, config):
    opts = {"jump-all": [(ax.OPT_RANGE_JUMP_TOKENS, 0)], "jump-none": [(ax.OPT_RANGE_JUMP_TOKENS, 1 << 20)],
            "serial": []}.get(config) or CONFIGS.get(config, [])
    mode = ax.COPY_SERIAL if config == "serial" else ax.COPY_PERIODIC
    for name in ("text", "dna"):
        arc, x = archives[name]
        d = _decoder(arc, opts)
        d.build_index()
        rp = ax.RangePlan(d, max_blocks=256, max_tokens=1 << 18)
        work = torch.full((rp.workspace_bytes,), POISON, dtype=torch.uint8, device="cuda")
        for part in (RANGES, RANGES[2:4], RANGES[:1], RANGES):  # closures of different sizes in one plan
            outs = [torch.full((ln,), 0xCC, dtype=torch.uint8, device="cuda") for _, ln in part]
            _say(name, config, "ranges", len(part))
            rp.decode([o for o, _ in part], [ln for _, ln in part], outs, work, copy_mode=mode)
            assert ax.workspace_status(work)[0] == 0
            for (off, ln), o in zip(part, outs):
                assert np.array_equal(o.cpu().numpy(), x[off: off + ln]), (name, off, ln)
        if mode == ax.COPY_SERIAL:
            continue
        for off, ln in RANGES[2:5]:
            w = torch.full((d.range_workspace(off, ln),), POISON, dtype=torch.uint8, device="cuda")
            out = torch.full((ln,), 0xCC, dtype=torch.uint8, device="cuda")
            _say(name, config, "range", off, ln)
            d.decode_range(off, ln, out, w)
            assert ax.workspace_status(w)[0] == 0
            assert np.array_equal(out.cpu().numpy(), x[off: off + ln]), (name, off, ln)


@pytest.mark.parametrize("config", list(CONFIGS) + ["serial"])
@pytest.mark.parametrize("graph", [0, 1])
def test_rounds_of_batches(archives, config, graph):
    """Batches, also replayed from a graph, with other work and a
    synchronization between the replays."""
    mode = ax.COPY_SERIAL if config == "serial" else ax.COPY_PERIODIC
    decs = [_decoder(arc) for arc, _ in archives.values()]
    outs = [torch.empty((x.size + 16,), dtype=torch.uint8, device="cuda") for _, x in archives.values()]
    bt = ax.Batch(decs, outs)
    for k, v in CONFIGS.get(config, []):
        bt.set_option(k, v)
    bt.set_option(ax.OPT_GRAPH, graph)
    for k in range(4):
        for o in outs:
            o.fill_(0xCC)
        torch.cuda.synchronize()
        _say("batch", config, "graph", graph, "decode", k)
        bt.decode(copy_mode=mode)
        assert bt.status()[0] == 0
        for (name, (_, x)), o in zip(archives.items(), outs):
            got = o.cpu().numpy()
            assert np.array_equal(got[: x.size], x) and (got[x.size:] == 0xCC).all(), (name, k)
