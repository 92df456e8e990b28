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
