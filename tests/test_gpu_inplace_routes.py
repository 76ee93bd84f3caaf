"""In-place realignments over long spans by the route that they take.

A span is D*cap elements; the sizes are in 16-byte vectors (one a column at D = 8).
Spans of more than 8192 vectors go, by their number (L*2*B*H) and the entry point:

* ``few``: at most 128 spans of 32768 vectors or more, chunks of 4096 vectors;
* ``table``: a greedy step's walk in the order that verification writes into the
  workspace, the rows one at a time or 32 at a time;
* ``sorted``: a realignment alone of at most 8192 spans and 64 rows, a walk whose
  waves order the rows; ``chunks``: the same of more than 64 rows;
* ``cache``: a realignment alone of more than 8192 spans.

A greedy step's workspace shows which of them wrote and read an order table: the
table's rows are checked one by one, and elsewhere its place is untouched."""
import numpy as np
import pytest
import torch

import oracle
from paper_2510_22876_amd import workloads as wl
from tests.gpu_util import (PAD_ID, alloc_outputs, bits, check_kv_full_vs_oracle, check_posmask_vs_oracle,
                            check_relocation_on_device, check_tokens_vs_oracle, check_verify_vs_oracle, i16, run_gpu, say)

pytestmark = pytest.mark.gpu

SENT = 0x3C3C3C3C


@pytest.fixture(scope="module", autouse=True)
def _lib():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    yield
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


def _case(W_in, ns, H, L=1, D=8, k=5, accept=("uniform",)):
    return wl.Workload("route", B=len(ns), k=k, V=40, logit_dtype="f32", logit_std=1.0, L=L, H=H, D=D,
                       prompt=("list", [int(n) for n in ns]), accept=accept, W_in=W_in, extra_cap=3)


def _rows(B, lo, hi, seed, top=None):
    ns = np.random.default_rng(seed).integers(lo, hi + 1, size=B)
    ns[seed % B] = hi if top is None else top
    return ns


EVEN = 32 * 1024   # columns (D = 8) from which on even rows go 32 at a time
# name: (case, route of a greedy step, rows at a time there, route of a realignment alone)
CASES = {
    # two stripes of the table's 1024 threads; uneven rows one at a time
    "table_two_stripes": (_case(8250, _rows(1100, 0, 8244, 1), H=1), "table", 1, "chunks"),
    # even long rows 32 at a time, the second group a single row
    "table_even_partial_group": (_case(EVEN + 200, _rows(33, EVEN, EVEN + 194, 2), H=8), "table", 32, "sorted"),
    "table_even_short": (_case(8300, _rows(33, 8000, 8294, 3), H=8), "table", 1, "sorted"),
    "table_four_movers": (_case(EVEN + 20, [EVEN + 14, EVEN, EVEN, EVEN - 9, EVEN], H=40), "table", 1, "sorted"),
    "nothing_moves": (_case(8206, [8200] * 40, H=7, accept=("fixed", 3)), "table", 1, "sorted"),
    # spans of half and of a quarter of a chunk share a workgroup (6 spans a row: some waves have none)
    "sorted_shares": (_case(8300, np.r_[8294, 4091, 4090, 4085, 2043, 2042, _rows(27, 0, 2060, 4)], H=3), "table", 1, "sorted"),
    "sorted_together": (_case(8200, _rows(64, 3800, 8194, 5), H=17), "table", 1, "sorted"),
    "sorted_together_shares": (_case(8400, np.r_[8394, _rows(50, 4200, 8394, 6), _rows(13, 0, 4000, 7)], H=18), "table", 1, "sorted"),
    # even rows alone: beyond 2048 spans without the rows that stay, the second group a few rows
    "sorted_even_many": (_case(8300, _rows(36, 8000, 8290, 14, 8294), H=32), "table", 1, "sorted"),
    "sorted_d24": (_case(2900, _rows(40, 100, 2894, 8), H=3, D=24), "table", 1, "sorted"),
    "far_left_walks": (_case(12000, _rows(40, 3000, 9000, 9), H=3), "table", 1, "sorted"),
    # chunks of 4096 vectors: lengths at their edges, shifts of both signs, shifts too long to hand over
    "few_edges": (_case(33000, [32994, 8187, 8186, 8185, 4091, 4090, 4085, 32983, 5000], H=1), "few", 0, "few"),
    "few_left": (_case(34000, [33400, 32000, 4090, 4096, 300], H=3), "few", 0, "few"),
    "few_far_left": (_case(40000, [33500, 16380, 4100, 10], H=2), "few", 0, "few"),
    "few_d128": (_case(2100, [2094, 2090, 767, 512, 511, 256, 30], H=2, D=128), "few", 0, "few"),
    # more than 64 rows alone: chunks of 4096 vectors, and of 8192 from 1536 spans on
    "chunks_4096": (_case(8300, _rows(65, 0, 8294, 10), H=2), "table", 1, "chunks"),
    "chunks_8192": (_case(8400, np.r_[_rows(60, 7900, 8394, 11), 8186, 8187, 8191, 70, 8190], H=13), "table", 1, "chunks"),
    "chunks_far_left": (_case(16000, np.r_[_rows(64, 100, 9000, 12), 12000], H=2), "table", 1, "chunks"),
}


def _geometry(w, seed=1):
    n, W_in, pad, cap = wl.initial_geometry(w, seed)
    return w.L * 2 * w.B * w.H, W_in * w.D // 8


def test_cases_lie_where_they_say():
    for name, (w, step, _, alone) in CASES.items():
        spans, longest = _geometry(w)
        assert longest > 8192 and spans <= 8192 and (spans <= 128 and longest >= 32768) == (step == "few"), name
        assert alone == ("few" if step == "few" else "sorted" if w.B <= 64 else "chunks"), name


def _table(o, w):
    """The order table's place at the end of a greedy workspace, and the rows at a time beside it."""
    from paper_2510_22876_amd import specdec as sd
    words = o.workspace.view(torch.int32).cpu().numpy()
    end = sd.workspace_bytes(w.B, w.k, w.V) // 4
    return words[end - 4 * w.B: end].reshape(w.B, 4), int(words[1])


def _check_table(o, w, r, rows_at_a_time):
    got, group = _table(o, w)
    assert group == rows_at_a_time, "rows at a time"
    assert sorted(got[:, 0]) == list(range(w.B)), "not a permutation of the rows"
    L = r.W_in - (w.k + 1)
    length = L - r.pad_in + r.out["n_acc"] + 1
    ok = (r.pad_in >= 0) & (r.pad_in <= L)
    moves = ok & (r.out["pad_out"] != r.pad_in)
    at = got[:, 0]
    assert np.array_equal(got[:, 1], r.pad_in[at])
    assert np.array_equal(got[:, 2], np.where(moves, r.out["pad_out"], r.pad_in)[at])
    assert np.array_equal(got[ok[at], 3], length[at[ok[at]]])
    count = int(moves.sum())
    assert moves[at[:count]].all() and not moves[at[count:]].any(), "moving rows come first"
    if count:
        lo, hi, classes = int(length[moves].min()), int(length[moves].max()), 7 if rows_at_a_time == 1 else 2
        cls = np.minimum((hi - length[at[:count]]) * classes // (hi - lo + 1), classes - 1)
        key = list(zip(cls, at[:count]))
        assert key == sorted(key), "classes of length, each in the rows' order"


def _step(w, seed, monkeypatch):
    """A greedy step in place; its workspace had a sentinel in every word."""
    from paper_2510_22876_amd import specdec as sd
    kept = {}
    init = sd.StepBuffers.__init__

    def filled(self, *a, **kw):
        init(self, *a, **kw)
        self.workspace.view(torch.int32).fill_(SENT)
        kept["o"] = self

    monkeypatch.setattr(sd.StepBuffers, "__init__", filled)
    r = run_gpu(w, seed=seed, variant="inplace", tokens="inplace")
    monkeypatch.setattr(sd.StepBuffers, "__init__", init)
    return r, kept["o"]


def _check(r, w):
    v = check_verify_vs_oracle(r)
    if r.src.numel() <= 1 << 26:
        check_kv_full_vs_oracle(r, v)
    check_posmask_vs_oracle(r, v)
    check_relocation_on_device(r, r.out["pad_out"], r.out["n_acc"], r.out["w_new"])
    check_tokens_vs_oracle(r, v)
    W = r.out["w_new"]
    assert torch.equal(i16(r.dst[..., W:, :]), i16(r.src[..., W:, :])), "columns beyond the new width were written"


@pytest.mark.parametrize("name", sorted(CASES))
def test_step(monkeypatch, name):
    w, route, rows_at_a_time, _ = CASES[name]
    say(f"in-place step {name}: route {route}")
    for seed in (1, 4):
        r, o = _step(w, seed, monkeypatch)
        _check(r, w)
        if route == "table":
            _check_table(o, w, r, rows_at_a_time)
        else:
            assert (_table(o, w)[0] == SENT).all(), "an order table that no launch reads"


@pytest.mark.parametrize("name", sorted(CASES))
def test_realignment_alone(name):
    w = CASES[name][0]
    say(f"in-place realignment {name}: route {CASES[name][3]}")
    for seed in (1, 4):
        _check(run_gpu(w, seed=seed, variant="inplace", api="split", tokens="inplace"), w)


@pytest.mark.parametrize("api", ["step", "split"])
@pytest.mark.parametrize("name", ["few_edges", "few_d128", "sorted_shares", "chunks_4096", "table_even_partial_group"])
def test_split_over_launches(monkeypatch, name, api):
    w = CASES[name][0]
    extra = w.B * ((w.W_in + w.k + 1 + 1023) // 1024 + 1)   # position-id and token workgroups: one launch holds them
    monkeypatch.setenv("SPECDEC_MAX_LAUNCH_ITEMS", str(256 * (extra + 40)))
    _check(run_gpu(w, seed=2, variant="inplace", api=api, tokens="inplace"), w)


def test_more_than_8192_spans(monkeypatch):
    """8250 spans: the walk 32 rows at a time (the second group a single row), and
    a realignment alone in the cache's order."""
    w = _case(8200, _rows(33, 0, 8194, 13), H=125)
    r, o = _step(w, 1, monkeypatch)
    check_verify_vs_oracle(r)
    check_relocation_on_device(r, r.out["pad_out"], r.out["n_acc"], r.out["w_new"])
    _check_table(o, w, r, 32)
    del r, o
    torch.cuda.empty_cache()
    r = run_gpu(w, seed=1, variant="inplace", api="split")
    check_relocation_on_device(r, r.out["pad_out"], r.out["n_acc"], r.out["w_new"])


@pytest.mark.parametrize("name", ["table_two_stripes", "sorted_shares", "few_edges", "chunks_4096"])
@pytest.mark.parametrize("api", ["step", "split"])
def test_rows_out_of_range_stay(name, api):
    """A padding out of range, and in a realignment alone also an accepted count:
    the row is flagged and keeps every byte, the others are the oracle's."""
    from paper_2510_22876_amd import specdec as sd
    w = CASES[name][0]
    n, W_in, pad, cap = wl.initial_geometry(w, 1)
    logits, draft, *_ = wl.logits_and_drafts(w, 1, device="cuda")
    src = wl.make_kv(w, pad, W_in, cap, 1, device="cuda")
    before = src.clone()
    bad = [2] if api == "step" else [2, 5]
    good = [i for i in range(w.B) if i not in bad]
    v = oracle.verify(logits[good].cpu(), w.logit_dtype, draft[good].cpu().numpy(), pad[good], W_in)
    i32 = lambda x: torch.as_tensor(np.ascontiguousarray(x, np.int32), device="cuda")
    given = pad.copy()
    given[2] = W_in
    o = alloc_outputs(w.B, w.k, w.V, W_in + w.k + 1)
    say(f"bad rows {name} {api}")
    if api == "step":
        sd.specdec_step(logits, draft, i32(given), W_in, src, src, o.tokens, o.n_acc, o.bonus, o.pad_out, o.w_new, o.pos,
                        o.mask, o.workspace, o.dev_status)
        want = sd.DEV_BAD_PAD_IN | sd.DEV_BAD_PAD_OUT
    else:
        n_acc = np.zeros(w.B, np.int32)
        n_acc[good] = v["n_acc"]
        n_acc[5] = w.k + 1
        sd.specdec_realign_kv(src, src, w.k, W_in, i32(given), i32(n_acc), i32([v["w_new"]]), o.dev_status)
        want = sd.DEV_BAD_PAD_IN | sd.DEV_BAD_ACCEPT
    torch.cuda.synchronize()
    assert int(o.dev_status) == want
    W = v["w_new"]
    for i in bad:
        assert torch.equal(i16(src[:, :, i]), i16(before[:, :, i])), f"row {i} was touched"
    pick = good if w.B <= 64 else good[:40] + good[-40:]
    where = [good.index(i) for i in pick]
    exp = oracle.realign_kv(np.ascontiguousarray(bits(before[:, :, pick])), w.k, W_in, pad[pick], v["n_acc"][where], W)
    assert np.array_equal(bits(src[:, :, pick])[..., :W, :], exp[..., :W, :])
