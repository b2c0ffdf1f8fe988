"""The order in which fg_path_run queues an iteration on its two streams, recorded without a device (tests/path_queue.py)."""
import itertools
import random

import pytest

from tests.path_queue import MAIN, SIDE, record

DIMS = [64, 96, 96, 96]


def sizes(n1):
    return [60_000, n1, 5_000, 300]


RIDES, OWN = dict(n=sizes(25_000)), dict(n=sizes(24_000))      # layer 1 as one launch beside a second stream: from 24576 positions on
MODEL = ["model", dict(dims=DIMS, n_max=[80_000, 40_000, 8_000, 1_024])]


def behind(calls):
    """For every launch, in order: (index of the call, stream, kernel, launches known to have ended when it starts: {launch's number}), and per call
    what it returned."""
    clock, events, out = {MAIN: set(), SIDE: set()}, {}, []
    n = 0
    for i, (*_, lines) in enumerate(calls):
        for op, stream, what, *_ in lines:
            s = int(stream)
            if op == "launch":
                out.append((i, s, what, frozenset(clock[s])))
                clock[s].add(n)
                n += 1
            elif op == "record":
                events[what] = set(clock[s])
            else:
                clock[s] |= events.get(what, set())      # (an event that was never recorded holds nobody up)
    return out


def orders():
    r = random.Random(7)
    return ["".join(k) for k in itertools.product("ro", repeat=6)] + ["rxoror", "orxoor", "roorooroo"] + ["".join(r.choices("rroooxnc", k=12)) for _ in range(40)]


@pytest.mark.parametrize("kinds", orders())
def test_steps_of_both_kinds_in_any_order_follow_each_other(tmp_path_factory, kinds):
    """Steps whose selection goes with the loader (r) and steps that put it on the second stream (o; x: whose announced successor is not the one that
    comes, n: without an update, c: in front of which the caller has copied the rows that were due), queued back to back: whatever a call queues waits
    for everything that the call before the last one queued, and for the copy of the rows that it left to the last one. (Sets of lists and halves
    of the update's workspace are used again then.)"""
    batches = [RIDES if k == "r" else OWN for k in kinds]
    script = [MODEL] + [["run", dict(it=i, batch=b, next=None if i + 1 == len(kinds) else (dict(n=sizes(20_000)) if k == "x" else batches[i + 1]),
                                     update=int(k != "n"), commit=k == "c")] for i, (k, b) in enumerate(zip(kinds, batches))]
    _, *calls = record(tmp_path_factory.getbasetemp(), script)
    launches = behind(calls)
    for i, k in enumerate(kinds):
        rc, selected, next_pruned, begun, _ = calls[i]
        mine = [name for j, _, name, _ in launches if j == i]
        assert rc == 0 and begun == 1 and next_pruned == (i + 1 < len(kinds) and k != "n")
        assert selected == next_pruned
        assert any("load_linear" in name for name in mine) == (k == "r")
    first = [min(n for n, x in enumerate(launches) if x[0] == i) for i in range(len(calls))] + [len(launches)]
    for n, (i, stream, name, before) in enumerate(launches):
        # the lists, the index and the rows that the call before this one put on the second stream (a caller's own copy in front of the call needs
        # the index only)
        if i and stream == MAIN and not (kinds[i] == "c" and n == first[i] and "copy_rows" in name):
            needed = {m for m in range(first[i - 1], first[i]) if launches[m][1] == SIDE}
            assert needed <= before, f"call {i}: {name} does not wait for {[launches[m][2] for m in sorted(needed - before)]} on the second stream"
        if i < 2:
            continue
        due = calls[i - 2][1] and kinds[i - 2] != "r"      # (a riding step's rows are copied by its own launches)
        assert due == ("copy_rows" in launches[first[i - 1]][2])      # the first launch of the call before this one
        needed = set(range(first[i - 1] + (1 if due else 0)))
        assert needed <= before, f"call {i}: {name} on stream {stream} does not wait for {[launches[m][2] for m in sorted(needed - before)]}"


@pytest.mark.parametrize("feat,compute", [("F32", "F32"), ("F16", "BF16")])
def test_no_launch_asks_for_more_lds_than_a_compute_unit_has(tmp_path_factory, feat, compute):
    """Rows of one 16-byte piece and up, on one stream and on two, below and above the sizes where layer 1 becomes one launch, forward and training."""
    piece = 4 if feat == "F32" else 8
    for d in (piece, 2 * piece, 4 * piece, 8 * piece):
        for train in (0, 1):
            script = [["model", dict(dims=[d, 64, 64, 64], n_max=[80_000, 40_000, 8_000, 1_024], feat=feat, compute=compute, fuse_small_layers=int(feat == "F32" and not train),
                                backward=train, weight_grads=train)]]
            script += [["run", dict(it=i, batch=dict(n=sizes(n1), own_rows_from_table=5 * int(feat == "F32" and not train)), overlap=overlap)]
                       for i, (n1, overlap) in enumerate((n1, o) for n1 in (5_000, 12_000, 25_000) for o in (0, 1))]
            _, *calls = record(tmp_path_factory.getbasetemp(), script)
            for rc, *_, lines in calls:
                assert rc == 0, rc
                for name, lds in ((x[2], int(x[3])) for x in lines if x[0] == "launch"):
                    assert lds <= 160 * 1024, f"{name} asks for {lds} bytes, rows of {d} {feat}"


# layer 1 as one launch, and the loader with the selection in it (on one stream, where nothing is pruned ahead)
@pytest.mark.parametrize("n1,overlap,at", [(25_000, 1, "no_ids"), (25_000, 1, "no_weights"), (25_000, 0, "no_weights"), (12_000, 0, "no_weights")])
def test_a_step_that_fails_behind_its_selection_leaves_its_rows_due(tmp_path_factory, n1, overlap, at):
    """The next mini-batch, or an upper layer, is refused when the selection has gone with the loader: the index names slots whose rows are not
    there, so the next update is refused until they are, nothing is promised, and the caller's stream is behind the second one."""
    good = dict(n=sizes(n1))
    now, later = (dict(good, no_weights=3), good) if at == "no_weights" else (good, dict(good, no_ids=2))
    calls = record(tmp_path_factory.getbasetemp(), [MODEL, ["run", dict(it=0, batch=good, next=now, overlap=overlap)], ["run", dict(it=1, batch=now, next=later, overlap=overlap)],
                                                    ["run", dict(it=2, batch=good, overlap=overlap, forget=True)]])[1:]
    assert calls[0][:2] == [0, overlap]
    rc, selected, next_pruned, begun, lines = calls[1]
    assert str(rc)[:2] in ("1:", "2:") and selected == 1 and begun == 1
    launches = behind(calls)
    copies = [x for x in launches if x[0] == 1 and "copy_rows" in x[2]]
    assert len(copies) == (at == "no_weights" and overlap) and next_pruned == len(copies)
    if at == "no_ids":
        waits = [x for x in lines if x[0] == "wait"]
        assert waits[-1][1] == str(MAIN) and ["record", str(SIDE), waits[-1][2]] in lines
    assert str(calls[2][0]).startswith("4:") and "fg_cache_update_commit" in calls[2][0]


@pytest.mark.parametrize("n1,overlap", [(25_000, 1), (25_000, 0), (12_000, 0)])
def test_rows_of_a_step_that_fails_can_be_committed(tmp_path_factory, n1, overlap):
    good = dict(n=sizes(n1))
    calls = record(tmp_path_factory.getbasetemp(), [MODEL, ["run", dict(it=0, batch=dict(good, no_weights=3), overlap=overlap)],
                                                    ["run", dict(it=1, batch=good, overlap=overlap, commit=True)], ["run", dict(it=2, batch=good, overlap=overlap)]])[1:]
    assert str(calls[0][0]).startswith("1:") and calls[0][1] == 1
    assert [c[:2] for c in calls[1:]] == [[0, 0], [0, 0]]


@pytest.mark.parametrize("one,d_in,d_out,most,nnz,n,overlap,p_grad", [
    (1, 128, 256, 17, 13, 25_000, 1, 0.3), (0, 128, 256, 18, 13, 25_000, 1, 0.3), (0, 128, 256, 1, 1, 25_000, 1, 0.3),      # what the rows have at most
    (1, 128, 256, 10, 8, 25_000, 1, 0.3), (0, 128, 256, 10, 7, 25_000, 1, 0.3), (1, 128, 256, 9, 7, 25_000, 1, 0.3),        # places of a row
    (1, 64, 128, 15, 7, 25_000, 1, 0.3), (0, 68, 128, 15, 7, 25_000, 1, 0.3),
    (1, 36, 64, 15, 13, 25_000, 1, 0.7), (0, 32, 64, 15, 13, 25_000, 1, 0.3),                                               # narrow rows
    (1, 128, 256, 15, 13, 24_576, 1, 0.3), (0, 128, 256, 15, 13, 24_575, 1, 0.3),                                           # two streams
    (1, 128, 256, 15, 13, 16_384, 0, 0.7), (0, 128, 256, 15, 13, 16_383, 0, 0.3), (0, 128, 64, 15, 13, 20_000, 0, 0.3),     # one
    (1, 64, 68, 15, 13, 20_000, 0, 0.5), (0, 64, 68, 15, 13, 20_000, 0, 0.6), (1, 68, 68, 15, 13, 20_000, 0, 0.6)])
def test_which_steps_load_and_multiply_in_one_launch(tmp_path_factory, one, d_in, d_out, most, nnz, n, overlap, p_grad):
    """Around every line of the rule (`HotPath.loads_and_multiplies` is the same one)."""
    from types import SimpleNamespace
    from paper_2301_07482_amd import binding as B, pipeline
    b = dict(n=[n, n, 1_000], nnz=[0, nnz * n, 5_000], own_rows_from_table=most)
    _, (rc, *_, lines) = record(tmp_path_factory.getbasetemp(), [["model", dict(dims=[d_in, d_out, 64], n_max=[1 << 19, 40_000, 8_000])],
                                                                ["run", dict(it=0, batch=b, overlap=overlap, p_grad=p_grad)]])
    kernels = [x[2] for x in lines if x[0] == "launch"]
    assert rc == 0 and any("load_linear" in k for k in kernels) == bool(one) != any("loader_fetch" in k for k in kernels)
    hp = SimpleNamespace(own_rows_from_table=lambda bt: True, h_code=[B.FG_F32] * 3, dims=[d_in, d_out, 64], most_neighbours=max(most, 2) if most > 1 else 99,
                         overlap_update=bool(overlap), p_grad=p_grad)
    assert pipeline.HotPath.loads_and_multiplies(hp, SimpleNamespace(n=b["n"], nnz=b["nnz"])) == bool(one)


def test_a_chosen_dense_kernel_leaves_the_selection_where_it_was(tmp_path_factory):
    """With a dense kernel chosen by `linear_tile` layer 1 is two launches; the selection and the next top-down pass are then on the second stream, as
    in a step that is two launches by its sizes."""
    calls = record(tmp_path_factory.getbasetemp(), [["model", dict(MODEL[1], fuse_small_layers=0)], ["tune", dict(key="linear_tile", value=32)], ["run", dict(it=0, batch=RIDES, next=OWN)],
                                                    ["tune", dict(key="linear_tile", value=0)]])
    rc, selected, next_pruned, _, lines = calls[2]
    assert rc == 0 and selected == 1 and next_pruned == 1
    assert {x[1] for x in lines if x[0] == "launch" and "update_digit" in x[2]} == {str(SIDE)}


@pytest.mark.parametrize("kernel,n1,n2,overlap,kwargs", [
    ("loader_fetch_update", 4_096, 300, 0, {}), ("loader_fetch_update", 16_000, 5_000, 0, {}), ("update_group", 0, 0, 0, {}),
    ("loader_fetch_update", 257_000, 300, 0, dict(dims=[32, 64, 64, 64])), ("update_digit", 261_000, 300, 0, dict(dims=[32, 64, 64, 64])),      # 64 chunks, 65
    ("loader_fetch_update", 8_000, 300, 0, dict(feat="F16", compute="BF16", fuse_small_layers=0)),
    ("update_group", 8_000, 300, 1, {}), ("update_digit", 24_000, 300, 1, {}),                                                  # beside, on the second stream
    ("load_linear", 20_000, 300, 0, {}), ("load_linear", 126_000, 300, 1, {}), ("update_digit", 131_000, 300, 1, {}),                    # 32 chunks, 33
])
def test_which_launch_takes_a_steps_selection(tmp_path_factory, kernel, n1, n2, overlap, kwargs):
    """Both loaders and the update's own launches, on both sides of the rule's lines; a launch that takes the selection along is the only one for it."""
    big = [1 << 20, 1 << 19, 1 << 17, 1 << 10]
    _, (rc, selected, _, _, lines) = record(tmp_path_factory.getbasetemp(), [["model", dict(dict(dims=DIMS, n_max=big), **kwargs)],
                                                                            ["run", dict(it=0, batch=dict(n=[2 * n1, n1, n2, min(n2, 300)]), overlap=overlap)]])
    updates = ("loader_fetch_update", "load_linear", "update_group_kernel", "update_digit")
    took = [x[2] for x in lines if x[0] == "launch" and any(u in x[2] for u in updates)]
    if kernel != "load_linear":      # (its launch may also come without a selection)
        took = [k for k in took if "load_linear" not in k]
    assert rc == 0 and took and all(kernel in k for k in took)


@pytest.mark.parametrize("how", ["next call", "commit", "neither"])
def test_rows_that_are_copied_on_the_second_stream_are_due_until_they_are_waited_for(tmp_path_factory, how):
    """A step whose selection goes with the loader and that prunes the next mini-batch ahead copies layer 1's rows on the second stream. It says, as every
    step that does so, that its rows are left to the next call or to fg_cache_update_commit: these wait for them."""
    first, after = record(tmp_path_factory.getbasetemp(), [MODEL, ["run", dict(it=0, batch=RIDES, next=RIDES)],
                                                           ["run", dict(it=1, batch=RIDES, commit=how == "commit", forget=how == "neither")]])[1:]
    assert first[:3] == [0, 1, 1]
    copied = max(i for i, x in enumerate(first[4]) if x[0] == "launch" and x[1] == str(SIDE))
    assert "copy_rows" in first[4][copied][2] and first[4][copied + 1][:2] == ["record", str(SIDE)]
    if how == "neither":
        assert str(after[0]).startswith("4:")
        return
    assert after[0] == 0 and not any("copy_rows_batch" in x[2] for x in after[4][:4] if x[0] == "launch")
    queued = [i for i, x in enumerate(after[4]) if x == ["wait", str(MAIN), first[4][copied + 1][2]]]
    assert queued and queued[0] < min(i for i, x in enumerate(after[4]) if x[0] == "launch") and len(queued) == (2 if how == "commit" else 1)
