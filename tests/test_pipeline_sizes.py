"""Sizes the host side of the iteration hands to the C calls, checked without a GPU (the calls are recorded, not made)."""
import types

import pytest


def _path(monkeypatch, n_max, on_host):
    """A HotPath of two layers with lists of n_max positions, as far as its top-down pass looks at it, and the recorded specs."""
    torch = pytest.importorskip("torch")
    from paper_2301_07482_amd import pipeline as P
    calls = []
    monkeypatch.setattr(P.B, "top_down_layers", lambda specs: calls.append(specs) or specs)
    monkeypatch.setattr(P.B, "fg_top_down", lambda *a: None)
    hp = P.HotPath.__new__(P.HotPath)
    lists = [torch.zeros(n, dtype=torch.int32) for n in n_max]
    hp.__dict__.update(L=2, n_max=n_max, dims=[128, 16, 16], feat_code=P.B.FG_F32, on_host=on_host, fused_input=True, feature_side=False,
                       use_cache=False, cache=None, one_launch_top_down=True, ws_td=None, ws_td_bytes=0, live=lists, hit=lists,
                       hit_pos=lists, hit_slot=lists, normal_pos=lists, input_ids=lists[0], self_ids=lists[1],
                       counts=torch.zeros((3, 3), dtype=torch.int64), input_log=torch.zeros((4, 3), dtype=torch.int64), input_slot=0)
    return P, hp, calls


def _batch(n, nnz, n_dev):
    return types.SimpleNamespace(n=list(n), nnz=list(nnz), n_dev=list(n_dev), ids=[None] * 3, start=[None] * 3, end=[None] * 3, col=[None] * 3)


@pytest.mark.parametrize("on_host", [0, 1])
def test_top_down_of_an_announced_mini_batch_stays_within_its_lists(monkeypatch, on_host):
    """A mini-batch whose sizes are still on the device comes with the sampler's bounds, which may exceed the node count (500
    here); the pass that runs ahead for it gets the sizes its lists were made for, with the input layer (host table) or without."""
    P, hp, calls = _path(monkeypatch, [500, 330, 30], on_host)
    bt = _batch([30 * 11 * 11, 330, 30], [0, 330 * 80, 300], [1, 1, None])
    hp._top_down(bt, 1, None, P._no_tick)
    assert len(calls[0]) == (3 if on_host else 2)
    for spec, n_max in zip(calls[0], reversed(hp.n_max)):
        assert spec["n"] <= n_max
    assert [s["n_src"] for s in calls[0] if s["n_src"]] == [330, 500]


def test_top_down_refuses_host_sizes_beyond_its_lists(monkeypatch):
    P, hp, calls = _path(monkeypatch, [500, 330, 30], 1)
    with pytest.raises(AssertionError):
        hp._top_down(_batch([501, 330, 30], [0, 13200, 300], [None] * 3), 1, None, P._no_tick)
    assert not calls


def test_binding_an_iteration_makes_no_view_of_the_input_layers_counts(monkeypatch):
    """`_bind` runs up to three times per iteration on the host's critical path; the input layer's counts, which only a table
    in host memory uses, are named by their address alone."""
    P, hp, _ = _path(monkeypatch, [500, 330, 30], 1)
    import torch

    class Log:      # anything but its address is too much
        base = torch.zeros((4, 3), dtype=torch.int64)

        def data_ptr(self):
            return self.base.data_ptr()

    hp.__dict__.update(ring=4, _lists=[{}, {}, {}], counts_log=torch.zeros((4, 3, 3)), stats_log=torch.zeros((4, 3, 4)), input_log=Log())
    hp._bind(7)
    assert hp._input_cnt(2) == Log.base[3, 2].data_ptr()


@pytest.mark.parametrize("n", [1, 589, 1767, 15903, 52000])
@pytest.mark.parametrize("kind", ["sage", "gcn", "bf16"])
def test_weight_gradient_workspace_is_that_of_the_widths_the_call_gets(kind, n):
    """The workspace a model is set up with serves every layer's call: a GCN layer's goes with half its input width, whose split may
    leave more partial results (15903 rows of 104 columns x 72: the call was refused)."""
    pytest.importorskip("torch")
    from paper_2301_07482_amd import pipeline as P
    size = P.B.fg_layer_backward_weights_bf16_workspace_bytes if kind == "bf16" else P.B.fg_layer_backward_weights_workspace_bytes
    for d_in in range(8, 520, 8):
        for d_out in (8, 72, 128, 136, 256, 512):
            width = d_in // 2 if kind == "gcn" else d_in
            assert P.weight_grad_workspace_bytes(kind, n, d_in, d_out) >= size(n, width, d_out), (d_in, d_out)


@pytest.mark.parametrize("begun", [0, 1])
def test_a_refused_iteration_keeps_what_the_one_before_left_to_it(monkeypatch, begun):
    """The row copy of the previous selection, whose rows the index names already, and the wait for the top-down pass that runs ahead
    stay due until a call has queued them."""
    pytest.importorskip("torch")
    from paper_2301_07482_amd import pipeline as P
    hp = P.HotPath.__new__(P.HotPath)
    call, specs = P.B.PathCall(), (P.B.UpdateLayer * 1)()
    hp.__dict__.update(L=2, use_cache=True, cache=P.B._p(4096), overlap_update=True, backward=False, feat=None, W={}, Wt={}, bias={}, p_grad=0.5,
                       fetch_with_loader=True, _row_copy_due=(3, specs), _td_for=(4, "announced"), _ready_waited=None,
                       _native=(P.B.Path(), call, (P.B.PathBatch(), P.B.PathBatch()), specs),
                       _pack=lambda *a: None, _pack_model=lambda *a: None, weight_grads_ahead=lambda bt: False)
    seen = []

    def refuse(path, batch, later, c):
        seen.append((bool(c.due), c.due_iter, c.promised))
        c.begun, c.selected, c.next_pruned = begun, 0, 0
        raise P.B.FgError(P.B.FG_ERR_INVALID_ARG, "refused")

    monkeypatch.setattr(P.B, "fg_path_run", refuse)
    main = types.SimpleNamespace(cuda_stream=0)
    with pytest.raises(P.B.FgError):
        hp._run_native(_batch([1, 1, 1], [0, 0, 0], [None] * 3), 4, main, True, None, True, False)
    assert seen == [(True, 3, 1)]
    assert (hp._row_copy_due, hp._td_for) == ((None, None) if begun else ((3, specs), (4, "announced")))


def test_rows_that_are_due_are_copied_when_the_cache_is_switched_off(monkeypatch):
    pytest.importorskip("torch")
    from paper_2301_07482_amd import pipeline as P
    hp = P.HotPath.__new__(P.HotPath)
    call, specs, order = P.B.PathCall(), (P.B.UpdateLayer * 1)(), []
    hp.__dict__.update(L=2, use_cache=False, cache=P.B._p(4096), overlap_update=True, backward=False, feat=None, W={}, Wt={}, bias={}, p_grad=0.5,
                       fetch_with_loader=True, _row_copy_due=(3, specs), _td_for=None, _ready_waited=None, ev_selected="selected", ws_upd_bytes=64,
                       ev_done=[None, types.SimpleNamespace(record=lambda st: order.append("recorded"))], _ws_upd=lambda it: 4096,
                       _native=(P.B.Path(), call, (P.B.PathBatch(), P.B.PathBatch()), specs),
                       _pack=lambda *a: None, _pack_model=lambda *a: None, weight_grads_ahead=lambda bt: False)
    monkeypatch.setattr(P.B, "fg_cache_update_commit", lambda cache, it, y, *a: order.append((cache.value, it, y is specs)))

    def run(path, batch, later, c):
        order.append((c.cache, bool(c.due)))
        c.begun = 1

    monkeypatch.setattr(P.B, "fg_path_run", run)
    main = types.SimpleNamespace(cuda_stream=0, wait_event=order.append)
    hp._run_native(_batch([1, 1, 1], [0, 0, 0], [None] * 3), 4, main, True, None, False, False)
    assert order == ["selected", (4096, 3, True), "recorded", (None, False)] and hp._row_copy_due is None
