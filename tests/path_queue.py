"""What fg_path_run queues, recorded in a process without a device (tests/c/hip_record.cpp in the place of the HIP runtime).

`Queue(recorder)` has to be made before anything else loads the library, so callers start a process of their own (`record`)."""
import ctypes as C
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MAIN, SIDE = 1, 2      # the two streams


def record(tmp_path, script):
    """Runs `script`, a list of calls of `Queue`'s methods [name, kwargs], in a process of its own; what each of them returns, as a list."""
    lib = str(tmp_path / "hip_record.so")
    if not os.path.exists(lib):
        rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I", os.path.join(rocm, "include"),
                        os.path.join(ROOT, "tests", "c", "hip_record.cpp"), "-o", lib], check=True)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), lib], input=json.dumps(script), capture_output=True, text=True, timeout=120, cwd=ROOT)
    assert r.returncode == 0, r.stderr
    return json.loads(r.stdout)


class Queue:
    def __init__(self, recorder):
        self.rec = C.CDLL(recorder, C.RTLD_GLOBAL)      # ahead of the HIP runtime
        self.rec.hip_record_log.restype = C.c_char_p
        sys.path.insert(0, ROOT)
        from paper_2301_07482_amd import binding as B
        self.B, self.at = B, 1 << 32

    def _mem(self, n=1 << 24):
        self.at += n
        return self.at

    def _log(self):
        lines = self.rec.hip_record_log().decode().split("\n")[:-1]
        self.rec.hip_record_clear()
        return [s.split(" ") for s in lines]

    def model(self, dims, n_max, feat="F32", compute="F32", fuse_small_layers=1, num_nodes=1 << 20, backward=0, weight_grads=0):
        B, L = self.B, len(dims) - 1
        self.cache = B.fg_cache_create(num_nodes, [1 << 16] * (L - 1), list(dims[1:L]), getattr(B, "FG_" + compute), 8, MAIN)
        P = self.P = B.Path()
        P.n_layers, P.model, P.feat_dtype, P.compute_dtype = L, B.FG_PATH_SAGE, getattr(B, "FG_" + feat), getattr(B, "FG_" + compute)
        P.fused_input, P.fuse_small_layers, P.ring, P.num_nodes, P.backward, P.weight_grads = 1, fuse_small_layers, 8, num_nodes, backward, weight_grads
        P.dims[:L + 1], P.n_max[:L + 1] = dims, n_max
        for l in range(L + 1):
            P.h[l], P.agg[l] = self._mem(), self._mem()
            P.dh[l], P.gnorm[l], P.dw[l], P.db[l] = (self._mem() for _ in range(4))
        for s in P.lists:
            for name in ("live", "hit", "hit_pos", "hit_slot", "normal_pos"):
                for l in range(L + 1):
                    getattr(s, name)[l] = self._mem()
            s.input_ids, s.self_ids = self._mem(), self._mem()
        for name in ("counts_log", "stats_log", "input_log", "ws_top_down", "ws_update", "ws_backward", "ws_weights"):
            setattr(P, name, self._mem(1 << 32))
        P.ws_top_down_bytes = P.ws_update_bytes = P.ws_update_stride = P.ws_backward_bytes = P.ws_weights_bytes = 1 << 28
        P.side = SIDE
        for name in ("ev_pruned", "ev_selected", "ev_next_pruned", "ev_gradients", "ev_weights"):
            setattr(P, name, self._event())
        P.ev_done[0], P.ev_done[1] = self._event(), self._event()
        self.weights = [None] + [(self._mem(), self._mem(), self._mem()) for _ in range(L)]
        self.specs = (B.UpdateLayer * (L - 1))()
        self.feat = self._mem()
        self.due = self.ahead = None      # (iteration) whose rows are due; the mini-batch that has been pruned ahead
        return self._log()

    def tune(self, key, value):
        self.B.fg_set_tuning(key, value)

    def _event(self):
        e = C.c_void_p()
        assert self.B._lib.fg_event_create(C.byref(e)) == 0
        return e.value

    def _batch(self, b, L):
        """b: dict(n=[...], and optionally own_rows_from_table, no_ids / no_weights: a layer that lacks them)"""
        x = self.B.PathBatch()
        x.labels_dev, x.col_ids1_dev, x.own_rows_from_table = self._mem(), self._mem(), b.get("own_rows_from_table", 5)
        for l, n in enumerate(b["n"]):
            y = x.layer[l]
            y.n, y.nnz = n, b["nnz"][l] if "nnz" in b else (b["n"][l - 1] if l else 0)
            for name in ("ids_dev", "start_dev", "end_dev", "col_dev", "gnorm_dev", "t_start_dev", "t_end_dev", "t_row_dev"):
                setattr(y, name, None if name == "ids_dev" and l == b.get("no_ids") else self._mem())
        return x

    def run(self, it, batch, next=None, update=1, overlap=1, commit=False, forget=False, p_grad=0.3):
        """One call, with what the previous one left. commit: the caller commits what is due first; forget: it drops that.
        -> [0 or the error, selected, next_pruned, begun, lines]"""
        B, L = self.B, self.P.n_layers
        if commit and self.due is not None:
            assert B._lib.fg_stream_wait_event(MAIN, self.P.ev_selected) == 0
            assert B._lib.fg_cache_update_commit(self.cache, self.due, L - 1, self.specs, self.P.ws_update + self.due % 2 * self.P.ws_update_stride,
                                                 self.P.ws_update_bytes, MAIN) == 0
            self.due = None
        if forget:
            self.due = self.ahead = None
        call = B.PathCall()
        call.iter, call.stream, call.cache, call.feat = it, MAIN, self.cache, self.feat
        for l in range(1, L + 1):
            call.w[l], _, call.bias[l] = self.weights[l] if l != batch.get("no_weights") else (None, None, None)
        if self.P.compute_dtype == B.FG_BF16:
            for l in range(1, L + 1):
                call.wt[l] = self.weights[l][1]
        call.p_grad, call.update, call.overlap, call.fetch_with_loader = p_grad, update, overlap, 1
        call.promised, call.pruned_ahead = self.ahead is not None, self.ahead == [it, batch]
        call.specs = self.specs
        if self.due is not None:
            call.due, call.due_iter = self.specs, self.due
        rc = B._lib.fg_path_run(C.byref(self.P), C.byref(self._batch(batch, L)), C.byref(self._batch(next, L)) if next is not None else None, C.byref(call))
        if call.begun:
            self.due = self.ahead = None
        if call.next_pruned:
            self.ahead = [it + 1, next]
        if call.selected:
            self.due = it
        return [f"{rc}: {B.fg_last_error()}" if rc else 0, call.selected, call.next_pruned, call.begun, self._log()]


if __name__ == "__main__":
    q = Queue(sys.argv[1])
    print(json.dumps([getattr(q, name)(**kwargs) for name, kwargs in json.load(sys.stdin)]))
