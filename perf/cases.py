"""The workloads whose speed is measured, each one pass of what a training program does with this framework.

Four kinds of pass ("path"):
  step    one iteration of the hot path (lookup and prune, loader, layers, cache update) on a resident mini-batch whose
          gradient norms are given: the headline benchmark's step
  train   the same iteration with the loss, the backward pass (embedding and weight gradients) and the cache update that
          takes its norms from it
  loop    a train iteration with the next mini-batches sampled on the device beside it: nothing prepared but the graph, the
          feature table and the seeds
  sample  one mini-batch drawn on the device, with the transposed blocks the backward pass walks

Sizes are those of the repository's own workloads (`fg_inputs.workload`), the large graphs with fewer nodes and the same
mini-batches: the feature table stays far larger than any cache of the chip. A resident mini-batch is used again once every
entry of its last use has left the cache by age, as a new one of an epoch would find it.
"""
import math

import torch

from fg_inputs import device as fdev
from fg_inputs import rng as ctr_rng
from fg_inputs import workload as wl
from paper_2301_07482_amd import pipeline as G

_LARGE = dict(nodes=27_750_000, degree=14.4, feat_dim=128, feat="f32", where="hbm", hidden=256, fanouts="15,10,5", batch=1024,
              model="sage", compute="f32", cache_share=0.1, t_stale=20, p_grad=0.3)


def listed():
    tiny = dict(nodes=10_000, degree=10.0, feat_dim=64, feat="f32", where="hbm", hidden=64, fanouts="10,5", batch=256, model="sage",
                compute="f32", cache_share=0.2, t_stale=10, p_grad=0.5)
    return [
        # a small graph that fits the caches of the chip: launches and host time decide
        dict(tiny, name="tiny_step", path="step"),
        dict(tiny, name="tiny_train", path="train"),
        # no size is a multiple of a tile: a user's own model on a mid-sized graph
        dict(tiny, name="ragged_train", path="train", nodes=500_003, degree=23.0, feat_dim=52, hidden=88, fanouts="12,7,4", batch=777,
             cache_share=0.15, t_stale=15, p_grad=0.4),
        # a products-like graph: dense neighbourhoods, 100 features
        dict(_LARGE, name="medium_step", path="step", nodes=2_400_000, degree=50.0, feat_dim=100, cache_share=0.2),
        # a papers-like graph, the headline workload's mini-batches: forward with the workload's and with the paper's thresholds,
        # training of both layer types
        dict(_LARGE, name="large_step", path="step"),
        dict(_LARGE, name="large_paper_step", path="step", t_stale=200, p_grad=0.9),
        dict(_LARGE, name="large_train", path="train"),
        dict(_LARGE, name="large_gcn_train", path="train", model="gcn"),
        # the mixed-precision workload: fp16 features, bf16 embeddings and weights, wide layers
        dict(name="mixed_train", path="train", nodes=3_000_000, degree=7.0, feat_dim=768, feat="f16", where="hbm", hidden=1024,
             fanouts="25,15", batch=1024, model="sage", compute="bf16", cache_share=0.15, t_stale=30, p_grad=0.3),
        # features too large for the card: read over the host link
        dict(_LARGE, name="large_host_step", path="step", nodes=3_468_750, where="host"),
        # sampling by itself, and the whole training loop with sampling in it
        dict(_LARGE, name="large_sample", path="sample"),
        dict(_LARGE, name="large_loop", path="loop"),
    ]


def draw(rng):
    """One more case: any kind of pass over the range from the tiny to the large workload."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    path = rng.choice(["step", "step", "train", "train", "loop", "sample"])
    layers = rng.choice([2, 3, 3])
    fanouts = [rng.randint(5, 15), rng.randint(3, 10), rng.randint(2, 5)][:layers]
    mixed = path != "sample" and rng.random() < 0.25
    hidden = 16 * rng.randint(8, 32) if mixed else 8 * rng.randint(8, 32)
    feat_dim = 8 * rng.randint(16, 64) if mixed else 4 * rng.randint(16, 32)
    model = "sage"
    if not mixed and path == "train" and rng.random() < 0.3:
        model, feat_dim = "gcn", 8 * (feat_dim // 8)
    t_stale = rng.choice([10, 15, 20, 30])
    return dict(path=path, nodes=log_int(10_000, 12_000_000), degree=round(rng.uniform(8.0, 40.0), 1), feat_dim=feat_dim,
                feat="f16" if mixed else "f32", where="hbm", hidden=hidden, fanouts=",".join(map(str, fanouts)), batch=log_int(200, 1024),
                model=model, compute="bf16" if mixed else "f32", cache_share=round(rng.uniform(0.05, 0.3), 2), t_stale=t_stale,
                p_grad=round(rng.uniform(0.2, 0.9), 2))


def _workload(case, seed):
    nodes = case["nodes"]
    train = 1_100_000 if nodes > 4_000_000 else None      # large graphs train on a subset of the nodes
    return wl.Workload("case", nodes, int(nodes * case["degree"]), case["feat_dim"], case["feat"], case["where"], case["hidden"],
                       tuple(int(f) for f in case["fanouts"].split(",")), case["batch"], train,
                       max(1, int(nodes * case["cache_share"])), case["t_stale"], case["p_grad"], case["compute"], 0, int(seed))


class _State:
    """What the program holds: the graph and its sampler, the feature table, the model with its cache, the mini-batches."""

    def __init__(self, case, seed):
        self.case, self.w = case, _workload(case, seed)
        w = self.w
        self.path = case["path"]
        self.train = self.path in ("train", "loop")
        self.hp, self.t, self.key = None, 0, int(seed) << 20
        graph = wl.make_graph(w)
        indptr, indices = fdev.chunglu_csr(graph)
        self.ds = G.DeviceSampler(indptr, indices, w.num_nodes, w.fanouts, w.batch, transposes=self.path != "step")
        period = min(w.t_stale + 4, (w.train_nodes or w.num_nodes) // w.batch)
        self.seeds = [torch.from_numpy(wl.seed_nodes(w, i).astype("int32")).cuda() for i in range(period)]
        self.labels = [torch.from_numpy(wl.node_labels(w, wl.seed_nodes(w, i))).cuda() for i in range(period)] if self.train else None
        if self.path != "sample":
            # the options of the headline benchmark
            self.hp = G.make_hotpath(w, fused_input=True, backward=self.train, weight_grads=self.train, model=case["model"],
                                     overlap_min_rows=65536, fuse_small_layers=True)[0]
            hp, L = self.hp, w.num_layers
            self.out = dict(h=[hp.H[l] for l in range(1, L + 1)], counts=hp.counts_log, stats=hp.stats_log)
            if self.train:
                self.out.update(norms=hp.gnorm[1:], dw=hp.dW[1:], db=hp.db[1:])
        if self.path in ("step", "train"):
            self._resident()
        elif self.path == "loop":
            self._ring()
        elif self.path == "sample":
            self.bufs = [self.ds.buffers() for _ in range(2)]
            for buf, counts in self.bufs:      # entries beyond the counts, and the seeds' row of the counts, are not written
                buf.zero_(), counts.zero_()
        if self.hp is not None:      # the cache as training finds it: every slot's age within the bound
            for _ in range(w.t_stale + 1):
                self.one()
        torch.cuda.synchronize()

    def __del__(self):
        if self.hp is not None:
            self.hp.close()

    def _resident(self):
        w, L = self.w, self.w.num_layers
        self.pool, self.ends = [], []
        for i in range(len(self.seeds)):
            # training keeps the layer sizes in device memory, as a loop that never waits for its sampler does
            bt = self.ds.sample(self.seeds[i], self.key + i, finish=not self.train, ready=False)
            if self.train:
                bt.labels = self.labels[i]
            else:
                bt.gnorm = {}
                for l in range(1, L):
                    bt.gnorm[l] = torch.empty(bt.n[l], dtype=torch.float32, device="cuda")
                    fdev.grad_norms(bt.ids[l], None, bt.n[l], int(ctr_rng.make_key(w.seed, 0x6AD, i, l)), bt.gnorm[l], torch.cuda.current_stream().cuda_stream)
            sizes = [len(bt.end[l]) for l in range(1, L + 1)]
            ends = torch.cat(bt.end[1:])
            bt.end[1:] = ends.split(sizes)
            self.pool.append(bt)
            self.ends.append((ends, ends.clone()))

    def _resident_pass(self):
        n, t = len(self.pool), self.t
        now, before = self.ends[(t + n // 2) % n]
        now.copy_(before)      # pruning empties rows of a mini-batch in place: put them back ahead of its next use
        self.hp.run(self.pool[t % n], t, next_bt=self.pool[(t + 1) % n])

    def _ring(self):
        self.side = torch.cuda.Stream()
        self.bufs = [self.ds.buffers() for _ in range(4)]
        self.consumed = [torch.cuda.Event() for _ in range(4)]
        torch.cuda.synchronize()
        self.queue = {t: self._sample_ahead(t) for t in (0, 1)}

    def _sample_ahead(self, t):
        with torch.cuda.stream(self.side):
            if t >= 4:
                self.side.wait_event(self.consumed[t % 4])
            bt = self.ds.sample(self.seeds[t % len(self.seeds)], self.key + t, finish=False, out=self.bufs[t % 4])
        bt.labels = self.labels[t % len(self.seeds)]
        return bt

    def _loop_pass(self):
        t = self.t
        self.queue[t + 2] = self._sample_ahead(t + 2)
        self.hp.run(self.queue.pop(t), t)
        self.consumed[t % 4].record()

    def _sample_pass(self):
        t = self.t
        self.ds.sample(self.seeds[t % len(self.seeds)], self.key + t, out=self.bufs[t % 2])
        self.out = self.bufs[t % 2]      # every array of the mini-batch, and its counts

    def one(self):
        {"step": self._resident_pass, "train": self._resident_pass, "loop": self._loop_pass, "sample": self._sample_pass}[self.path]()
        self.t += 1
        return self.out


def prepare(case, seed):
    return _State(case, seed)


def run(state):
    return state.one()


def _sizes(case):
    """Expected nodes n[l] and edges e[l] of a mini-batch (no overlap but that of draws among `nodes` nodes)."""
    fan = [int(f) for f in case["fanouts"].split(",")]
    L, n, e = len(fan), [0.0] * (len(fan) + 1), [0.0] * (len(fan) + 1)
    n[L] = float(case["batch"])
    for l in range(L, 0, -1):
        e[l] = n[l] * min(fan[l - 1], case["degree"])
        n[l - 1] = case["nodes"] * (1.0 - math.exp(-(n[l] + e[l]) / case["nodes"]))
    return L, n, e


def work(case):
    L, n, e = _sizes(case)
    d = [case["feat_dim"]] + [case["hidden"]] * L
    ein, ec = (4 if case["feat"] == "f32" else 2), (4 if case["compute"] == "f32" else 2)
    drawn = sum(n[l] * 20 + e[l] * 8 for l in range(1, L + 1)) + n[0] * 4     # row pointers, neighbours, ranges, columns, ids
    if case["path"] == "sample":
        return {"bytes": drawn + sum(n[l - 1] * 8 + e[l] * 4 for l in range(2, L + 1)), "flops": 0.0}
    # table rows of the input nodes and the mini-batch once, weights, outputs of every layer, admitted rows
    k = [0] + [(1 if case["model"] == "gcn" else 2) * d[l - 1] for l in range(1, L + 1)]
    bytes_ = n[0] * d[0] * ein + sum(n[l] * 13 + e[l] * 4 for l in range(1, L + 1)) + sum(k[l] * d[l] * ec for l in range(1, L + 1))
    bytes_ += sum(n[l] * d[l] * ec for l in range(1, L + 1)) + sum(case["p_grad"] * n[l] * d[l] * ec for l in range(1, L))
    flops = sum(2.0 * n[l] * k[l] * d[l] + e[l] * d[l - 1] for l in range(1, L + 1))
    if case["path"] in ("train", "loop"):
        bytes_ += sum(k[l] * d[l] * 4 for l in range(1, L + 1)) + sum(n[l] * 4 for l in range(1, L))
        flops += sum(2.0 * n[l] * k[l] * d[l] for l in range(1, L + 1)) + sum(2.0 * n[l] * k[l] * d[l] + e[l] * d[l - 1] for l in range(2, L + 1))
    if case["path"] == "loop":
        bytes_ += drawn
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    if case["path"] == "sample":
        return "exact"
    # The fp32 products of two different kernels (three-way bf16 splits, fp32 matrix instructions) are 2e-7 apart, single values
    # 1.5e-6. A ReLU output that is zero in one and barely above zero in the other lets a whole gradient through or not:
    # 3.4e-4 of a weight gradient, single values 0.02. Norms that differ in the last bit may change places at the admission.
    if case["compute"] == "bf16":
        return {"rel": 1e-2, "max": 0.1, "differ": 2e-3}
    if case["path"] in ("train", "loop"):
        return {"rel": 1.4e-3, "max": 0.08, "differ": 2e-3}
    return {"rel": 1e-6, "max": 8e-6, "differ": 0.0}
