"""Phase-parallel epoch loop over the C ABI (the paper's phase-parallel algorithm, one GPU).

Sequencing only: every partition step, the scale-and-reduce and the optimizer step are
library calls; the partitions of a phase are independent of each other, so they are processed
in turn on the one GPU, on several HIP streams (``streams`` > 1), or, where they are small enough to be bound by the number of
their launches, in merged launches; their gradients are kept resident for the reduction.
"""
from __future__ import annotations

import torch

from . import binding as g
from .controller import Controller


# Full-graph steps are merged, at most MERGE_STEPS at a time, while a step's workspace is at most this large (each merged step needs one of
# its own, so this also bounds the memory).  A workspace holds the partial sums of every layer, at most 512 tiles of 64 KiB and their column
# sums, whatever the number of rows: a further layer counts for them, as it does not make the launches longer.  Eight steps on R-MAT graphs of
# 10 edges a row, one by one / merged by two / four / eight, us, workspace of one step:
#   GraphSAGE 100-256-256-47     60 MiB 1496/919/654/529       164 MiB 2524/2056/1773/1675   409 MiB 5581/4912/4569/4366   543 MiB 7307/6512/6148/5987
#     eight layers, 256 wide    178 MiB 5043/3503/2692/2214    455 MiB 9020/7500/6692/6349   683 MiB 14129/12509/11602/11225
#   GCN 64-128-16                14 MiB 676/385/225/148        142 MiB 1654/1267/1085/1032
#     eight layers, 64 wide      27 MiB 2214/1428/947/706      184 MiB 6292/4398/3477/3057
# From 2^16 rows on products are large launches, and a step that makes them is not merged (744 MiB of three layers 9580/9599/9601/9593); what the
# limit keeps from it is wide models of many layers, for their memory's sake (eight layers on uniform graphs, 973 MiB 20101/18916/18149/17702).
MERGE_WORKSPACE_BYTES = 512 << 20
MERGE_LAYER_BYTES = 34 << 20
MERGE_STEPS = 8


def _groups(active, most):
    """(slot, partition) of a phase, in runs of at most ``most``."""
    slots = list(enumerate(active))
    return [slots[lo:lo + most] for lo in range(0, len(slots), most)]


class PhaseParallelTrainer:
    """Holds theta, the optimizer state and the per-partition buffers across phases.

    ``parts``: list of ``Partition``; ``xs`` / ``ys`` / ``masks``: per-partition device
    tensors (features, int32 labels, uint8 train mask or None).  ``max_active`` = M, the
    number of partitions per phase.  Full-graph mode (one iteration per phase and epoch).
    ``dropout_rate`` / ``dropout_seed``: hidden-layer dropout; the masks of a phase are drawn with
    batch_id = the number of optimizer steps taken so far.
    ``streams``: number of streams (default priority) the steps of a phase are spread over, each with a
    workspace of its own; 1 = everything on the current stream, small steps in merged launches.  The result does not depend on it.
    """

    def __init__(self, parts, model, xs, ys, masks, theta0, estimator, max_active, optimizer=None,
                 dropout_rate=0.0, dropout_seed=0, streams=1):
        self.parts, self.model, self.xs, self.ys, self.masks = parts, model, xs, ys, masks
        self.estimator, self.max_active = estimator, max_active
        self.opt = optimizer if optimizer is not None else g.optimizer_desc()
        dev = theta0.device
        self.P = g.grp_param_count(model)
        self.ld = (self.P + 3) // 4 * 4
        self.theta = theta0.detach().clone().to(torch.float32).contiguous()
        self.m = torch.zeros(self.P, device=dev)
        self.v = torch.zeros(self.P, device=dev)
        self.update = torch.zeros(self.P, device=dev)
        self.opts = g.step_opts(estimator=estimator, full_graph=True, dropout_rate=dropout_rate,
                                dropout_seed=dropout_seed)
        self.grads = torch.zeros(max_active, self.ld, device=dev)
        self.stats = g.new_stats(max_active, device=dev)
        ws_bytes = max(g.grp_step_workspace_bytes(p, model, self.opts) for p in parts)
        n_lanes = max(1, min(int(streams), max_active))
        self.side = [torch.cuda.Stream(device=dev) for _ in range(n_lanes)] if n_lanes > 1 else []
        merge_bytes = MERGE_WORKSPACE_BYTES + MERGE_LAYER_BYTES * (model.n_layers - 1)
        if not self.side and ws_bytes <= merge_bytes and model.arch != g.ARCH_GAT:      # (an attention model's steps are not merged)
            n_lanes = min(MERGE_STEPS, max_active)
        self.ws = [torch.empty(ws_bytes, dtype=torch.uint8, device=dev) for _ in range(n_lanes)]
        self.step_count = 0
        self.history = []          # per optimizer step: device tensor views are copied lazily

    def phases(self):
        K, M = len(self.parts), self.max_active
        return [list(range(lo, min(K, lo + M))) for lo in range(0, K, M)]

    def run_phase(self, active):
        self.opts.batch_id = self.step_count
        record = lambda slot: self.stats[slot * g.STATS_BYTES:(slot + 1) * g.STATS_BYTES]
        if self.side:
            main = torch.cuda.current_stream()
            ready = main.record_event()
            for st in self.side:      # the side streams start once theta (and everything before) is ready
                st.wait_event(ready)
            for slot, p in enumerate(active):
                lane = slot % len(self.ws)
                g.grp_train_step(self.parts[p], self.model, self.opts, self.xs[p], self.ys[p], self.masks[p], self.theta, self.ws[lane],
                                 self.grads[slot], record(slot), stream=self.side[lane])
            for st in self.side:      # the reduction waits for every step
                main.wait_stream(st)
        else:
            for group in _groups(active, len(self.ws)):
                g.grp_train_steps([self.parts[p] for _, p in group], self.model, [self.opts] * len(group), [self.xs[p] for _, p in group],
                                  [self.ys[p] for _, p in group], [self.masks[p] for _, p in group], self.theta, self.ws[:len(group)],
                                  [self.grads[slot] for slot, _ in group], [record(slot) for slot, _ in group])
        g.grp_aggregate(self.grads, self.ld, self.stats, len(active), self.P, self.estimator, self.update)
        self.step_count += 1
        g.grp_optimizer_step(self.opt, self.P, self.step_count, self.theta, self.update, self.m, self.v)
        self.history.append(self.stats[:len(active) * g.STATS_BYTES].clone())

    def run_epoch(self):
        for active in self.phases():
            self.run_phase(active)

    def losses(self):
        """Mean loss of the active partitions for every optimizer step so far (host floats)."""
        return [float(g.read_stats(h)["loss"].mean()) for h in self.history]


class MiniBatchTrainer:
    """The phase-parallel loop in mini-batch mode (GraphSAGE): every epoch each partition visits its
    training nodes once in the order ``grp_epoch_seeds`` gives, ``batch_size`` seeds per iteration; an epoch
    has as many iterations as the partition with the most training nodes needs, and a partition whose
    nodes are used up takes part with a zero gradient that still counts in the average.  The sampler's
    batch_id is the number of iterations done so far (``iteration``).  Within an iteration the phases run as
    in ``PhaseParallelTrainer``.  Sequencing only: the seed order, sampling, steps, reduction and update
    are library calls.
    ``lanes``: the steps of a phase are independent, and a mini-batch step is a chain of ~40 small launches
    that leaves most of the chip idle; that many steps (each with a workspace of its own) are made with merged launches.
    The result does not depend on it.
    ``graphs``: the steps of every such group of partitions are captured once in a HIP graph (full batches; the seeds and the
    batch id are read from device buffers that are rewritten before each replay), so an iteration costs the
    host three launches instead of ~40.  A group that has a batch shorter than ``batch_size`` among its steps runs uncaptured, in merged
    launches (replaying a graph of the others beside it is slower: partitions of 1000 to 15 000 training nodes, an epoch in 8 lanes 11.4 against
    8.7 ms).  Same bits as without.
    """

    def __init__(self, parts, model, xs, ys, masks, theta0, estimator, max_active, batch_size, fanouts,
                 sampler_seed, optimizer=None, dropout_rate=0.0, dropout_seed=0, lanes=1, graphs=False):
        self.dropout_rate, self.dropout_seed = dropout_rate, dropout_seed
        self.parts, self.model, self.xs, self.ys, self.masks = parts, model, xs, ys, masks
        self.estimator, self.max_active = estimator, max_active
        self.batch_size, self.fanouts, self.sampler_seed = int(batch_size), tuple(fanouts), sampler_seed
        self.opt = optimizer if optimizer is not None else g.optimizer_desc()
        dev = theta0.device
        self.P = g.grp_param_count(model)
        self.ld = (self.P + 3) // 4 * 4
        self.theta = theta0.detach().clone().to(torch.float32).contiguous()
        self.m = torch.zeros(self.P, device=dev)
        self.v = torch.zeros(self.P, device=dev)
        self.update = torch.zeros(self.P, device=dev)
        self.grads = torch.zeros(max_active, self.ld, device=dev)
        self.stats = g.new_stats(max_active, device=dev)
        width = (max(max(p.n for p in parts), 1) + 63) // 64 * 64
        self.all_seeds = torch.zeros(len(parts), width, dtype=torch.int32, device=dev)
        self.seeds = [self.all_seeds[i, :max(p.n, 1)] for i, p in enumerate(parts)]
        self.n_train = [g.grp_epoch_seeds(p, mk, sampler_seed, 0, sd) for p, mk, sd in zip(parts, masks, self.seeds)]
        self.iters = max(1, max(-(-c // self.batch_size) for c in self.n_train))
        probe = g.step_opts(estimator=estimator, full_graph=False, seeds=self.seeds[0][:1], fanouts=self.fanouts)
        ws_bytes = 0
        for p, sd, c in zip(parts, self.seeds, self.n_train):       # the workspace is sized from the seed count alone
            probe.n_seeds = max(1, min(self.batch_size, c))
            ws_bytes = max(ws_bytes, g.grp_step_workspace_bytes(p, model, probe))
        n_lanes = max(1, min(int(lanes), max_active))
        self.ws = [torch.empty(ws_bytes, dtype=torch.uint8, device=dev) for _ in range(n_lanes)]
        self.graphs = bool(graphs)
        self.side = torch.cuda.Stream(device=dev) if self.graphs else None     # where steps are captured
        self.bid_dev = torch.zeros(1, dtype=torch.int64, device=dev)          # the batch id of the captured steps
        self.batch_seeds = torch.zeros(len(parts), self.batch_size, dtype=torch.int32, device=dev) if self.graphs else None
        self.captured = {}                                                     # partition -> the graph of its group's steps
        self.step_count = 0
        self.epoch = 0
        self.iteration = 0
        self.history = []

    def phases(self):
        K, M = len(self.parts), self.max_active
        return [list(range(lo, min(K, lo + M))) for lo in range(0, K, M)]

    def run_epoch(self):
        B = self.batch_size
        counts = [g.grp_epoch_seeds(p, mk, self.sampler_seed, self.epoch, sd)
                  for p, mk, sd in zip(self.parts, self.masks, self.seeds)]
        assert counts == self.n_train

        def steps(group, opts):                        # the steps of a group, in merged launches
            g.grp_train_steps([self.parts[p] for _, p in group], self.model, opts, [self.xs[p] for _, p in group],
                              [self.ys[p] for _, p in group], None, self.theta, self.ws[:len(group)], [self.grads[slot] for slot, _ in group],
                              [self.stats[slot * g.STATS_BYTES:(slot + 1) * g.STATS_BYTES] for slot, _ in group])

        def uncaptured(group, it):
            live, opts = [], []
            for slot, p in group:
                lo, hi = it * B, min((it + 1) * B, counts[p])
                if hi <= lo:                               # no seeds left: a zero gradient and an empty record
                    self.grads[slot].zero_()
                    self.stats[slot * g.STATS_BYTES:(slot + 1) * g.STATS_BYTES].zero_()
                    continue
                live.append((slot, p))
                opts.append(g.step_opts(estimator=self.estimator, full_graph=False, seeds=self.seeds[p][lo:hi], fanouts=self.fanouts,
                                        sampler_seed=self.sampler_seed, batch_id=self.iteration, dropout_rate=self.dropout_rate,
                                        dropout_seed=self.dropout_seed))
            if live:
                steps(live, opts)

        def replay(group):                                 # (captured at first use)
            first = group[0][1]
            if first not in self.captured:
                opts = [g.step_opts(estimator=self.estimator, full_graph=False, seeds=self.batch_seeds[p], fanouts=self.fanouts,
                                    sampler_seed=self.sampler_seed, batch_id_dev=self.bid_dev, dropout_rate=self.dropout_rate,
                                    dropout_seed=self.dropout_seed) for _, p in group]
                main = torch.cuda.current_stream()
                self.side.wait_stream(main)
                with torch.cuda.stream(self.side):         # once uncaptured first: nothing lazy (a kernel's first load) is left for the capture
                    steps(group, opts)
                main.wait_stream(self.side)
                graph = torch.cuda.CUDAGraph()
                torch.cuda.synchronize()
                with torch.cuda.graph(graph, stream=self.side):
                    steps(group, opts)
                for _, p in group:
                    self.captured[p] = (graph, opts)
            self.captured[first][0].replay()

        for it in range(self.iters):
            lo, hi = it * B, (it + 1) * B
            if self.graphs:
                self.bid_dev.fill_(self.iteration)
            for active in self.phases():
                groups = _groups(active, len(self.ws))
                full = [self.graphs and all(hi <= counts[p] for _, p in group) for group in groups]
                if any(full):                              # the phase's seeds in one copy (rows without a full batch are not read)
                    a, z = active[0], active[-1] + 1
                    width = min(hi, self.all_seeds.shape[1]) - lo
                    self.batch_seeds[a:z, :width].copy_(self.all_seeds[a:z, lo:lo + width])
                for group, whole in zip(groups, full):
                    replay(group) if whole else uncaptured(group, it)
                g.grp_aggregate(self.grads, self.ld, self.stats, len(active), self.P, self.estimator, self.update)
                self.step_count += 1
                g.grp_optimizer_step(self.opt, self.P, self.step_count, self.theta, self.update, self.m, self.v)
                self.history.append(self.stats[:len(active) * g.STATS_BYTES].clone())
            self.iteration += 1
        self.epoch += 1

    def losses(self):
        return [float(g.read_stats(h)["loss"].mean()) for h in self.history]


class SweepingTrainer:
    """Phase-parallel training over sweeping partitions: the graph is split once into chunks
    (``grp_chunks_build``); every super-epoch each worker's partition base + swept chunk is
    rebuilt on the GPU (``grp_partition_from_chunks``) and its rows of the global feature /
    label / mask tensors are gathered by ``l2g``; the controller decides after each epoch
    whether to switch.  theta and the optimizer state persist across super-epochs.
    ``minibatch = dict(batch_size=, fanouts=, sampler_seed=[, lanes=, graphs=])``: every epoch is a mini-batch epoch
    (``MiniBatchTrainer``) over the current partitions; the epoch number and the iteration count run on
    across super-epochs.
    """

    def __init__(self, src, dst, n_nodes, n_chunks, chunk_seed, model, x, y, train_mask, theta0, estimator,
                 max_active, total_epochs, optimizer=None, controller=None, dropout_rate=0.0, dropout_seed=0,
                 minibatch=None):
        self.minibatch = minibatch
        self.iteration = 0
        self.chunks = g.grp_chunks_build(src, dst, n_nodes, n_chunks, chunk_seed)
        self.dropout_rate, self.dropout_seed = dropout_rate, dropout_seed
        self.model, self.x, self.y, self.train_mask = model, x, y, train_mask
        self.estimator, self.max_active = estimator, max_active
        self.opt = optimizer if optimizer is not None else g.optimizer_desc()
        self.ctl = controller if controller is not None else Controller(total_epochs, n_chunks)
        self.theta = theta0.detach().clone().to(torch.float32).contiguous()
        P = g.grp_param_count(model)
        self.m = torch.zeros(P, device=self.theta.device)
        self.v = torch.zeros(P, device=self.theta.device)
        self.step_count = 0
        self.inner = None
        self.switches = []
        self.epoch = 0
        self._losses = []

    def _build(self):
        parts, xs, ys, masks = [], [], [], []
        for base, swept in self.ctl.pairs():
            part = g.grp_partition_from_chunks(self.chunks, base, swept)
            l2g = torch.from_numpy(part.array("l2g")).to(self.x.device)
            mask = torch.from_numpy(part.base_mask()).to(self.x.device)
            if self.train_mask is not None:            # the training nodes among the base chunk's nodes
                mask = g.grp_gather_rows(self.train_mask, l2g, keep=mask)
            parts.append(part)
            xs.append(g.grp_gather_rows(self.x, l2g))  # this worker's rows of the global tensors
            ys.append(g.grp_gather_rows(self.y, l2g))
            masks.append(mask)
        if self.minibatch is not None:
            mb = self.minibatch
            tr = MiniBatchTrainer(parts, self.model, xs, ys, masks, self.theta, self.estimator, self.max_active,
                                  mb["batch_size"], mb["fanouts"], mb["sampler_seed"], self.opt,
                                  dropout_rate=self.dropout_rate, dropout_seed=self.dropout_seed, lanes=mb.get("lanes", 1),
                                  graphs=mb.get("graphs", False))
            tr.epoch, tr.iteration = self.epoch, self.iteration
        else:
            tr = PhaseParallelTrainer(parts, self.model, xs, ys, masks, self.theta, self.estimator, self.max_active, self.opt,
                                      dropout_rate=self.dropout_rate, dropout_seed=self.dropout_seed)
        tr.theta, tr.m, tr.v, tr.step_count = self.theta, self.m, self.v, self.step_count   # carried state
        return tr

    def run_epoch(self):
        if self.inner is None:
            self.inner = self._build()
        first = len(self.inner.history)
        self.inner.run_epoch()
        self.step_count = self.inner.step_count
        if self.minibatch is not None:
            self.iteration = self.inner.iteration
        for h in self.inner.history[first:]:
            rec = g.read_stats(h)
            self._losses.append(float(rec["loss"].mean()))
            self.ctl.observe_stats(rec)                   # the deficit is derived from the records inside the library
        if self.ctl.end_epoch():
            self.switches.append(self.epoch)
            for p in self.inner.parts:
                p.destroy()
            self.inner = None
        self.epoch += 1

    def losses(self):
        return list(self._losses)
