// fg_path_run: one iteration of the hot path, the sequence of the library's calls that a training loop makes per mini-batch, queued
// from one call. Nothing here computes: it fills in what the calls take and orders two streams by events.
//
// A small iteration is bound by the host that queues it: from Python, a foreign call with 20 to 30 arguments per launch took 66 us for
// an iteration of the smallest workload (10 k nodes, 256 seeds x 10 x 5) whose launches kept the GPU busy for 50. Queued from here the
// host needed 40: step 57 -> 50 us, training iteration 90 -> 78 with the kernels of that time, which was what the GPU needed; with
// fewer and shorter ones it is 33.5 and 62.
#include "update_group.h"

namespace {

#define FG_TRY(call)                  \
    do {                              \
        fg_status_t rc_ = (call);     \
        if (rc_ != FG_OK) return rc_; \
    } while (0)

// an iteration's view of the model's buffers
struct Iter {
    const fg_path_t& P;
    const fg_path_call_t& C;
    const fg_path_lists_t& S;
    int64_t* counts;      // [layers + 1][3]
    int64_t* stats;       // [layers + 1][4]
    int64_t* input_counts;
    int64_t it;
    const fg_path_batch_t* next = nullptr;      // a mini-batch whose top-down pass may run on the second stream behind a selection that goes with the loader
    int32_t *next_pruned = nullptr, *rows_due = nullptr;      // the call's `next_pruned` and `selected`

    Iter(const fg_path_t& p, const fg_path_call_t& c, int64_t iter)
        : P(p), C(c), S(p.lists[iter % 3]), counts(p.counts_log + iter % p.ring * (p.n_layers + 1) * 3), stats(p.stats_log + iter % p.ring * (p.n_layers + 1) * 4),
          input_counts(p.input_log + iter % p.ring * 3), it(iter) {}

    int esz(int code) const { return code == FG_F32 ? 4 : 2; }
    int h_code(int l) const { return l == 0 ? P.feat_dtype : (l < P.n_layers ? P.compute_dtype : (int)FG_F32); }
    int64_t row_bytes(int l) const { return (int64_t)P.dims[l] * esz(h_code(l)); }
    int agg_code() const { return P.compute_dtype == FG_F32 ? FG_F32 : FG_BF16; }
    bool cached() const { return C.cache && P.n_layers > 1; }
    bool gcn() const { return P.model == FG_PATH_GCN; }
    bool one_launch(int l, int64_t n) const { return P.fuse_small_layers && l >= 2 && fg_one_launch_layer(n, P.dims[l - 1], P.dims[l]); }
    // lookup, prune, V_normal for layers L .. 0 (or 1 with the fused loader)
    fg_status_t top_down(const fg_path_batch_t& b, void* stream) const {
        const int L = P.n_layers;
        const bool fused = P.fused_input && !b.reads_rows_once;
        fg_top_down_layer_t y[FG_PATH_MAX_LAYERS + 1] = {};
        int count = 0;
        for (int l = L; l >= (fused ? 1 : 0); --l, ++count) {
            fg_top_down_layer_t& t = y[count];
            const fg_path_layer_t& B = b.layer[l];
            t.cache_layer = cached() && l >= 1 && l < L ? l : 0;
            t.ids_dev = B.ids_dev;
            t.n = (int32_t)B.n;
            t.live_dev = l == L ? nullptr : S.live[l];
            if (l >= 1) {
                t.row_start_dev = B.start_dev;
                t.row_end_dev = B.end_dev;
                t.col_dev = B.col_dev;
                t.nnz = B.nnz;
                t.n_src = (int32_t)b.layer[l - 1].n;
                t.live_src_dev = fused && l == 1 ? nullptr : S.live[l - 1];
            }
            t.hit_dev = S.hit[l];
            t.hit_pos_dev = S.hit_pos[l];
            t.hit_slot_dev = S.hit_slot[l];
            t.normal_pos_dev = S.normal_pos[l];
            t.normal_ids_dev = l == 0 ? S.input_ids : (fused && l == 1 ? S.self_ids : nullptr);
            t.counts_dev = l || !P.fused_input ? counts + 3 * l : input_counts;
            t.n_dev = B.n_dev;
        }
        return fg_top_down(C.cache, it, count, y, P.ws_top_down, P.ws_top_down_bytes, stream);
    }

    void update_specs(const fg_path_batch_t& b, bool own_norms, fg_update_layer_t* y) const {
        for (int l = 1; l < P.n_layers; ++l) {
            fg_update_layer_t& u = y[l - 1];
            u = fg_update_layer_t{};
            u.layer = l;
            u.n = (int32_t)b.layer[l].n;
            u.ids_dev = b.layer[l].ids_dev;
            u.live_dev = S.live[l];
            u.hit_dev = S.hit[l];
            u.gnorm_dev = own_norms ? P.gnorm[l] : b.layer[l].gnorm_dev;
            u.h_dev = P.h[l];
            u.h_stride = row_bytes(l);
            u.stats_dev = stats + 4 * l;
            u.n_dev = b.layer[l].n_dev;
        }
    }
    void* ws_update() const { return (char*)P.ws_update + it % 2 * P.ws_update_stride; }

    // `behind`: layers whose weight gradients may still be under way on the other stream; theirs is the front of the workspace
    // update: described, to ride along
    fg_status_t weight_grads(const fg_path_batch_t& b, int first, int last, void* stream, int behind = 0, const UpdBatch* update = nullptr) const {
        fg_weight_grad_layer_t y[FG_PATH_MAX_LAYERS] = {}, up[FG_PATH_MAX_LAYERS] = {};
        for (int l = first; l <= last; ++l) {
            fg_weight_grad_layer_t& w = y[l - first];
            // (a GCN layer's input rows are the propagated rows: by-position half, then list-order half)
            const int width = gcn() ? P.dims[l - 1] / 2 : P.dims[l - 1], code = gcn() ? (int)FG_F32 : h_code(l - 1);
            w.h_src_dev = gcn() ? P.mean_pos[l] : P.h[l - 1];
            w.src_stride = (int64_t)width * esz(code);
            w.src_dtype = (fg_dtype_t)code;
            w.n_src = (int32_t)(gcn() ? b.layer[l].n : b.layer[l - 1].n);
            w.agg_dev = P.agg[l];
            w.agg_stride = (int64_t)width * esz(agg_code());
            w.dh_dev = P.dh[l];
            w.dh_stride = (int64_t)P.dims[l] * 4;
            if (l < P.n_layers) {
                w.h_dev = P.h[l];
                w.h_stride = row_bytes(l);
            }
            w.rows_dev = S.normal_pos[l];
            w.n_rows_dev = counts + 3 * l + 2;
            w.max_rows = b.layer[l].n;
            w.n = (int32_t)b.layer[l].n;
            w.dw_dev = P.dw[l];
            w.db_dev = P.db[l];
            w.d_in = width;
            w.d_out = P.dims[l];
        }
        for (int i = 0; i < behind; ++i) {
            up[i].max_rows = b.layer[last + 1 + i].n;
            up[i].d_in = gcn() ? P.dims[last + i] / 2 : P.dims[last + i];
            up[i].d_out = P.dims[last + 1 + i];
        }
        size_t front = behind ? fg_backward_weights_all_workspace_bytes((fg_dtype_t)P.compute_dtype, behind, up) : 0;
        if (front > P.ws_weights_bytes) front = P.ws_weights_bytes;      // (refused by the call)
        return fg_backward_weights_with((fg_dtype_t)P.compute_dtype, last - first + 1, y, (char*)P.ws_weights + front, P.ws_weights_bytes - front, update, stream);
    }

    // Whether the weight gradients take longer than the cache update beside them, where it is launches of its own (the figures are from when
    // it always was): 17 us and 18.5 per 10^9 products (in bf16 six times as
    // many) against 25 us and 1.2 per MB of admitted rows, from traces. Iterations with the update / with the weight gradients on the
    // second stream, us: 67 k x 256 x 256 377 / 385, GCN 313 / 317, mixed 16 k x 1536 x 1024 289 / 295, training loop 403 / 414, 30 k x 192 x 144
    // 189 / 198; where the rule says no 31 k x 104 x 88 181 / 175, 34 k x 116 x 64 172 / 166, GCN 37 k x 96 x 256 admitting 0.9 of its rows 194 / 191.
    bool weights_last(const fg_path_batch_t& b) const {
        double products = 0.0, admitted = 0.0;
        for (int l = 1; l <= P.n_layers; ++l) {
            const double n = (double)b.layer[l].n;
            products += n * (gcn() ? 1 : 2) * P.dims[l - 1] * P.dims[l] / (P.compute_dtype == FG_BF16 ? 6.0 : 1.0);
            if (l < P.n_layers) admitted += (double)C.p_grad * n * (double)row_bytes(l);
        }
        return 17.0 + 18.5e-9 * products > 25.0 + 1.2e-6 * admitted;
    }

    // Whether the loader and the dense update of layer 1 are one call: where nobody reads the means and the nodes' own rows later. (A training
    // iteration does; with both written from the one launch it took what the two take, 122 us against 121.)
    // - A row's neighbours have to have a slot (15 of them, 7 of rows of more than 64 values where there are no more than 7 on average), but for two: those
    //   behind the slots are read one by one. The layer by itself, 54 k rows x (128 + 128) x 256, two launches / one, us: 15 each 127 / 114,
    //   8 or 20 122 / 140, 4 or 25 126 / 167, 7 each 90 / 76, 3 or 10 87 / 105; one row of 500 in 500 167 / 357. Steps of blocks with 14 neighbours on average or
    //   fewer, by the most that a row has: 16 6 us faster in one launch, 18 3, 20 5 slower, 25 15 slower; with 7 or fewer on average 8 and 9 4 us
    //   faster, 10 3 slower, 12 9 slower (means of 71 to 273 steps each).
    // - Rows of more than 32 values: half of the operand is padding below that. Step of 71 k positions x 32 x 64, 6 neighbours, 82 / 99; 80 k x 64 96 / 95.
    // - Beside a second stream from 24 Ki positions on: its workgroups fill the chip, so that work there waits for it, and the layers above have to be long
    //   enough to hide that. Steps of positions x columns, us: 20.5 k x 72 77 / 84.5, 24.6 k x 96 83 / 81, x 256 103 / 102, 31 k x 256 119 / 109, 45 k x 96 125 / 117.
    //   Of 4041 steps of 15 k to 110 k positions, 36 to 128 x 64 to 256 values and 5 to 15 neighbours one is the faster one by 10 us on average, and by more
    //   than 5 % the slower one in 140.
    // - On one stream the selection rides with either loader, and what is left is what the layer saves: not where 64 columns or fewer leave
    //   most of its wavefronts without a product, nor for rows of at most 64 values with most positions admitted (their copies are a launch behind it). Of 2374
    //   steps it is faster by 3.5 us on average, with the two exceptions by 5.2, and by more than 5 % the slower one in 16.
    bool loads_and_multiplies(const fg_path_batch_t& b, int l) const {
        const int64_t n = b.layer[1].n, nnz = b.layer[1].nnz, most = b.own_rows_from_table, places = P.dims[0] > 64 && nnz <= 7 * n ? 7 : 15;
        if (l != 1 || !P.fused_input || b.reads_rows_once || !b.col_ids1_dev || most < 2 || most > places + 2) return false;
        if (h_code(0) != FG_F32 || h_code(1) != FG_F32 || P.compute_dtype != FG_F32 || P.dims[0] <= 32) return false;
        if (C.overlap ? n < 24576 : P.dims[1] <= 64 || (P.dims[0] <= 64 && C.p_grad > 0.5f)) return false;
        return fg_tuning(FG_TUNE_LINEAR_TILE) == 0 && fg_one_launch_load(nnz, n, P.dims[0], P.dims[1]) != 0;
    }

    // Whether the selection of a step's update goes with the loader's launch.
    bool selects_with_loader(const fg_path_batch_t& b) const {
        if (!cached() || gcn() || !P.fused_input || b.reads_rows_once || !b.col_ids1_dev || !C.fetch_with_loader) return false;
        if (!(h_code(0) == FG_F32 && agg_code() == FG_F32) && !(h_code(0) == FG_F16 && agg_code() == FG_BF16)) return false;
        int chunks = 0;
        int64_t most = 0;
        for (int l = 1; l < P.n_layers; ++l) {
            const int64_t n = b.layer[l].n;
            chunks += (int)fg_ceil_div(n > 0 ? n : 1, GRP_CHUNK);
            most = n > most ? n : most;
        }
        if (loads_and_multiplies(b, 1)) return chunks <= fg_load_linear_update_chunks;
        return !C.overlap && fg_loader_takes_update(b.layer[1].n, P.dims[0], (fg_dtype_t)h_code(0), most, chunks);
    }

    // The selection has gone with the loader: the index is final for this iteration, and with a second stream the next mini-batch is looked up and pruned
    // there beside the layers above. (What that pass overwrites was last read two iterations ago, in front of the event recorded here. The layers above
    // and the row copies of this iteration are not: the next iteration records them if it puts its selection on the second stream, see fg_path_run.)
    // *due_from: first of the update's layers whose admitted rows are still to be copied. With a second stream layer 1, most of them, is copied there
    // as well, beside the layers above (in the seed layer's launch, whose workgroups take half a compute unit each, 16 k rows took 15 us more: large
    // step 181.3 us, 175.8 so; medium 180.1, 173.7; with the paper's thresholds 164.8, 159.9).
    fg_status_t selected(const fg_update_call* ride, const UpdBatch& selection, int* due_from) const {
        fg_update_selected(*ride);      // the rows are due until all their copies are queued: a call that fails in between leaves a cache that says so
        *rows_due = 1;
        *due_from = 0;
        if (!next) return FG_OK;
        FG_HIP(hipEventRecord((hipEvent_t)P.ev_pruned, (hipStream_t)C.stream));
        FG_HIP(hipStreamWaitEvent((hipStream_t)P.side, (hipEvent_t)P.ev_pruned, 0));
        fg_status_t rc = Iter(P, C, it + 1).top_down(*next, P.side);
        if (rc == FG_OK) {
            fg_row_copy_batch copies;
            fg_update_row_copies(selection, &copies);
            copies.n = 1;
            rc = fg_launch_row_copies(copies, (hipStream_t)P.side);
        }
        FG_HIP(hipEventRecord((hipEvent_t)P.ev_next_pruned, (hipStream_t)P.side));
        if (rc != FG_OK) {      // nobody is told to wait for what did get there
            FG_HIP(hipStreamWaitEvent((hipStream_t)C.stream, (hipEvent_t)P.ev_next_pruned, 0));
            return rc;
        }
        *due_from = 1;
        *next_pruned = 1;
        return FG_OK;
    }

    // the row copies that are due, and about how much they write
    static double due_copies(const UpdBatch& U, int from, fg_row_copy_batch* copies) {
        fg_update_row_copies(U, copies);
        double bytes = 0.0;
        for (int i = from; i < U.n_layers; ++i) {
            copies->c[i - from] = copies->c[i];
            bytes += (double)U.l[i].p_grad * (double)U.l[i].n * (double)U.l[i].row_bytes;
        }
        copies->n = U.n_layers - from;
        return bytes;
    }

    // ride: an update whose selection may go with the loader; *rode: it has. Up to 4 MB of its rows go with a seed layer of one launch: on one stream
    // 0.95 to 1.00 of the time with a launch of their own up to 0.5 MB, 0.99 to 1.00 up to 4, from 6 MB on level (quartiles of 1200 steps; 27 MB
    // took 195 us in one of them, 186 to 190 with their own).
    fg_status_t forward(const fg_path_batch_t& b, bool once, const fg_fetch_layer_t* fetch, int n_fetch, const fg_update_call* ride, const UpdBatch* selection,
                        bool* rode, int* due_from) const {
        const int L = P.n_layers;
        const bool fused = P.fused_input && !once;
        void* st = C.stream;
        const int64_t d0b = row_bytes(0);
        if (!fused)
            FG_TRY(fg_gather(C.feat, P.num_nodes, d0b, d0b, S.input_ids, S.normal_pos[0], (once ? input_counts : counts) + 2, b.layer[0].n, P.h[0],
                             b.layer[0].n, d0b, P.on_host, st));
        for (int l = 1; l <= L; ++l) {
            const fg_path_layer_t& B = b.layer[l];
            const int32_t n = (int32_t)B.n, n_in = (int32_t)b.layer[l - 1].n;
            const int in_code = h_code(l - 1), out_code = h_code(l), relu = l < L ? 1 : 0;
            const int64_t in_b = row_bytes(l - 1), out_b = row_bytes(l), agg_b = (int64_t)P.dims[l - 1] * esz(agg_code()), *n_normal = counts + 3 * l + 2;
            if (gcn()) {
                const int half = P.dims[l - 1] / 2;
                if (fused && l == 1)
                    FG_TRY(fg_gather_aggregate_gcn(B.start_dev, B.end_dev, B.col_dev, B.nnz, n, S.normal_pos[1], n_normal, n, b.layer[0].ids_dev, n_in,
                                                   (const float*)C.feat, P.num_nodes, d0b, P.dims[0], P.mean_pos[1], (float*)P.agg[1], st));
                else
                    FG_TRY(fg_aggregate_gcn(B.start_dev, B.end_dev, B.col_dev, B.nnz, n, S.normal_pos[l], n_normal, n, (const float*)P.h[l - 1], n_in, in_b,
                                            P.dims[l - 1], P.mean_pos[l], (float*)P.agg[l], st));
                FG_TRY(fg_linear(P.mean_pos[l], n, half * 4, FG_F32, P.agg[l], half * 4, S.normal_pos[l], n_normal, n, half, P.dims[l], C.w[l], FG_F32,
                                 C.bias[l], relu, P.h[l], n, out_b, (fg_dtype_t)out_code, st));
                continue;
            }
            if (one_launch(l, B.n)) {
                fg_row_copy_batch copies;
                bool copied = false;
                const bool due = *rode && l == L && *due_from < selection->n_layers && due_copies(*selection, *due_from, &copies) <= 4.0 * 1024.0 * 1024.0;
                FG_TRY(fg_aggregate_linear_with(B.start_dev, B.end_dev, B.col_dev, B.nnz, n, S.normal_pos[l], n_normal, n, (const float*)P.h[l - 1], n_in, in_b,
                                                P.dims[l - 1], P.dims[l], (const float*)C.w[l], C.bias[l], relu, nullptr, agg_b, (float*)P.h[l], n, out_b,
                                                due ? &copies : nullptr, due ? &copied : nullptr, st));
                if (copied) *due_from = selection->n_layers;
                continue;
            }
            const bool own_rows = l == 1 && fused && b.own_rows_from_table;
            if (loads_and_multiplies(b, l)) {
                FG_TRY(fg_gather_aggregate_linear_ids_with(B.start_dev, B.end_dev, b.col_ids1_dev, B.nnz, n, S.normal_pos[1], n_normal, n, B.ids_dev,
                                                           (const float*)C.feat, P.num_nodes, d0b, P.dims[0], P.dims[1], (const float*)C.w[1], C.bias[1], relu,
                                                           (float*)P.agg[1], agg_b, (float*)P.h[1], n, out_b, n_fetch ? C.cache : nullptr, n_fetch,
                                                           n_fetch ? fetch : nullptr, selection, rode, st));
                if (*rode) FG_TRY(selected(ride, *selection, due_from));
                continue;
            }
            if (fused && l == 1) {
                if (b.col_ids1_dev) {
                    FG_TRY(fg_gather_aggregate_ids_with(B.start_dev, B.end_dev, b.col_ids1_dev, B.nnz, n, S.normal_pos[1], n_normal, n, B.ids_dev, C.feat, P.num_nodes, d0b,
                                                        P.dims[0], (fg_dtype_t)in_code, P.agg[1], agg_b, (fg_dtype_t)agg_code(), own_rows ? nullptr : P.h[0], d0b, n_in,
                                                        n_fetch ? C.cache : nullptr, n_fetch, n_fetch ? fetch : nullptr, selection, rode, st));
                    if (*rode) FG_TRY(selected(ride, *selection, due_from));
                } else
                    FG_TRY(fg_gather_aggregate(B.start_dev, B.end_dev, B.col_dev, B.nnz, n, S.normal_pos[1], n_normal, n, b.layer[0].ids_dev, n_in, C.feat,
                                               P.num_nodes, d0b, P.dims[0], (fg_dtype_t)in_code, P.agg[1], agg_b, (fg_dtype_t)agg_code(), P.h[0], d0b, n_in, st));
            } else {
                FG_TRY(fg_aggregate(B.start_dev, B.end_dev, B.col_dev, B.nnz, n, S.normal_pos[l], n_normal, n, P.h[l - 1], n_in, in_b, P.dims[l - 1],
                                    (fg_dtype_t)in_code, P.agg[l], agg_b, (fg_dtype_t)agg_code(), st));
            }
            if (own_rows) {
                FG_TRY(fg_linear_ids(C.feat, (int32_t)P.num_nodes, in_b, (fg_dtype_t)in_code, B.ids_dev, P.agg[1], agg_b, S.normal_pos[1], n_normal, n, P.dims[0],
                                     P.dims[1], C.w[1], (fg_dtype_t)P.compute_dtype, C.bias[1], L > 1 ? 1 : 0, P.h[1], n, out_b, (fg_dtype_t)out_code, st));
                continue;
            }
            FG_TRY((C.wt[l] ? fg_linear_wt : fg_linear)(P.h[l - 1], n_in, in_b, (fg_dtype_t)in_code, P.agg[l], agg_b, S.normal_pos[l], n_normal, n, P.dims[l - 1],
                                                        P.dims[l], C.wt[l] ? C.wt[l] : C.w[l], (fg_dtype_t)P.compute_dtype, C.bias[l], relu, P.h[l], n, out_b,
                                                        (fg_dtype_t)out_code, st));
        }
        return FG_OK;
    }

    // the second stream goes on behind what this one has queued
    fg_status_t side_follows() const {
        FG_HIP(hipEventRecord((hipEvent_t)P.ev_gradients, (hipStream_t)C.stream));
        FG_HIP(hipStreamWaitEvent((hipStream_t)P.side, (hipEvent_t)P.ev_gradients, 0));
        return FG_OK;
    }
    // the embedding gradients and their norms; `ahead`: with the weight gradients of the upper layers on the second stream
    fg_status_t backward(const fg_path_batch_t& b, bool ahead) const {
        const int L = P.n_layers;
        void* st = C.stream;
        FG_TRY(fg_softmax_xent_grad((const float*)P.h[L], (int64_t)P.dims[L] * 4, b.labels_dev, (int32_t)b.layer[L].n, P.dims[L], P.dh[L], (int64_t)P.dims[L] * 4, st));
        const auto layer_backward = gcn() ? fg_layer_backward_gcn : fg_layer_backward;
        for (int l = L; l > 1; --l) {
            if (l == 2 && ahead) {
                FG_TRY(side_follows());
                FG_TRY(weight_grads(b, 2, L, P.side));
            }
            const fg_path_layer_t& B = b.layer[l];
            const int32_t n = (int32_t)B.n, n_in = (int32_t)b.layer[l - 1].n;
            const void* h = l < L ? P.h[l] : nullptr;
            const int64_t h_stride = (int64_t)P.dims[l] * esz(h_code(l)), *n_normal = counts + 3 * l + 2;
            const uint8_t* live = l < L ? S.live[l] : nullptr;
            const int64_t dh_b = (int64_t)P.dims[l] * 4, dh_in_b = (int64_t)P.dims[l - 1] * 4;
            if (!gcn() && P.compute_dtype == FG_BF16)
                FG_TRY(fg_layer_backward_bf16(P.dh[l], dh_b, h, h_stride, n, S.normal_pos[l], n_normal, n, live, S.hit[l], B.start_dev, B.end_dev, B.t_start_dev,
                                              B.t_end_dev, B.t_row_dev, B.nnz, n_in, P.dims[l - 1], P.dims[l], C.w[l], P.dh[l - 1], dh_in_b, P.gnorm[l - 1],
                                              P.ws_backward, P.ws_backward_bytes, st));
            else
                FG_TRY(layer_backward(P.dh[l], dh_b, (const float*)h, h_stride, n, S.normal_pos[l], n_normal, n, live, S.hit[l], B.start_dev, B.end_dev, B.t_start_dev,
                                      B.t_end_dev, B.t_row_dev, B.nnz, n_in, P.dims[l - 1], P.dims[l], (const float*)C.w[l], P.dh[l - 1], dh_in_b, P.gnorm[l - 1],
                                      P.ws_backward, P.ws_backward_bytes, st));
        }
        return FG_OK;
    }
};

fg_status_t check_batch(const fg_path_t& P, const fg_path_batch_t& b) {
    for (int l = 0; l <= P.n_layers; ++l)
        if (b.layer[l].n < 0 || b.layer[l].n > P.n_max[l] || b.layer[l].nnz < 0)
            FG_FAIL(FG_ERR_SHAPE, "fg_path_run: layer %d has %lld positions (%lld edges), its lists hold %d", l, (long long)b.layer[l].n, (long long)b.layer[l].nnz, P.n_max[l]);
    return FG_OK;
}

}  // namespace

extern "C" fg_status_t fg_path_run(const fg_path_t* path, const fg_path_batch_t* batch, const fg_path_batch_t* next, fg_path_call_t* call) {
    if (!path || !batch || !call) FG_FAIL(FG_ERR_INVALID_ARG, "fg_path_run: NULL pointer");
    call->selected = call->next_pruned = call->begun = 0;
    const fg_path_t& P = *path;
    if (P.n_layers < 1 || P.n_layers > FG_PATH_MAX_LAYERS || P.ring < 1) FG_FAIL(FG_ERR_INVALID_ARG, "fg_path_run: n_layers = %d must be in 1..%d", P.n_layers, FG_PATH_MAX_LAYERS);
    if (call->iter < 0) FG_FAIL(FG_ERR_INVALID_ARG, "fg_path_run: iteration %lld is negative", (long long)call->iter);
    FG_TRY(check_batch(P, *batch));
    if (next) FG_TRY(check_batch(P, *next));
    Iter I(P, *call, call->iter);
    const int L = P.n_layers;
    const hipStream_t main = (hipStream_t)call->stream, side = (hipStream_t)P.side;
    const bool do_update = call->update && I.cached();
    if (call->promised) FG_HIP(hipStreamWaitEvent(main, (hipEvent_t)P.ev_next_pruned, 0));      // behind the previous selection on that stream
    auto commit = [&](int64_t iter, int n, const fg_update_layer_t* y) -> fg_status_t {
        FG_TRY(fg_cache_update_commit(call->cache, iter, n, y, (char*)P.ws_update + iter % 2 * P.ws_update_stride, P.ws_update_bytes, main));
        FG_HIP(hipEventRecord((hipEvent_t)P.ev_done[iter % 2], main));
        return FG_OK;
    };
    bool rows_queued = false;
    if (call->due) {      // the rows the previous iteration admitted
        rows_queued = call->promised && fg_update_rows_are_queued(call->cache, call->due_iter);
        if (!call->promised) FG_HIP(hipStreamWaitEvent(main, (hipEvent_t)P.ev_selected, 0));
        if (rows_queued)      // in front of the event just waited for
            fg_update_committed({call->cache, call->due_iter, 0.f, L - 1, call->due, nullptr, 0});
        else
            FG_TRY(commit(call->due_iter, L - 1, call->due));
    }
    call->begun = 1;
    if (!call->pruned_ahead) FG_TRY(I.top_down(*batch, main));
    // With norms from outside the update's selection does not depend on the layers
    UpdBatch selection;
    fg_update_call ride = {};
    bool may_ride = false, rode = false;
    int due_from = 0;
    if (do_update && !P.backward && I.selects_with_loader(*batch)) {
        I.update_specs(*batch, false, call->specs);
        ride = {call->cache, call->iter, call->p_grad, L - 1, call->specs, I.ws_update(), P.ws_update_bytes};
        FG_TRY(fg_update_describe("fg_cache_update_all", ride, &selection, &may_ride));
    }
    const bool beside = do_update && call->overlap && !P.backward && !may_ride;
    if (may_ride && call->overlap) I.next = next;
    I.next_pruned = &call->next_pruned;
    I.rows_due = &call->selected;
    if (beside) {      // the update's selection and the next top-down pass on the second stream
        if (!call->pruned_ahead) {
            FG_HIP(hipEventRecord((hipEvent_t)P.ev_pruned, main));
            FG_HIP(hipStreamWaitEvent(side, (hipEvent_t)P.ev_pruned, 0));
        } else if (rows_queued || !call->due) {
            // Iteration it - 1's selection went with its loader: its layers and row copies have recorded nothing. They are on this stream in front of
            // here (as is a copy that the caller has queued).
            FG_HIP(hipEventRecord((hipEvent_t)P.ev_done[(call->iter + 1) % 2], main));
        }
        // What it overwrites (half it % 2 of the workspace, set (it + 1) % 3 of the lists) was last read by iteration it - 2 and its row copy. If that
        // iteration's rows were left to it - 1, it - 1 recorded this event behind their copy, or behind itself where they had been copied already;
        // else they are in front of a wait of this stream: ev_pruned, of it - 1 or of this iteration.
        FG_HIP(hipStreamWaitEvent(side, (hipEvent_t)P.ev_done[call->iter % 2], 0));
        I.update_specs(*batch, false, call->specs);
        FG_TRY(fg_cache_update_select(call->cache, call->iter, call->p_grad, L - 1, call->specs, I.ws_update(), P.ws_update_bytes, side));
        FG_HIP(hipEventRecord((hipEvent_t)P.ev_selected, side));
        call->selected = 1;
        if (next) {
            const Iter N(P, *call, call->iter + 1);
            FG_TRY(N.top_down(*next, side));
            FG_HIP(hipEventRecord((hipEvent_t)P.ev_next_pruned, side));
            call->next_pruned = 1;
        }
    }
    fg_fetch_layer_t fetch[FG_PATH_MAX_LAYERS] = {};
    const bool once = batch->reads_rows_once != 0, fused = P.fused_input && !once;
    int n_fetch = 0;
    if (I.cached()) {
        for (int l = 1; l < L; ++l) {
            fg_fetch_layer_t& f = fetch[n_fetch++];
            f.layer = l;
            f.hit_slot_dev = I.S.hit_slot[l];
            f.hit_pos_dev = I.S.hit_pos[l];
            f.n_hit_dev = I.counts + 3 * l + 1;
            f.max_hits = f.h_rows = batch->layer[l].n;
            f.h_dev = P.h[l];
            f.h_stride = I.row_bytes(l);
        }
        if (!(call->fetch_with_loader && fused && !I.gcn() && batch->col_ids1_dev)) {      // else the id-column loader takes the fetch along
            FG_TRY(fg_cache_fetch_all(call->cache, n_fetch, fetch, main));
            n_fetch = 0;
        }
    }
    FG_TRY(I.forward(*batch, once, fetch, n_fetch, &ride, may_ride ? &selection : nullptr, &rode, &due_from));
    if (rode) {
        if (due_from < selection.n_layers) {
            fg_row_copy_batch copies;
            Iter::due_copies(selection, due_from, &copies);
            FG_TRY(fg_launch_row_copies(copies, main));
        }
        if (call->next_pruned) {      // some of the copies are on the second stream
            fg_update_rows_queued(ride, P.ev_next_pruned);
        } else {
            fg_update_committed(ride);
            call->selected = 0;
        }
        return FG_OK;
    }
    // A training iteration ends with its weight gradients and the cache update beside each other: in the same two launches where a group of
    // workgroups decides the update, else on two streams, the longer of the two on this one, where it does not wait for an event to be
    // seen by the other.
    const bool train = P.backward && P.weight_grads, two_streams = train && call->overlap, ahead = two_streams && call->ahead && L > 1;
    if (P.backward) FG_TRY(I.backward(*batch, ahead));
    if (train && do_update && !call->selected) {
        I.update_specs(*batch, true, call->specs);
        const fg_update_call u = {call->cache, call->iter, call->p_grad, L - 1, call->specs, I.ws_update(), P.ws_update_bytes};
        UpdBatch U;
        bool rides;
        FG_TRY(fg_update_describe("fg_cache_update_all", u, &U, &rides));
        if (rides) {
            FG_TRY(I.weight_grads(*batch, 1, ahead ? 1 : L, main, ahead ? L - 1 : 0, &U));
            fg_update_queued(u);
            if (ahead) {
                FG_HIP(hipEventRecord((hipEvent_t)P.ev_weights, side));
                FG_HIP(hipStreamWaitEvent(main, (hipEvent_t)P.ev_weights, 0));
            }
            return FG_OK;
        }
    }
    const bool update_beside = two_streams && do_update && I.weights_last(*batch), weights_beside = two_streams && !update_beside;
    if (two_streams) FG_TRY(I.side_follows());
    if (train) FG_TRY(I.weight_grads(*batch, 1, ahead ? 1 : L, weights_beside ? side : main, ahead ? L - 1 : 0));
    if (call->selected) {      // only the admitted rows are left to copy: by the next call, if its top-down pass is on the second stream
        if (!call->next_pruned) {
            FG_HIP(hipStreamWaitEvent(main, (hipEvent_t)P.ev_selected, 0));
            FG_TRY(commit(call->iter, L - 1, call->specs));
            call->selected = 0;
        }
    } else if (do_update) {
        I.update_specs(*batch, P.backward != 0, call->specs);
        FG_TRY(fg_cache_update_all(call->cache, call->iter, call->p_grad, L - 1, call->specs, I.ws_update(), P.ws_update_bytes, update_beside ? side : main));
    }
    if (two_streams) {      // the next iteration reads the cache, and overwrites what the weight gradients read
        FG_HIP(hipEventRecord((hipEvent_t)P.ev_weights, side));
        FG_HIP(hipStreamWaitEvent(main, (hipEvent_t)P.ev_weights, 0));
    }
    return FG_OK;
}

// These order streams of one device. A kernel's end already makes what it wrote visible to the whole device; without the flag a record
// also writes the caches back for the host and the other devices and the stream stands still for it, 5 to 7 us behind every record
// (large step 213 -> 210 us, its training iteration 2.5 % and its training loop 4 % faster).
extern "C" fg_status_t fg_event_create(void** event) {
    if (!event) FG_FAIL(FG_ERR_INVALID_ARG, "fg_event_create: NULL pointer");
    FG_HIP(hipEventCreateWithFlags((hipEvent_t*)event, hipEventDisableTiming | hipEventDisableSystemFence));
    return FG_OK;
}

extern "C" fg_status_t fg_event_record(void* event, void* stream) {
    FG_HIP(hipEventRecord((hipEvent_t)event, (hipStream_t)stream));
    return FG_OK;
}

extern "C" fg_status_t fg_stream_wait_event(void* stream, void* event) {
    FG_HIP(hipStreamWaitEvent((hipStream_t)stream, (hipEvent_t)event, 0));
    return FG_OK;
}

extern "C" fg_status_t fg_event_destroy(void* event) {
    FG_HIP(hipEventDestroy((hipEvent_t)event));
    return FG_OK;
}
