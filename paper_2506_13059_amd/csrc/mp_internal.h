// Host-side declarations shared by the kernel translation units and the C-ABI layer.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mp {

// ------------------------------------------------------------------------------------------------
// Value pass: streams rows (keys + values, or value centroids with ready-made scores) and produces
// one online-softmax partial (m, l, acc[128]) per (unit, chunk, head).  A stream may be cut into two
// sources with different chunk sizes (large chunks first, small ones last) to shorten the drain.
// ------------------------------------------------------------------------------------------------
constexpr int kChunkRowsMin = 512;     // smallest chunk of the dense kernel: 4 waves, one strip of 128 rows each
constexpr int kPartStride = 132;       // floats per (unit, chunk, head): m, l, pad, pad, acc[128]
constexpr int kMaxSources = 4;
constexpr float kSmallScale = 0x1p-80f, kLargeScale = 0x1p30f;      // (see mp_stream8.hip)

// One stream of rows.  Row j of unit u lives at K + (u*unit_rows + idx)*128 (elements) where idx = rows ?
// rows[u*rows_stride + j] : j.  The number of rows is *count_dev (clamped to count_max) or count_max.
struct RowSource {
    const uint16_t* K;         // bf16 keys; unused when scores != nullptr
    const uint16_t* V;         // bf16 values (or value centroids)
    long long unit_rows;       // rows per unit in K / V
    const int32_t* rows;       // optional gather list
    long long rows_stride;     // entries per unit in rows / scores
    const int32_t* count_dev;  // optional per-unit row count on the device
    int32_t count_max;         // upper bound of the row count (fixes the chunk count)
    const float* scores;       // optional [U, rows_stride, G] ready-made logits in log2 units
    // optional, all three or none: K and V hold 128-byte rows of e4m3 codes; the value row idx stands for
    // code * row_scale[idx][1], the key row for (its cluster's centroid) + code * row_scale[idx][0], and the
    // centroid's share of the logit is read ready-made: slot_base[row_slot[j]] for list position j.  count_dev[n_units] is
    // not zero if any row has had a value scale outside [kSmallScale, kLargeScale)
    const float* row_scale;    // [U, unit_rows, 2]
    const int32_t* row_slot;   // [U, rows_stride]
    const float* slot_base;    // [U, base_stride, 8] log2 units, column layout as written by the scoring kernel
    long long base_stride;
    int32_t chunk0;            // first chunk id of this source inside a unit
    int32_t n_chunks;          // ceil(count_max / chunk_rows)
    int32_t chunk_rows;        // rows per workgroup of this source, a multiple of 64
    int32_t row0;              // first list position this source covers: [row0, row0 + count_max)
    int32_t guest;             // 1: src[0] of the launch, a scored source with n_chunks == 0, rides along: its rows
                               // are shared out evenly over this source's chunks
};

struct ValuePassParams {
    const uint16_t* q;         // bf16 [U*G, 128]
    float* partials;           // [U, chunks_per_unit, G, kPartStride]
    int32_t n_units;
    int32_t chunks_per_unit;
    int32_t n_sources;
    float scale_log2e;         // softmax scale * log2(e)
    RowSource src[kMaxSources];
};

hipError_t launch_value_pass(const ValuePassParams& p, int G, hipStream_t stream);
// The same launch on the matrix cores: bf16 rows that start on 16 bytes, chunk_rows a multiple of 64.
hipError_t launch_value_stream(const ValuePassParams& p, int G, hipStream_t stream);
// ... of one source of rows in order, all of them (dense calls).
hipError_t launch_value_dense(const ValuePassParams& p, int G, hipStream_t stream);
// ... of a decode step whose centroid terms ride along with its selected keys: they have a wave of their own.
hipError_t launch_value_terms(const ValuePassParams& p, int G, hipStream_t stream);
// ... of which one source's rows are listed 8-bit rows.
hipError_t launch_value_stream8(const ValuePassParams& p, int G, hipStream_t stream);

// Merge of the partials of a unit into the output: out bf16 [U*G, 128], lse fp32 [U*G] (optional).
hipError_t launch_merge(const float* partials, int n_units, int chunks_per_unit, int G, uint16_t* out,
                        float* lse, hipStream_t stream);

// ------------------------------------------------------------------------------------------------
// Centroid scoring + budgeted selection (one launch per level)
// ------------------------------------------------------------------------------------------------
struct ScoreParams {
    const uint16_t* q;          // bf16 [U*G, 128]
    const uint16_t* Kc;         // bf16 [U, tab_rows, 128]: fine rows, then coarse rows from row fcap
    const int32_t* N;           // [U, tab_rows]
    long long tab_rows;
    int fcap;
    int levels, n_fine, n_coarse;
    long long key_budget, coarse_budget;
    double scale;
    const int32_t* cstart;      // [U, cstart_stride] first child of each coarse cluster
    long long cstart_stride;
    const int32_t* fstart;      // [U, fstart_stride] first stored row of each fine cluster
    long long fstart_stride;
    // working arrays in global memory, used by a level with more than lds_cap entries
    double* lg;                 // [U, G, lg_stride]
    long long lg_stride;
    unsigned long long* g_keys; // [U, g_stride]
    uint32_t* g_wts;
    int32_t* g_ids;
    int32_t* g_aux;
    int32_t* g_aux2;
    uint8_t* g_flags;
    long long g_stride;
    // per-position views of the last call (for the getters): the key each entry was ranked by (all
    // ones: took no part) and, per unit and level, what the keys are (key_mode, see launch_scatter_selection)
    unsigned long long* key_c;  // [U, c_stride] coarse
    uint8_t* flag_c;            // [U, c_stride] promising
    long long c_stride;
    unsigned long long* key_f;  // [U, f_stride] fine, by candidate position
    uint8_t* flag_f;            // [U, f_stride] selected, by candidate position
    long long f_stride;
    int32_t* key_mode;          // [U, 2] coarse, fine
    int32_t* cand;              // [U, f_stride] candidate fine ids (two levels)
    int32_t* n_cand;            // [U]
    // outputs for the value pass
    int32_t* rows;              // [U, rows_stride] stored rows of the selected keys
    long long rows_stride;
    int32_t* n_rows;            // [U]
    // optional (both or none; keys stored as residuals from their cluster's centroid): per selected cluster, in
    // the order of a compact list, q . centroid in log2 units, eight columns (see fine_epilogue), and per row of
    // `rows` the position of its cluster in that list
    float* sel_base;            // [U, f_stride, 8]
    int32_t* row_slot;          // [U, rows_stride]
    int32_t* mp_rows;           // [U, mp_stride] centroid-table row of each centroid term
    float* mp_scores;           // [U, mp_stride, G] (l + ln N) * log2(e)
    long long mp_stride;
    int32_t* n_mp;              // [U]
    int use_mp;
    int32_t* counters;          // [U, 4]
    int n_tail;
    // optional (two levels): workgroups per unit that work out e^l and the logits of all fine clusters while the coarse level
    // is being scored (early_logits in mp_score.hip): how many, what they leave, and per unit how many of them are done -- zero
    // before and after a launch
    int helpers;
    double* early;              // [U, early_stride, 2, heads in fours] logits, then e^l of a fine cluster
    long long early_stride;
    int32_t* early_done;        // [U]
    // optional: rows the caller hands over with this step (a generation loop's new token) are copied
    // into the tail buffers by the workgroup of their unit before anything else; the value pass,
    // a later launch, then finds them there.  app_n arrays (0 = none), 256-byte rows.
    int app_n;
    const void* app_src[3];     // [U, 128] bf16 each
    void* app_dst[3];           // [U, app_dst_rows, 128] bf16 each
    long long app_dst_rows;
    int app_row;
    int lds_cap;                // entries of a level that fit the LDS working arrays
    int G, U;
};

// n_compute_units: of the device the launch goes to (decides whether units get a second, shadow workgroup).  helpers_run: no where
// (tests) units' workgroups take what the helpers of the launch before left.
hipError_t launch_score_select(const ScoreParams& p, int n_compute_units, bool helpers_run, hipStream_t stream);
size_t score_smem_bytes(int G, int cap);

// Later assignment steps of a Lloyd sequence mark the points that may have changed cluster: bit i of marks[u][first_mark(x0,
// b) + c] stands for point x0 + 64 c + i of block b.  Every word of a block is written; no array: nothing is marked.
struct MoveMarks {
    const int32_t* old_ids;        // [U, assign_stride] the assignment before
    unsigned long long* marks;     // [U, stride]
    long long stride;
    const int32_t* moved_before;   // [U, cnt_stride]: did the step before move a point of block b?  If none, its centroids are as they
                                   // were, and so is the assignment.  (no array: they may have changed in any case)
    int32_t* moved_now;            // the same of this step, cleared here and set by launch_move_means
};
// What an assignment step leaves for the next one, which then has to look at the centroids that have changed only: per point, the
// score of its cluster's centroid and a bound on the scores of all others (see assign_changed_kernel).
struct AssignState {
    float2* scores;                // [U, stride] by point; none: nothing is kept
    long long stride;
    const uint32_t* changed;       // [U, changed_stride] by cluster: did its centroid change since the step that left `scores`?
    long long changed_stride;      // (no array: the step looks at all centroids)
};
// Blocks of at most max_pts points and max_k centroids: whether their centroids stay in LDS, and whether steps keep and use such
// a state.  (In smaller blocks a step is a chain of latencies, and that with a state is no shorter: builds of five iterations, us,
// without / with: 1500 points x 93 centroids, 6 blocks 186 / 193; 1024 x 32, 24 blocks 187 / 194; 2000 x 60, 1 block 139.5 / 143, 64
// blocks 277 / 265; 8192 x 256, 1 block 194 / 177; 8192 x 512, 64 blocks 977 / 911.)
constexpr int kResidentMaxK = 512;
constexpr bool assign_is_resident(int max_pts, int max_k) { return max_k > 0 && max_k <= kResidentMaxK && max_pts >= 1024; }
constexpr bool assign_keeps_state(int max_pts, int max_k) { return assign_is_resident(max_pts, max_k) && (long long)max_pts * max_k >= 1 << 20; }
constexpr int first_mark(int x0, int b) { return (x0 >> 6) + b; }
inline long long marks_of(long long points, int blocks) { return (points >> 6) + blocks + 1; }
// ------------------------------------------------------------------------------------------------
// Index construction helpers (member lists, gathers, per-cluster means)
// ------------------------------------------------------------------------------------------------
// Nearest-centroid assignment (fp64 definition, lowest index among equal distances) of the points of
// nb blocks per unit.  blocks_dev: int32 [nb][4] = {first point, end point, first centroid, end
// centroid}; assign[u][t] receives the centroid row of point t.  amb_list [U, list_stride] (at least
// as long as the point range) and amb_cnt [U, cnt_stride >= nb] are workspace; amb_cnt must be all zero on
// entry, and the call leaves amb_cnt_next [U, cnt_stride] all zero for the next one (two arrays used in turn
// save a fill launch per step).  max_pts / max_k: the
// largest point / centroid count of a block (max_k = 0: not known; it only selects the kernel).
hipError_t launch_assign(const uint16_t* X, long long x_unit_rows, const int32_t* blocks_dev, int nb, int max_pts,
                         int max_k, int U, const uint16_t* C, long long c_unit_rows, int32_t* assign,
                         long long assign_stride, int32_t* amb_list, long long list_stride, int32_t* amb_cnt,
                         int32_t* amb_cnt_next, int cnt_stride, const MoveMarks& mv, const AssignState& st, hipStream_t s);
// The coarse level of a range of blocks in one launch: `iters` Lloyd iterations over the fine working centroids X of each
// block, then the fine clusters in their new order.  blocks: int32 [nb][4] = {first fine id, end, first coarse id, end}.
struct CoarseLevel {
    const uint16_t* X;           // bf16 [U, x_unit_rows, 128] by fine id
    long long x_unit_rows;
    const int32_t* blocks;
    int f0;                      // first fine id of the range (list positions count from it)
    int iters;
    // first centroids: cluster j < old_end starts from its stored key centroid, any other from point
    // (seed_x0 < 0 ? the block's first : seed_x0) + seeds[u][j]
    int old_end;
    const int32_t* seeds;        // [U, seed_stride]
    long long seed_stride;
    int seed_x0;
    // results: plist[u][position] = old fine id, newid[u][old fine id], cof[u][new fine id] (all of list_stride), and
    // in Kc the working centroids: fine rows in the new order, coarse rows from row fcap
    int32_t* plist;
    int32_t* newid;
    int32_t* cof;
    long long list_stride;
    uint16_t* Kc;                // bf16 [U, tab_rows, 128]
    long long tab_rows;
    int fcap;
    int k_cap, n_cap;            // (set by the launch)
};
hipError_t launch_coarse_level(CoarseLevel p, int nb, int U, int max_pts, int max_k, hipStream_t s);
// Member lists of all blocks in one launch (stable counting sort by cluster id):
// start[u][id] = first list position of cluster id, counted from point p_first; the entry after the
// last block's last cluster receives the end position; list[u][position] = point index.
hipError_t launch_block_lists(const int32_t* ids, long long ids_stride, const int32_t* blocks_dev, int nb,
                              int max_k_per_block, int p_first, int U, int32_t* start, long long start_stride,
                              int32_t* list, long long list_stride, hipStream_t s);
// The rows t0 and up of a gather's sources once more, in sequence order (arrays of unit_rows rows a unit; null: not wanted).
struct SequenceCopy {
    void *K, *V;
    long long unit_rows;
    int t0;
};

// The stored rows of a range in cluster order, dst row dst_row0 + p = source row list[p] for p < n, and the tables of its fine
// clusters [f0, f1), members list[start[f] .. start[f + 1]) ascending: means as launch_cluster_means gives them, counts, sums.
struct StoredRows {
    const void *K, *V;             // 256-byte rows
    long long src_unit_rows;
    const int32_t* list;
    long long list_stride;
    const int32_t* start;
    long long start_stride;
    int f0, f1, n;
    void *dstK, *dstV;
    long long dst_unit_rows;
    int dst_row0;
    SequenceCopy seq;
    uint16_t *value_means, *key_means;   // [U, tab_rows, 128]; key means optional (the means of K's rows)
    bool key_keeps;                // an empty cluster's key mean stays as it is (else zeros)
    int32_t* counts;               // [U, tab_rows]
    long long tab_rows;
    double *value_sums, *key_sums; // [U, sum_unit_rows, 128], optional
    long long sum_unit_rows;
    bool all_by_place;             // set by the launch: a cluster's wave stores no rows,
    int long_cluster;              // or not those of clusters of more members
};
hipError_t launch_stored_rows(StoredRows p, int U, hipStream_t s);
// Rows in cluster order into 8-bit storage: dstK / dstV receive 128 e4m3 codes per row, scales [U, dst_unit_rows, 2] the
// rows' fp32 scales {key, value} (scale = max|x| / 448, 1 for a zero row; code = round-to-nearest-even(x / scale)).
// For a value row x is the row; for a key row x = fp32(key) - fp32(Kc[ids[point]]), the residual from the key
// centroid of the point's fine cluster (ids [U, ids_stride] by local point, Kc [U, kc_unit_rows, 128] bf16).
hipError_t launch_gather_quantize_rows(const void* srcK, const void* srcV, long long src_unit_rows, const int32_t* list,
                                       long long list_stride, const int32_t* ids, long long ids_stride,
                                       const uint16_t* Kc, long long kc_unit_rows, int n, int U, void* dstK, void* dstV,
                                       float* scales, long long dst_unit_rows, int dst_row0, const SequenceCopy& seq,
                                       int32_t* unusual, hipStream_t s);
// mean_out row (out_row0 + id) = bf16(fp64 sum of the member rows in list order / count); sum_out (optional)
// receives the fp64 sums themselves, row = id; range_out (optional) [U, sum_unit_rows] the exponent fields of a cluster's
// largest magnitude (<< 16) and smallest nonzero one (subnormals count as 1; 255 where there is none); changed_out (optional,
// with range_out, mean_out holding the rows of before) [U, sum_unit_rows] whether the row is another one now.
hipError_t launch_cluster_means(const uint16_t* X, long long x_unit_rows, const int32_t* list, long long list_stride,
                                const int32_t* start, long long start_stride, int k0, int k, int U,
                                uint16_t* mean_out, long long out_unit_rows, int out_row0, const uint16_t* fallback,
                                long long fb_unit_rows, int32_t* count_out, long long count_stride, int count_off,
                                double* sum_out, long long sum_unit_rows, uint32_t* range_out, uint32_t* changed_out, hipStream_t s);
// Later Lloyd iterations: sums, counts and centroids of the clusters whose members differ between old_ids and new_ids.
// `range` is what launch_cluster_means left for the same points.
struct MoveMeans {
    const uint16_t* X;             // points
    long long x_unit_rows;
    const int32_t* blocks;         // [nb][4]: x0, x1, k0, k1
    const int32_t* old_ids;        // [U, ids_stride] cluster of each point behind sum, count and C
    const int32_t* new_ids;
    long long ids_stride;
    const unsigned long long* marks;   // [U, marks_stride] of the points whose two ids may differ
    long long marks_stride;
    int32_t* moved;                // [U, moved_stride]: set for blocks of which a point moved, or may have
    int moved_stride;
    uint16_t* C;                   // [U, c_unit_rows, 128], row = cluster id
    long long c_unit_rows;
    int32_t* count;                // [U, count_stride]
    long long count_stride;
    double* sum;                   // [U, sum_unit_rows, 128]
    long long sum_unit_rows;
    const uint32_t* range;         // [U, range_stride]
    long long range_stride;
    uint32_t* changed;             // [U, range_stride] by cluster, for blocks of which a point is marked: did its centroid change? (or null)
    int per;                       // clusters of a workgroup (set by the launch)
};
hipError_t launch_move_means(MoveMeans p, int nb, int max_k, int U, hipStream_t s);
// Coarse clusters [c0, c1) from their children: sumK, sumV [U, fcap, 128] fp64 member sums of the fine clusters (key sums at
// row key_map ? key_map[f - f0] : f), cstart = first child of each coarse cluster, counts [U, tab_rows] members of the fine
// clusters; writes rows fcap + c of Kc, Vc [U, tab_rows, 128] and of counts.
struct CoarseTables {
    const double *sumK, *sumV;
    const int32_t* key_map;        // [U, fcap]
    int f0;
    const int32_t* cstart;
    long long cstart_stride;
    int32_t* counts;
    int c0, c1;
    uint16_t *Kc, *Vc;
    const uint16_t* key_fallback;  // Kc, or null
    int fcap;
    long long tab_rows;
};
hipError_t launch_coarse_from_children(const CoarseTables& p, int U, hipStream_t s);
struct StoredOrder {
    const int32_t* start;          // [U, start_stride] first list position of a cluster
    long long start_stride;
    const int32_t* list;           // [U, ncap]
    const int32_t* ids;            // [U, ids_stride], or null: fot is in place already
    long long ids_stride;
    const int32_t* cof;            // [U, fcap], or null: one level
    int f0, f1, c0, c1, n_pts, pt0, fcap, ccap;
    long long ncap;
    int32_t *fstart, *perm, *fot, *cstart;
};
hipError_t launch_stored_order(const StoredOrder& p, int U, hipStream_t s);
// Device-to-device copies of `rows` rows each, several in one launch (a copy of its own is 5 us whatever its size).
struct CopyBatch {
    struct Part {
        const void* src;
        void* dst;
        long long spitch, dpitch;
        unsigned long long width;
        unsigned unit;             // bytes moved at a time: what pointers, pitches and width are multiples of
    };
    static constexpr int kParts = 8;
    Part part[kParts];
    int n = 0;
    void add(void* dst, size_t dpitch, const void* src, size_t spitch, size_t width);
    hipError_t launch(int rows, hipStream_t s);
};
hipError_t launch_fill(int32_t* dst, int n, int32_t value, hipStream_t s);
// Views of the last scoring launch, by cluster id.  keys [U, pos_stride] by position; key_mode[2*u + level]
// says what they are: 0 = order-preserving image of the rank key r = log mean_h e^{l - LSE_h}; 1 = complement
// of the bit pattern of sum_h e^{l - LSE_h} (then r = log(sum) - log G).  r_out receives r (NaN: took no part).
hipError_t launch_scatter_selection(const int32_t* cand, long long cand_stride, const int32_t* n_cand_dev,
                                    int n_cand_fixed, const uint8_t* flag, const unsigned long long* keys,
                                    const int32_t* key_mode, int level, int G, long long pos_stride, int n_ids, int U,
                                    uint8_t* sel_out, double* r_out, hipStream_t s);

}  // namespace mp
