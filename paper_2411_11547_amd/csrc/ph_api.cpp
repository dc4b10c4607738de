// Host runtime and C ABI of libpairhmm (include/ph.h).
//
// A plan is built once per problem shape: it validates the batch structure
// and lengths, assigns every read length to a kernel configuration (lanes P
// per pair, rows K per lane; the paper's (p, k) template grid, Section
// III-B/III-C), counts the pairs of every length bin, and allocates the
// device scratch.  A forward call then enqueues, on the caller's stream:
//   1. (explicit-parameter mode) exponentiation of the log10 parameters;
//   2. the call's preparation: the book of the work lists, which were built by
//      (length bin, haplotype length) at plan creation (Section III-A stage 3 /
//      Section III-C), and the chain code stream;
//   3. one persistent FP32 sweep per non-empty bin, longest bin first, as
//      parallel branches (Section III-C runs one kernel per index list on its
//      own stream);
//   4. the FP64 sweep over the pairs whose FP32 sum fell below the rescue
//      threshold, one persistent launch for reads of up to 255 bases, one for
//      those of up to 511 and two for longer ones.
// The FP32 launches are captured into a HIP graph by the first call and when other
// problem and output pointers come again, and replayed while these stay.  Small calls
// are one launch (k_one).
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <cmath>
#include <fstream>
#include <memory>
#include <mutex>
#include <sstream>
#include <string>
#include <vector>

#include "../../include/ph.h"
#include "ph_internal.h"
#include "ph_rules.h"

using namespace ph;

namespace {

thread_local std::string g_err;

ph_status fail(ph_status st, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    g_err = buf;
    return st;
}

}  // namespace

namespace ph {
// ph_plan_create with the longest chain given (0: chosen, and returned), along
// whose columns the FP32 row sums are grouped; out NULL: the choice alone,
// without a GPU call
ph_status plan_create(const ph_shape *shape, const ph_plan_opts *opts, int &chain_cols, ph_plan **out);

// the calling thread's message for ph_last_error(), set by other host sources
void set_last_error(const char *msg) { g_err = msg ? msg : ""; }
}  // namespace ph

namespace {

#define HIPCHK(x)                                                                           \
    do {                                                                                    \
        hipError_t e_ = (x);                                                                \
        if (e_ != hipSuccess) return fail(PH_ERR_HIP, "%s: %s", #x, hipGetErrorString(e_)); \
    } while (0)

// haplotype-length bucket of the binning key (16-column buckets below 1024,
// 128-column buckets above; the kernels' pair_key uses the same)
int hap_bucket(int64_t n) { return n < 1024 ? (int)(n >> 4) : 64 + (int)std::min<int64_t>((n - 1024) >> 7, 63); }

constexpr int kSideStreams = 4;
constexpr int kStageEvents = 5;

std::once_flag g_lut_once;
hipError_t g_lut_status = hipSuccess;
std::once_flag g_lut_adj_once;
hipError_t g_lut_adj_status = hipSuccess;

// adjoint checkpoint workspaces: the grid of a launch shrinks to fit
constexpr int64_t kAdjWsFloats = (int64_t)1 << 30;    // 4 GiB, FP32 pass
constexpr int64_t kAdjWs64Doubles = (int64_t)1 << 28;  // 2 GiB, FP64 pass


int rescue_class_of(int m) { return m < 128 ? 0 : m < 256 ? 1 : m < 512 ? 2 : 3; }
// pairs of the classes that a rescue launch sweeps
int64_t rescue_pairs(const int64_t *class_pairs, int group)
{
    return group == 0 ? class_pairs[0] + class_pairs[1] : class_pairs[std::min(group + 1, 3)];
}

std::vector<TuneEntry> default_table(int force_p)
{
    std::vector<TuneEntry> t;
    if (force_p) {
        for (int K = 1; K <= 16; ++K)
            if (fwd32_supported(force_p, K) && force_p * K - 1 <= kMaxReadLen)
                t.push_back({force_p * K - 1, force_p, K});
        return t;
    }
    TuneEntry b[kMaxBins];
    const int nb = builtin_table(b);
    t.assign(b, b + nb);
    return t;
}

// Table for the single-launch sweep: reads shorter than 48 share the K = 3 bin.
std::vector<TuneEntry> single_table()
{
    std::vector<TuneEntry> t;
    for (int K = 3; K <= 16; ++K) t.push_back({16 * K - 1, 16, K});
    for (int K = 5; K <= 16; ++K) t.push_back({64 * K - 1, 64, K});
    return t;
}

ph_status read_table(const char *path, std::vector<TuneEntry> &t)
{
    std::ifstream f(path);
    if (!f) return fail(PH_ERR_INVALID, "cannot open tune table %s", path);
    std::string line;
    t.clear();
    while (std::getline(f, line)) {
        if (line.empty() || line[0] == '#') continue;
        const std::string body = line.substr(0, line.find('#'));
        std::istringstream ss(body);
        TuneEntry e;
        if (!(ss >> e.max_m >> e.P >> e.K)) return fail(PH_ERR_INVALID, "bad tune line: %s", line.c_str());
        if (!fwd32_supported(e.P, e.K)) return fail(PH_ERR_UNSUPPORTED, "tune entry P=%d K=%d not compiled", e.P, e.K);
        if (e.max_m > e.P * e.K - 1 || e.max_m < 1)
            return fail(PH_ERR_INVALID, "tune entry max_m=%d exceeds P*K-1 for P=%d K=%d", e.max_m, e.P, e.K);
        if (ss >> e.n_split) {
            if (!(ss >> e.P2 >> e.K2) || e.n_split < 1)
                return fail(PH_ERR_INVALID, "bad haplotype-length split in tune line: %s", line.c_str());
            if (!fwd32_supported(e.P2, e.K2))
                return fail(PH_ERR_UNSUPPORTED, "tune entry P=%d K=%d not compiled", e.P2, e.K2);
            if (e.max_m > e.P2 * e.K2 - 1)
                return fail(PH_ERR_INVALID, "tune entry max_m=%d exceeds P*K-1 for P=%d K=%d", e.max_m, e.P2, e.K2);
            const bool edge = e.n_split < 1024 ? e.n_split % 16 == 0
                                               : (e.n_split - 1024) % 128 == 0 && e.n_split <= 1024 + 63 * 128;
            if (!edge)
                return fail(PH_ERR_INVALID, "haplotype-length split %d is not a bucket edge (a multiple of 16 "
                            "below 1024, 1024 + a multiple of 128 up to 9088)", e.n_split);
        }
        t.push_back(e);
    }
    std::sort(t.begin(), t.end(), [](const TuneEntry &a, const TuneEntry &b) { return a.max_m < b.max_m; });
    if (t.empty()) return fail(PH_ERR_INVALID, "empty tune table %s", path);
    // neighbouring ranges with the same configuration form one bin
    std::vector<TuneEntry> merged;
    for (const TuneEntry &e : t) {
        const TuneEntry *b = merged.empty() ? nullptr : &merged.back();
        if (b && b->P == e.P && b->K == e.K && b->n_split == e.n_split && b->P2 == e.P2 && b->K2 == e.K2)
            merged.back().max_m = e.max_m;
        else
            merged.push_back(e);
    }
    // each split adds its second bin right after its parent
    t.clear();
    for (const TuneEntry &e : merged) {
        t.push_back(e);
        if (e.n_split) {
            TuneEntry a;
            a.max_m = e.max_m;
            a.P = e.P2;
            a.K = e.K2;
            t.push_back(a);
        }
    }
    if ((int)t.size() > kMaxBins - 1)
        return fail(PH_ERR_INVALID, "tune table has more than %d distinct bins", kMaxBins - 1);
    return PH_OK;
}

}  // namespace

struct ph_plan {
    int device = 0;
    int cus = 0;
    ph_plan_opts opts{};
    double threshold = 1e-28;
    int32_t nb = 0, nr = 0, nh = 0;
    int64_t P = 0, cells = 0, nread_bases = 0, nhap_bases = 0;
    int32_t max_m = 0, max_n = 0;

    std::vector<TuneEntry> table;      // bin b = table[table.size()-1-b] (longest first)
    std::vector<int> bin_grid;         // persistent grid per bin (0 = empty)
    int64_t class_pairs[kRescueClasses] = {0, 0, 0, 0};
    int rescue_grid[kRescueGroups] = {};
    int plain_K = 0, plain_grid = 0;
    // reads longer than kMaxReadLen: one extra bin swept in windows
    int long_bin = -1, windows = 0, windows64 = 0, long_grid = 0, long64_grid = 0;
    bool long_few = false;
    int64_t long_pairs = 0, bnd_stride = 0;
    float *d_bnd32 = nullptr;
    double *d_bnd64 = nullptr;
    int32_t *d_long_rescue = nullptr;
    int32_t *d_progress = nullptr;  // columns done of every window: FP32, FP64 rescaled, FP64 plain
    int split_at = -1;     // offset of the haplotype-length split table in d_m2bin (-1: none)
    std::vector<std::pair<int, int>> launch_order;  // FP32 stage: (bin, side stream) in launch order
    bool single = false;   // one persistent FP32 launch over all bins
    int single_grid = 0;
    // binned mode: work lists built from the shape at plan creation, with
    // chain tiles; the call copies the book image and writes the chain codes
    std::vector<int64_t> bin_tiles;    // tiles per bin
    std::vector<int64_t> bin_cols;     // columns of each bin's longest tile
    double binned_ns = 0;              // time that all tiles take a full GPU
    int32_t chain_rec_base = 0;        // records of the lists; FP64 records of chain pairs follow
    bool chain_tiles = false;
    Book *d_book_img = nullptr;
    uint8_t *d_chain_codes = nullptr;
    // small plans: one launch, one pair per wave (k_one)
    bool one = false;
    bool one_reads[2] = {};            // some read of up to 255 bases, some longer one
    int one_max_m = 0;
    OneRec *d_one = nullptr;
    uint8_t *d_one_rescued = nullptr;  // per output of the last call: 1 if the pair went to FP64

    int64_t *d_out_offset = nullptr;
    int16_t *d_m2bin = nullptr;
    int32_t *d_bin_G = nullptr;
    int32_t *d_hist = nullptr;
    PairRec *d_recs = nullptr;
    Book *d_book = nullptr;
    int32_t *d_bad = nullptr;          // ph_validate: count of base codes above 4
    int32_t *d_rescue = nullptr;
    double *d_lin = nullptr;
    int64_t lin_cap = 0;

    hipStream_t cap = nullptr;
    hipStream_t side[kSideStreams] = {};
    hipEvent_t fork = nullptr, join[kSideStreams] = {};
    hipEvent_t ev[kStageEvents] = {};
    bool stages_recorded = false;

    // Captured launches: they hold for the pointers that they were captured with.
    struct Captured {
        hipGraph_t graph = nullptr;
        hipGraphExec_t exec = nullptr;
        std::vector<const void *> key, last;  // pointers of the graph, of the last call
        hipEvent_t ran = nullptr;             // after the graph's last launch, once marked
        bool marked = false;
    };
    Captured fwd[2];  // the FP32 stage of the forward ([0]) and of the Viterbi score ([1])
    bool events_captured = false;  // a caller's capture took the events of a call

    hipStream_t last_stream = nullptr;
    bool forward_done = false;

    // host copy of the shape (adjoint tables are built from it on demand)
    std::vector<int32_t> h_rb, h_hb;
    std::vector<int64_t> h_ro, h_ho, h_out_off;

    // adjoint: records grouped by (P, K) configuration, tiled G = 64/P at a
    // time; persistent launches over the tiles of all configurations or of one,
    // each workgroup with its own checkpoint slice
    struct AdjLaunch {
        std::vector<AdjRun> runs;
        int64_t tile_begin = 0;
        int32_t ntiles = 0, lds = 0, grid = 0;
        int64_t ws_stride = 0;  // floats per workgroup
        double time = 0;        // as adj_launch_time
    };
    bool adj_built = false;
    ph_status adj_status = PH_OK;
    std::string adj_error;
    std::vector<AdjLaunch> adj_launches;
    AdjRec *d_adj_recs = nullptr;
    AdjTile *d_adj_tiles = nullptr;
    float *d_ws = nullptr;
    // gradients of reads with several pairs: per-pair rows, then a
    // fixed-order sum per read (no float atomics)
    float *d_grad_pair = nullptr;
    AdjRedRead *d_red = nullptr;
    int32_t n_red = 0;
    bool adj_zero = false;  // some read has no pair: its rows are zeroed
    int32_t *d_adj_ctr = nullptr;  // [2][kAdj64Classes] FP64 queue lengths, cursors; then the tile cursors
    // FP64 pass over the pairs the FP32 pass leaves out: queues per class,
    // [2][kAdj64Classes] counters (lengths, cursors), per-workgroup checkpoints
    int32_t *d_q64 = nullptr;
    double *d_ws64 = nullptr;
    int64_t q64_stride = 0, ws64_stride = 0;
    int32_t grid64 = 0, hs_bytes64 = 0;
    int k64_max = 1, k64_only = 0;  // the FP64 pass's largest class, and the only one (0: several)
    hipEvent_t ev_adj[2] = {};
    bool adj_recorded = false;
    Captured adj;
};

namespace {

void drop_captured(ph_plan::Captured &c)
{
    if (c.exec) (void)hipGraphExecDestroy(c.exec);
    if (c.graph) (void)hipGraphDestroy(c.graph);
    c.exec = nullptr;
    c.graph = nullptr;
    c.key.clear();
    c.marked = false;
}

// (a graph that may still run is waited for before it goes; events that were last
// recorded into a caller's capture say nothing about it)
void drop_graphs(ph_plan *p)
{
    const bool fwd = p->fwd[0].exec || p->fwd[1].exec;
    if (p->events_captured && (fwd || p->adj.exec)) {
        int dev = p->device;
        (void)hipGetDevice(&dev);
        (void)hipSetDevice(p->device);
        (void)hipDeviceSynchronize();
        (void)hipSetDevice(dev);
    } else {
        if (p->stages_recorded && fwd) (void)hipEventSynchronize(p->ev[3]);
        if (p->adj_recorded && p->adj.exec) (void)hipEventSynchronize(p->ev_adj[1]);
    }
    for (auto *c : {&p->fwd[0], &p->fwd[1], &p->adj}) drop_captured(*c);
}

void free_plan(ph_plan *p)
{
    if (!p) return;
    drop_graphs(p);
    void *bufs[] = {p->d_out_offset, p->d_m2bin, p->d_bin_G, p->d_hist, p->d_recs, p->d_book, p->d_bad, p->d_rescue, p->d_lin,
                    p->d_book_img, p->d_chain_codes, p->d_one, p->d_one_rescued,
                    p->d_bnd32, p->d_bnd64, p->d_long_rescue, p->d_progress,
                    p->d_adj_recs, p->d_adj_tiles, p->d_ws, p->d_adj_ctr, p->d_q64, p->d_ws64, p->d_grad_pair, p->d_red};
    for (auto &e : p->ev_adj)
        if (e) (void)hipEventDestroy(e);
    for (auto *c : {&p->fwd[0], &p->fwd[1], &p->adj})
        if (c->ran) (void)hipEventDestroy(c->ran);
    for (void *b : bufs)
        if (b) (void)hipFree(b);
    for (auto &e : p->ev)
        if (e) (void)hipEventDestroy(e);
    for (auto &e : p->join)
        if (e) (void)hipEventDestroy(e);
    if (p->fork) (void)hipEventDestroy(p->fork);
    for (auto &s : p->side)
        if (s) (void)hipStreamDestroy(s);
    if (p->cap) (void)hipStreamDestroy(p->cap);
    delete p;
}

template <typename T>
ph_status dalloc(T **ptr, size_t count)
{
    size_t bytes = std::max<size_t>(count, 1) * sizeof(T);
    hipError_t e = hipMalloc((void **)ptr, bytes);
    if (e != hipSuccess) return fail(PH_ERR_NOMEM, "hipMalloc(%zu): %s", bytes, hipGetErrorString(e));
    return PH_OK;
}

ph_status check_problem(const ph_plan *p, const ph_problem *pb)
{
    if (!pb) return fail(PH_ERR_INVALID, "problem is NULL");
    if (pb->num_batches != p->nb || pb->num_reads != p->nr || pb->num_haps != p->nh)
        return fail(PH_ERR_PLAN_MISMATCH, "problem has %d batches, %d reads, %d haplotypes; plan has %d, %d, %d",
                    pb->num_batches, pb->num_reads, pb->num_haps, p->nb, p->nr, p->nh);
    if (p->P == 0) return PH_OK;
    if (!pb->batch_read_begin || !pb->batch_hap_begin || !pb->read_offset || !pb->hap_offset ||
        !pb->read_bases || !pb->hap_bases)
        return fail(PH_ERR_INVALID, "problem has a NULL array");
    return PH_OK;
}

// Whether the plan's adjoint takes 64 lanes for every pair (adj_wide).
bool adjoint_wide(const ph_plan *p)
{
    if (p->P > kAdjWidePairs) return false;
    int only = -1;
    std::vector<int64_t> n;  // haplotypes of all pairs
    for (int32_t q = 0; q < p->nb; ++q)
        for (int32_t r = p->h_rb[q]; r < p->h_rb[q + 1] && p->h_hb[q] < p->h_hb[q + 1]; ++r) {
            int P = 0, K = 0;
            if (!adj_config((int)(p->h_ro[r + 1] - p->h_ro[r]), false, P, K)) return false;
            if (P == 64 || (only >= 0 && only != K)) return true;
            only = K;
            for (int32_t h = p->h_hb[q]; h < p->h_hb[q + 1]; ++h) n.push_back(p->h_ho[h + 1] - p->h_ho[h]);
        }
    if (n.empty()) return false;
    std::sort(n.begin(), n.end(), [](int64_t a, int64_t b) { return a > b; });
    return adj_wide(p->P, only, n[0], (int64_t)n.size() > kAdjAlone ? n[kAdjAlone] : 0);
}

// Steps of a tile of P lanes per pair: every lane reaches column n + 2 (the absorbing
// row of the rescaled states sums column n into column n + 2), rounded up to whole
// checkpoint intervals.
int adj_steps(int n, int P)
{
    constexpr int CK = kAdjC * kAdjR;  // steps per checkpoint
    return (n + P + 1 + CK - 1) / CK * CK;
}
// LDS bytes of a lane group's haplotype codes, one byte per column, and of a workgroup
int adj_hs_bytes(int S, int P) { return (S + P + 2 + 15) / 16 * 16; }
int64_t adj32_lds_bytes(int P, int K, int S)
{
    return (int64_t)adj_e_bytes(P, K) + 64 / P * (int64_t)adj_hs_bytes(S, P) + adj_ck_lds_bytes(K);
}

// From this many tiles on the ends of the launches count less than what a
// kernel for every configuration gains.
constexpr int64_t kAdjApartTiles = 32768;

ph_status build_adjoint(ph_plan *p)
{
    if (p->adj_built) return p->adj_status;
    p->adj_built = true;
    struct Item {
        AdjRec r;
        int P, K;
    };
    std::vector<Item> items;
    items.reserve((size_t)p->P);
    const bool wide = adjoint_wide(p);
    std::vector<AdjRedRead> red;
    int64_t grow = 0;  // per-pair gradient rows handed out so far
    std::vector<char> has_pair(p->nr, 0);
    for (int32_t q = 0; q < p->nb; ++q) {
        const int32_t H = p->h_hb[q + 1] - p->h_hb[q];
        int n_longest = 0;
        for (int32_t h = p->h_hb[q]; h < p->h_hb[q + 1]; ++h)
            n_longest = std::max(n_longest, (int)(p->h_ho[h + 1] - p->h_ho[h]));
        for (int32_t r = p->h_rb[q]; r < p->h_rb[q + 1]; ++r) {
            const int m = (int)(p->h_ro[r + 1] - p->h_ro[r]);
            int P = 0, K = 0;
            if (!adj_config(m, wide, P, K) || !adj_supported(P, K)) {
                p->adj_status = PH_ERR_UNSUPPORTED;
                p->adj_error = "adjoint supports reads up to 319 bases";
                return p->adj_status;
            }
            if (H > 0) has_pair[r] = 1;
            // the longest haplotype that is accepted does not depend on the plan's
            // other pairs: what the LDS holds with the lanes of a large plan
            int Pn = 0, Kn = 0;
            adj_config(m, false, Pn, Kn);
            if (H > 0 && adj32_lds_bytes(Pn, Kn, adj_steps(n_longest, Pn)) > 64 * 1024) {
                p->adj_status = PH_ERR_UNSUPPORTED;
                p->adj_error = "haplotype too long for the adjoint sweep";
                return p->adj_status;
            }
            // a read with several pairs: pair h's rows at grow + h m
            if (H > 1) red.push_back(AdjRedRead{grow, p->h_ro[r], m, H});
            for (int32_t h = p->h_hb[q]; h < p->h_hb[q + 1]; ++h) {
                Item it{};
                it.r.read = r;
                it.r.hap = h;
                it.r.out = (int32_t)(p->h_out_off[q] + (int64_t)(r - p->h_rb[q]) * H + (h - p->h_hb[q]));
                it.r.n = (int32_t)(p->h_ho[h + 1] - p->h_ho[h]);
                it.r.direct = H == 1 ? 1 : 0;
                it.r.grow = H == 1 ? 0 : grow + (int64_t)(h - p->h_hb[q]) * m;
                it.P = P;
                it.K = K;
                items.push_back(it);
            }
            if (H > 1) grow += (int64_t)H * m;
        }
    }
    for (int32_t r = 0; r < p->nr; ++r) p->adj_zero = p->adj_zero || !has_pair[r];
    if (red.size() >= ((size_t)1 << 31)) {
        p->adj_status = PH_ERR_UNSUPPORTED;
        p->adj_error = "too many reads with several pairs";
        return p->adj_status;
    }
    // configuration, then longest haplotype first
    std::sort(items.begin(), items.end(), [](const Item &a, const Item &b) {
        if (a.P != b.P) return a.P > b.P;
        if (a.K != b.K) return a.K > b.K;
        if (a.r.n != b.r.n) return a.r.n > b.r.n;
        return a.r.out < b.r.out;
    });
    // the tiles of every configuration, G records each, longest first
    struct Config {
        int P, K;
        size_t begin, end;             // items
        std::vector<int> S;            // steps of each tile
        size_t group[kAdjGroups + 1];  // first tile of each group (adj_group), the longest tiles' group first
    };
    std::vector<AdjRec> recs(items.size());
    std::vector<Config> configs;
    for (size_t i = 0; i < items.size();) {
        Config c{items[i].P, items[i].K, i, i, {}, {}};
        while (c.end < items.size() && items[c.end].P == c.P && items[c.end].K == c.K) ++c.end;
        const size_t G = 64 / c.P;
        for (size_t a = i; a < c.end; a += G) {
            // (the tile's first record has its longest haplotype)
            c.S.push_back(adj_steps(items[a].r.n, c.P));
            for (size_t b = a; b < std::min(a + G, c.end); ++b) {
                recs[b] = items[b].r;
                recs[b].S = c.S.back();
            }
        }
        for (int g = 0, t = 0; g <= kAdjGroups; ++g) {
            while (t < (int)c.S.size() && (g == kAdjGroups || adj_group(c.S[t]) > kAdjGroups - 1 - g)) ++t;
            c.group[g] = t;
        }
        i = c.end;
        configs.push_back(std::move(c));
    }
    // a launch over the tiles of the groups g0 .. g1 - 1 (as in Config::group) of
    // configuration only, or (-1) of all
    auto launch_of = [&](int g0, int g1, int only) {
        ph_plan::AdjLaunch L;
        double longest = 0, total = 0;
        for (size_t k = 0; k < configs.size(); ++k) {
            const Config &c = configs[k];
            const size_t t0 = c.group[g0], t1 = c.group[g1], G = 64 / c.P;
            if (t0 == t1 || (only >= 0 && (int)k != only)) continue;
            const size_t first = c.begin + t0 * G;
            const AdjRun r{c.P, c.K, (int32_t)(std::min(c.begin + t1 * G, c.end) - first), adj_hs_bytes(c.S[t0], c.P),
                           (int64_t)first};
            L.runs.push_back(r);
            L.lds = std::max(L.lds, (int)adj32_lds_bytes(c.P, c.K, c.S[t0]));
            L.ws_stride = std::max<int64_t>(
                L.ws_stride, ((int64_t)(c.S[t0] / (kAdjC * kAdjR)) * (3 * r.K + 3) * 64 + 63) / 64 * 64);
            L.ntiles += (int32_t)(t1 - t0);
            longest = std::max(longest, (double)c.S[t0] * adj_step(c.K));
            for (size_t t = t0; t < t1; ++t) total += (double)c.S[t] * adj_step(c.K);
        }
        if (L.runs.empty()) return L;
        const bool one = L.runs.size() == 1;
        L.grid = (int32_t)std::max<int64_t>(
            1, std::min<int64_t>({L.ntiles, (int64_t)p->cus * adj32_blocks_per_cu(one ? L.runs[0].P : 0, L.runs[0].K, L.lds),
                                  kAdjWsFloats / L.ws_stride}));
        L.time = adj_launch_time(longest, total, L.grid);
        return L;
    };
    // the launches over the groups g0 .. g1 - 1, and which launches the groups make:
    // the cut with the least time
    auto launches_of = [&](int g0, int g1) {
        std::vector<ph_plan::AdjLaunch> l = {launch_of(g0, g1, -1)};
        if (l[0].ntiles >= kAdjApartTiles && l[0].runs.size() > 1) {
            l.clear();
            for (size_t k = 0; k < configs.size(); ++k) {
                l.push_back(launch_of(g0, g1, (int)k));
                if (l.back().runs.empty()) l.pop_back();
            }
        }
        if (l[0].runs.empty()) l.clear();
        return l;
    };
    std::vector<ph_plan::AdjLaunch> best[kAdjGroups + 1];  // of the groups before g
    std::vector<int> begin[kAdjGroups + 1], end[kAdjGroups + 1];  // their groups
    double best_time[kAdjGroups + 1] = {};
    for (int g1 = 1; g1 <= kAdjGroups; ++g1) {
        best_time[g1] = INFINITY;
        for (int g0 = 0; g0 < g1; ++g0) {
            const auto l = launches_of(g0, g1);
            double time = best_time[g0];
            for (const auto &x : l) time += x.time;
            if (time >= best_time[g1]) continue;
            best_time[g1] = time;
            best[g1] = best[g0];
            begin[g1] = begin[g0];
            end[g1] = end[g0];
            for (const auto &x : l) {
                best[g1].push_back(x);
                begin[g1].push_back(g0);
                end[g1].push_back(g1);
            }
        }
    }
    p->adj_launches = best[kAdjGroups];
    // the order of the tiles of launches over several configurations: longest first
    std::vector<AdjTile> order;
    int64_t ws_total = 0;
    for (size_t l = 0; l < p->adj_launches.size(); ++l) {
        ph_plan::AdjLaunch &L = p->adj_launches[l];
        L.tile_begin = (int64_t)order.size();
        ws_total = std::max(ws_total, (int64_t)L.grid * L.ws_stride);
        if (L.runs.size() == 1) continue;
        struct Timed {
            int64_t time;
            AdjTile tile;
        };
        std::vector<Timed> tiles;
        int32_t run = 0;
        for (const Config &c : configs) {
            const size_t t0 = c.group[begin[kAdjGroups][l]], t1 = c.group[end[kAdjGroups][l]], before = tiles.size();
            if (t0 == t1) continue;
            for (size_t t = t0; t < t1; ++t)
                tiles.push_back(Timed{(int64_t)c.S[t] * adj_step(c.K), {run, (int32_t)(t - t0)}});
            std::inplace_merge(tiles.begin(), tiles.begin() + before, tiles.end(),
                               [](const Timed &x, const Timed &y) { return x.time > y.time; });
            ++run;
        }
        for (const Timed &x : tiles) order.push_back(x.tile);
    }
    // FP64 pass: sized for the longest haplotype and the largest class of
    // the plan; the grid is bounded by the workspace budget
    int n_max = 1, k64_max = 1, k64_min = kAdj64Classes;
    for (const auto &it : items) n_max = std::max(n_max, it.r.n);
    for (int32_t r = 0; r < p->nr; ++r) {
        const int m = (int)(p->h_ro[r + 1] - p->h_ro[r]);
        const int k = (m + 64) / 64;
        if (k >= 1 && k <= kAdj64Classes) {
            k64_max = std::max(k64_max, k);
            k64_min = std::min(k64_min, k);
        }
    }
    const int S64 = ((n_max + 63 + kAdjC64 - 1) / kAdjC64) * kAdjC64;
    p->hs_bytes64 = ((S64 + 64 + 2 + 15) / 16) * 16;  // one code byte per column
    if ((int64_t)adj64_e_bytes(k64_max) + p->hs_bytes64 > 64 * 1024) {
        p->adj_status = PH_ERR_UNSUPPORTED;
        p->adj_error = "haplotype too long for the FP64 adjoint sweep";
        return p->adj_status;
    }
    p->k64_max = k64_max;
    p->k64_only = k64_min == k64_max ? k64_max : 0;
    p->ws64_stride = ((int64_t)(S64 / kAdjC64) * (3 * k64_max + 3) * 64 + 31) / 32 * 32;
    p->grid64 = (int32_t)std::max<int64_t>(
        1, std::min<int64_t>({(int64_t)p->cus * adj64_blocks_per_cu(p->k64_only), kAdjWs64Doubles / p->ws64_stride,
                              (int64_t)items.size()}));
    p->q64_stride = (int64_t)items.size();
    ph_status st;
    if ((st = dalloc(&p->d_adj_recs, recs.size()))) return p->adj_status = st;
    if ((st = dalloc(&p->d_ws, (size_t)std::max<int64_t>(ws_total, 1)))) return p->adj_status = st;
    if ((st = dalloc(&p->d_adj_tiles, order.size()))) return p->adj_status = st;
    if ((st = dalloc(&p->d_adj_ctr, (size_t)2 * kAdj64Classes + p->adj_launches.size()))) return p->adj_status = st;
    if ((st = dalloc(&p->d_q64, (size_t)kAdj64Classes * p->q64_stride))) return p->adj_status = st;
    if ((st = dalloc(&p->d_ws64, (size_t)p->grid64 * p->ws64_stride))) return p->adj_status = st;
    if ((st = dalloc(&p->d_grad_pair, (size_t)std::max<int64_t>(grow, 1) * 7))) return p->adj_status = st;
    if ((st = dalloc(&p->d_red, std::max<size_t>(red.size(), 1)))) return p->adj_status = st;
    p->n_red = (int32_t)red.size();
    hipError_t e = hipMemcpy(p->d_adj_recs, recs.data(), recs.size() * sizeof(AdjRec), hipMemcpyHostToDevice);
    if (e == hipSuccess && !order.empty())
        e = hipMemcpy(p->d_adj_tiles, order.data(), order.size() * sizeof(AdjTile), hipMemcpyHostToDevice);
    if (e != hipSuccess) return p->adj_status = fail(PH_ERR_HIP, "hipMemcpy: %s", hipGetErrorString(e));
    if (!red.empty()) {
        e = hipMemcpy(p->d_red, red.data(), red.size() * sizeof(AdjRedRead), hipMemcpyHostToDevice);
        if (e != hipSuccess) return p->adj_status = fail(PH_ERR_HIP, "hipMemcpy: %s", hipGetErrorString(e));
    }
    return PH_OK;
}

// Longer chains make fewer, longer tiles, whose last round runs on part of
// the GPU: a plan halves the chain length (down to 1,024 columns) until it
// has this many chain tiles, 8 per wave of a launch of 3 waves per SIMD on
// 256 CUs.  (The mixed batch keeps 4,096 columns; the uniform batch, one bin
// of 64,000 reads against 8 haplotypes, gets 2,048.)
constexpr int64_t kChainMinTiles = 24576;

// Haplotypes hb0 .. hb1 - 1 cut into runs for chains of at most max_cols
// stream columns: f(first haplotype, haplotypes, columns) for each.
template <typename F>
void chain_segments(int32_t hb0, int32_t hb1, const int64_t *ho, int max_cols, F f)
{
    int32_t h0 = hb0, H = 0;
    int64_t len = 0;
    for (int32_t h = hb0; h < hb1; ++h) {
        const int64_t n = ho[h + 1] - ho[h];
        if (H && n >= kChainMinHap && H < kChainMaxHaps && len + kChainSep + n <= max_cols) {
            H += 1;
            len += kChainSep + n;
        } else {
            if (H) f(h0, H, len);
            h0 = h;
            H = 1;
            len = n;
        }
    }
    if (H) f(h0, H, len);
}

// Chain tiles of a plan with chains of at most max_cols columns.
int64_t chain_tile_count(const ph_plan *p, int32_t nb, const int32_t *rb, const int32_t *hb, const int64_t *ro,
                         const int64_t *ho, const std::vector<int16_t> &m2bin, int max_cols)
{
    const int nbins = (int)p->table.size();
    int64_t tiles = 0;
    std::vector<int32_t> cnt(nbins, 0);
    for (int32_t q = 0; q < nb; ++q) {
        int64_t chains = 0;
        chain_segments(hb[q], hb[q + 1], ho, max_cols, [&](int32_t, int32_t H, int64_t) { chains += H >= 2; });
        if (!chains) continue;
        for (int32_t r = rb[q]; r < rb[q + 1]; ++r) cnt[m2bin[std::min<int64_t>(ro[r + 1] - ro[r], kMaxReadLen + 1)]] += 1;
        for (int b = 0; b < nbins; ++b) {
            const int P = p->table[nbins - 1 - b].P;
            if (b != p->long_bin && P >= 16) tiles += chains * (cnt[b] / (64 / P));
            cnt[b] = 0;
        }
    }
    return tiles;
}

// The longest chains that still leave kChainMinTiles chain tiles (or 1,024 columns).
int choose_chain_cols(const ph_plan *p, int32_t nb, const int32_t *rb, const int32_t *hb, const int64_t *ro,
                      const int64_t *ho, const std::vector<int16_t> &m2bin)
{
    const bool chains_ok = kChains && 2 * p->P < ((int64_t)1 << 31);
    int cols = kChainMaxCols;
    while (chains_ok && cols > 1024) {
        const int64_t n = chain_tile_count(p, nb, rb, hb, ro, ho, m2bin, cols);
        if (n == 0 || n >= kChainMinTiles) break;
        cols /= 2;
    }
    return cols;
}

// The FP32 work lists of a binned plan (Section III-C), built once from the
// shape: records of every bin, bin b's range and tiles in the book image.
// A bin's records are its chain tiles, longest chain first, then single
// pairs, longest haplotype first.  A chain tile holds G = 64/P reads of one
// batch and length bin, each against the same run of the batch's
// haplotypes (at most kChainMaxHaps haplotypes and max_cols stream
// columns, every haplotype after the first at least kChainMinHap long), in
// pieces of at most piece_cols columns, each with the lead that keeps the
// groups of the row sums where the whole chain has them;
// bins of fewer than 16 lanes and the reads of a batch's bin that do not
// fill a tile take single pairs.  A haplotype-length split applies to
// single pairs only (sending chains whose stream reaches the split length
// to the split's bin was slower on the mixed batch).
bool build_lists(ph_plan *p, const int32_t *rb, const int32_t *hb, const int64_t *ro, const int64_t *ho,
                 const std::vector<int64_t> &out_off, const std::vector<int16_t> &m2bin,
                 const std::vector<int16_t> &split, int max_cols, int piece_cols, std::vector<PairRec> &recs, Book &img)
{
    const int nbins = (int)p->table.size();
    auto binP = [&](int b) { return p->table[nbins - 1 - b].P; };
    auto split_bin = [&](int b, int64_t len) {
        return (split[b] < kBuckets && hap_bucket(len) >= split[b]) ? (int)split[kMaxBins + b] : b;
    };
    // chain tiles can place the FP64 record of a pair at chain_rec_base + out
    const bool chains_ok = kChains && 2 * p->P < ((int64_t)1 << 31);
    struct Tile {
        int64_t len;   // sort key: stream or haplotype length
        int64_t first; // into `pool`
        int32_t count;
    };
    std::vector<std::vector<Tile>> chain_tiles(nbins), singles(nbins);
    std::vector<PairRec> pool;
    pool.reserve((size_t)p->P);
    std::vector<std::pair<int, int32_t>> by_bin;
    struct Seg {
        int32_t h0, H;
        int64_t len;
    };
    std::vector<Seg> segs;
    for (int32_t q = 0; q < p->nb; ++q) {
        const int32_t H = hb[q + 1] - hb[q];
        if (H == 0) continue;
        // runs of haplotypes for chains
        segs.clear();
        chain_segments(hb[q], hb[q + 1], ho, max_cols,
                       [&](int32_t h0, int32_t n, int64_t len) { segs.push_back(Seg{h0, n, len}); });
        by_bin.clear();
        for (int32_t r = rb[q]; r < rb[q + 1]; ++r) {
            const int64_t m = ro[r + 1] - ro[r];
            by_bin.push_back({m2bin[std::min<int64_t>(m, kMaxReadLen + 1)], r});
        }
        std::stable_sort(by_bin.begin(), by_bin.end(),
                         [](const std::pair<int, int32_t> &a, const std::pair<int, int32_t> &b) { return a.first < b.first; });
        auto out_of = [&](int32_t r, int32_t h) {
            return (int32_t)(out_off[q] + (int64_t)(r - rb[q]) * H + (h - hb[q]));
        };
        auto add_single = [&](int b, int32_t r, int32_t h) {
            const int64_t n = ho[h + 1] - ho[h];
            const int bb = b == p->long_bin ? b : split_bin(b, n);
            singles[bb].push_back(Tile{n, (int64_t)pool.size(), 1});
            pool.push_back(PairRec{r, h, out_of(r, h), (int32_t)n});
        };
        size_t i = 0;
        while (i < by_bin.size()) {
            const int b = by_bin[i].first;
            size_t e = i;
            while (e < by_bin.size() && by_bin[e].first == b) ++e;
            const int cnt = (int)(e - i);
            const int G = 64 / binP(b);
            for (const Seg &sg : segs) {
                const bool chain = chains_ok && b != p->long_bin && sg.H >= 2 && binP(b) >= 16;
                const int nt = chain ? cnt / G : 0;
                // the chain in pieces of at most piece_cols columns
                for (int32_t h = sg.h0; nt && h < sg.h0 + sg.H;) {
                    const int64_t pos = ho[h] - ho[sg.h0] + (int64_t)kChainSep * (h - sg.h0);  // in the chain
                    int64_t len = ho[h + 1] - ho[h];
                    int32_t e2 = h + 1;
                    while (e2 < sg.h0 + sg.H && len + kChainSep + ho[e2 + 1] - ho[e2] <= piece_cols) {
                        len += kChainSep + ho[e2 + 1] - ho[e2];
                        ++e2;
                    }
                    const int32_t n = chain_n(e2 - h, (int)(pos % ring_chunk(binP(b))));
                    for (int t = 0; t < nt; ++t) {
                        chain_tiles[b].push_back(Tile{len, (int64_t)pool.size(), G});
                        for (int g = 0; g < G; ++g) {
                            const int32_t r = by_bin[i + (size_t)t * G + g].second;
                            pool.push_back(PairRec{r, h, out_of(r, h), n});
                        }
                    }
                    h = e2;
                }
                for (size_t k = i + (size_t)nt * G; k < e; ++k)
                    for (int32_t h = sg.h0; h < sg.h0 + sg.H; ++h) add_single(b, by_bin[k].second, h);
            }
            i = e;
        }
    }
    auto longest_first = [](const Tile &a, const Tile &b) { return a.len > b.len; };
    recs.clear();
    recs.reserve(pool.size());
    p->bin_tiles.assign(nbins, 0);
    p->bin_cols.assign(nbins, 0);
    p->binned_ns = 0;
    p->chain_tiles = false;
    int64_t tiles = 0;
    for (int b = 0; b < nbins; ++b) {
        std::stable_sort(chain_tiles[b].begin(), chain_tiles[b].end(), longest_first);
        std::stable_sort(singles[b].begin(), singles[b].end(), longest_first);
        img.bin_rec_begin[b] = (int32_t)recs.size();
        img.bin_tile_begin[b] = (int32_t)tiles;
        for (const Tile &t : chain_tiles[b])
            for (int g = 0; g < t.count; ++g) recs.push_back(pool[(size_t)t.first + g]);
        for (const Tile &t : singles[b]) recs.push_back(pool[(size_t)t.first]);
        const int G = 64 / binP(b);
        for (const auto *l : {&chain_tiles[b], &singles[b]})
            if (!l->empty()) p->bin_cols[b] = std::max(p->bin_cols[b], l->front().len);
        p->bin_tiles[b] = (int64_t)chain_tiles[b].size() + ((int64_t)singles[b].size() + G - 1) / G;
        int64_t steps = 0;
        for (const Tile &t : chain_tiles[b]) steps += t.len + kBinnedSteps;
        for (size_t k = 0; k < singles[b].size(); k += G) steps += singles[b][k].len + kBinnedSteps;
        p->binned_ns += bin_ns((double)steps, binP(b), p->table[nbins - 1 - b].K);
        p->binned_ns += kSingleNs * std::min(binP(b), 16) * (double)singles[b].size();
        p->chain_tiles = p->chain_tiles || !chain_tiles[b].empty();
        tiles += p->bin_tiles[b];
    }
    img.bin_rec_begin[nbins] = (int32_t)recs.size();
    img.bin_tile_begin[nbins] = (int32_t)tiles;
    p->chain_rec_base = (int32_t)recs.size();
    // every pair exactly once
    std::vector<uint8_t> seen((size_t)p->P, 0);
    for (const PairRec &r : recs) {
        const int32_t cnt = r.n < 0 ? chain_haps(r.n) : 1;
        for (int32_t k = 0; k < cnt; ++k) {
            const int64_t o = (int64_t)r.out + k;
            if (o < 0 || o >= p->P || seen[(size_t)o]) return false;
            seen[(size_t)o] = 1;
        }
    }
    for (uint8_t v : seen)
        if (!v) return false;
    return true;
}

// A plan takes the one-pair launch (its bins would run on side streams in turn).
bool one_pair_plan(const ph_plan *p, const int32_t *rb, const int32_t *hb, const int64_t *ro, const int64_t *ho)
{
    double steps = 0, row_steps = 0;
    int64_t long_pairs = 0;
    for (int32_t q = 0; q < p->nb; ++q) {
        const int64_t R = rb[q + 1] - rb[q], H = hb[q + 1] - hb[q];
        int64_t K_sum = 0, long_reads = 0;
        for (int32_t r = rb[q]; r < rb[q + 1]; ++r) {
            const int m = (int)(ro[r + 1] - ro[r]);
            K_sum += (m + 64) >> 6;
            long_reads += m > 255;
        }
        const double tile = (double)(ho[hb[q + 1]] - ho[hb[q]] + kOneSteps * H);
        steps += (double)R * tile;
        row_steps += (double)K_sum * tile;
        long_pairs += long_reads * H;
    }
    const double one = one_pair_ns(p->P, steps, row_steps, p->max_n, p->max_m, long_pairs);
    double stream[kSideStreams] = {};
    const int nbins = (int)p->table.size();
    int next = 0;
    for (int b = 0; b < nbins; ++b) {
        const TuneEntry &e = p->table[nbins - 1 - b];
        if (p->bin_cols[b]) stream[next++ % kSideStreams] += tile_ns(p->bin_cols[b], e.P, e.K);
    }
    return within_binned(one, kBinnedNs + kNextBinNs * (next - 1), p->binned_ns,
                         *std::max_element(stream, stream + kSideStreams));
}

// The one-pair launches of a call with reads of up to 255 bases and longer ones.
// Two launches, one after the other, each take at least one pair's sweep; in one,
// every pair holds the longer reads' tables (25 KB up to 511 bases, 6 a CU; 50 KB
// beyond, 3 a CU).  One launch wins up to about three rounds of 1,536 pairs and
// loses from five (us, two / one; reads of 60-300 bases x 400: 1,500 pairs 80 /
// 48, 4,000 168 / 112, 6,000 218 / 141, 8,000 185 / 186, 12,000 261 / 266;
// 60-260 x 360: 4,000 107 / 92, 6,000 130 / 125, 8,000 152 / 166, 12,000 198 /
// 235; 60-260 x 1,000: 4,000 226 / 198, 8,000 328 / 369), with reads over 511
// bases up to the one round of 768 that kOneLongPairs allows (60-600 bases, 100
// pairs 345 / 300, 700 pairs 350 / 300).
constexpr int kOneUpTo511Pairs = 4096;
hipError_t launch_one_pairs(const SweepArgs &sa, const OneArgs &oa, const bool *reads, int max_m, int pairs,
                            hipStream_t s)
{
    if (reads[0] && reads[1]) {
        if (max_m <= 511 && pairs <= kOneUpTo511Pairs) return launch_one(sa, oa, kOneUpTo511, pairs, s);
        if (pairs <= kOneLongPairs) return launch_one(sa, oa, kOneUpTo1023, pairs, s);
    }
    hipError_t e = reads[1] ? launch_one(sa, oa, kOneLong, pairs, s) : hipSuccess;
    if (e == hipSuccess && reads[0]) e = launch_one(sa, oa, kOneShort, pairs, s);
    return e;
}

// The pairs of a small plan in the one-pair list, longest sweep first.  The
// lead of a pair puts the groups of its FP32 row sum where its tile in the
// work lists has them: that tile flushes the sum after the columns j with
// j + lane + position = 0 mod its chunk (lane: the one that holds the row past
// the read's last; position: the haplotype's first column in its chain), the
// one-pair tile after those with j + lane' + lead = 0.
std::vector<OneRec> one_list(const ph_plan *p, const std::vector<PairRec> &recs, const Book &img, const int64_t *ro,
                             const int64_t *ho)
{
    struct Item {
        int64_t work;
        OneRec r;
    };
    std::vector<Item> items;
    items.reserve((size_t)p->P);
    const int nbins = (int)p->table.size();
    for (int b = 0; b < nbins; ++b) {
        const TuneEntry &e = p->table[nbins - 1 - b];
        const int chunk = ring_chunk(e.P);
        for (int32_t i = img.bin_rec_begin[b]; i < img.bin_rec_begin[b + 1]; ++i) {
            const PairRec &r = recs[(size_t)i];
            const int m = (int)(ro[r.read + 1] - ro[r.read]), K = (m + 64) / 64;
            const int shift = m / e.K - m / K;
            int64_t pos = r.n < 0 ? chain_lead(r.n) : 0;
            for (int32_t k = 0; k < (r.n < 0 ? chain_haps(r.n) : 1); ++k) {
                const int32_t n = (int32_t)(ho[r.hap + k + 1] - ho[r.hap + k]);
                const int lead = (int)(((pos + shift) % chunk + chunk) % chunk);
                items.push_back(Item{K * ((int64_t)n + 64), OneRec{r.read, r.hap + k, r.out + k, n, lead, chunk}});
                pos += n + kChainSep;
            }
        }
    }
    std::sort(items.begin(), items.end(), [](const Item &a, const Item &b) {
        return a.work != b.work ? a.work > b.work : a.r.out < b.r.out;
    });
    std::vector<OneRec> one;
    one.reserve(items.size());
    for (const Item &i : items) one.push_back(i.r);
    return one;
}

}  // namespace

extern "C" {

void ph_plan_opts_default(ph_plan_opts *o)
{
    if (!o) return;
    memset(o, 0, sizeof(*o));
    o->rescue_threshold = 1e-28;
    o->use_graph = 1;
}

const char *ph_last_error(void) { return g_err.c_str(); }

const char *ph_version(void) { return "libpairhmm 0.1 gfx950"; }

ph_status ph_plan_create(const ph_shape *shape, const ph_plan_opts *opts_in, ph_plan **out)
{
    g_err.clear();
    if (!shape || !out) return fail(PH_ERR_INVALID, "shape or out is NULL");
    *out = nullptr;
    int chain_cols = 0;
    return plan_create(shape, opts_in, chain_cols, out);
}

}  // extern "C"

namespace ph {

ph_status plan_create(const ph_shape *shape, const ph_plan_opts *opts_in, int &chain_cols, ph_plan **out)
{
    ph_plan_opts opts;
    if (opts_in) opts = *opts_in; else ph_plan_opts_default(&opts);
    const int32_t nb = shape->num_batches, nr = shape->num_reads, nh = shape->num_haps;
    if (nb < 0 || nr < 0 || nh < 0) return fail(PH_ERR_INVALID, "negative counts");
    if (nb > 0 && (!shape->batch_read_begin || !shape->batch_hap_begin))
        return fail(PH_ERR_INVALID, "batch arrays are NULL");
    if (!shape->read_offset || !shape->hap_offset) return fail(PH_ERR_INVALID, "offset arrays are NULL");
    if (opts.force_p && opts.force_p != 4 && opts.force_p != 8 && opts.force_p != 16 && opts.force_p != 32 &&
        opts.force_p != 64)
        return fail(PH_ERR_INVALID, "force_p must be 0, 4, 8, 16, 32 or 64");

    // --- shape validation ---------------------------------------------------
    const int32_t *rb = shape->batch_read_begin, *hb = shape->batch_hap_begin;
    const int64_t *ro = shape->read_offset, *ho = shape->hap_offset;
    if (ro[0] != 0 || ho[0] != 0) return fail(PH_ERR_INVALID, "read_offset[0] and hap_offset[0] must be 0");
    int32_t max_m = 0, max_n = 0;
    for (int32_t r = 0; r < nr; ++r) {
        int64_t m = ro[r + 1] - ro[r];
        if (m < 1) return fail(PH_ERR_INVALID, "read %d has length %lld", r, (long long)m);
        if (m > kMaxLongReadLen)
            return fail(PH_ERR_UNSUPPORTED, "read %d has length %lld > %d", r, (long long)m, kMaxLongReadLen);
        max_m = std::max<int32_t>(max_m, (int32_t)m);
    }
    for (int32_t h = 0; h < nh; ++h) {
        int64_t n = ho[h + 1] - ho[h];
        if (n < 1) return fail(PH_ERR_INVALID, "haplotype %d has length %lld", h, (long long)n);
        if (n > (1 << 30)) return fail(PH_ERR_UNSUPPORTED, "haplotype %d is too long", h);
        max_n = std::max<int32_t>(max_n, (int32_t)n);
    }
    if (nb > 0 && (rb[0] != 0 || hb[0] != 0)) return fail(PH_ERR_INVALID, "batch ranges must start at 0");
    std::vector<int64_t> out_off(nb + 1, 0);
    for (int32_t q = 0; q < nb; ++q) {
        if (rb[q + 1] < rb[q] || hb[q + 1] < hb[q] || rb[q + 1] > nr || hb[q + 1] > nh)
            return fail(PH_ERR_INVALID, "batch %d has a bad read or haplotype range", q);
        out_off[q + 1] = out_off[q] + (int64_t)(rb[q + 1] - rb[q]) * (hb[q + 1] - hb[q]);
    }
    const int64_t P = nb ? out_off[nb] : 0;
    if (P >= (int64_t)1 << 31) return fail(PH_ERR_UNSUPPORTED, "%lld pairs exceed 2^31 - 1", (long long)P);

    std::unique_ptr<ph_plan, void (*)(ph_plan *)> p(new ph_plan, free_plan);
    p->opts = opts;
    p->threshold = opts.rescue_threshold > 0 ? opts.rescue_threshold : 1e-28;
    p->nb = nb; p->nr = nr; p->nh = nh; p->P = P;
    p->nread_bases = ro[nr];
    p->nhap_bases = ho[nh];
    p->max_m = max_m;
    p->max_n = max_n;

    // --- length bins (host only: a bad table is reported before any GPU call) --
    if (opts.tune_table_path) {
        ph_status st = read_table(opts.tune_table_path, p->table);
        if (st != PH_OK) return st;
    } else if (opts.single_launch && !opts.force_p) {
        p->table = single_table();
    } else {
        p->table = default_table(opts.force_p);
    }
    if (max_m > kMaxReadLen) {
        // the longest bin, swept in windows, never tuned
        if (opts.plain) return fail(PH_ERR_UNSUPPORTED, "plain mode supports reads up to %d bases", kMaxReadLen);
        if ((int)p->table.size() >= kMaxBins) return fail(PH_ERR_INVALID, "too many bins");
        p->table.push_back(TuneEntry{kMaxLongReadLen, 64, kLongRows / 64});
        p->long_bin = 0;  // bins are numbered longest first
    }
    const int nbins = (int)p->table.size();
    if (max_m > p->table.back().max_m)
        return fail(PH_ERR_UNSUPPORTED, "read length %d exceeds the longest configured bin (%d)", max_m,
                    p->table.back().max_m);
    std::vector<int16_t> m2bin(kMaxReadLen + 2, 0);
    for (int m = 1; m <= kMaxReadLen + 1; ++m) {
        int e = 0;
        while (e < nbins - 1 && p->table[e].max_m < m) ++e;
        m2bin[m] = (int16_t)(nbins - 1 - e);
    }
    std::vector<int32_t> binG(nbins);
    for (int b = 0; b < nbins; ++b) binG[b] = 64 / p->table[nbins - 1 - b].P;
    // haplotype-length splits: split[b] = first bucket sent to bin split[kMaxBins + b]
    // (kBuckets: none); the alt entry follows its parent, so its bin is b - 1
    std::vector<int16_t> split(2 * kMaxBins, 0);
    bool any_split = false;
    for (int b = 0; b < nbins; ++b) {
        const TuneEntry &e = p->table[nbins - 1 - b];
        split[b] = (int16_t)(e.n_split ? hap_bucket(e.n_split) : kBuckets);
        split[kMaxBins + b] = (int16_t)(e.n_split ? b - 1 : b);
        any_split = any_split || e.n_split;
    }
    int64_t cells = 0, few_items = 0;  // few_items: windows of the long pairs at kLongK32Few rows per lane
    for (int32_t q = 0; q < nb; ++q) {
        const int64_t H = hb[q + 1] - hb[q];
        int64_t nsum = 0;
        for (int32_t h = hb[q]; h < hb[q + 1]; ++h) nsum += ho[h + 1] - ho[h];
        for (int32_t r = rb[q]; r < rb[q + 1]; ++r) {
            const int m = (int)(ro[r + 1] - ro[r]);
            const int bin = m2bin[std::min(m, kMaxReadLen + 1)];
            cells += (int64_t)m * nsum;
            if (bin == p->long_bin) {  // every pair of the long bin gets a boundary slot
                p->long_pairs += H;
                few_items += H * (m / (64 * kLongK32Few) + 1);
                for (int32_t h = hb[q]; h < hb[q + 1]; ++h)
                    p->bnd_stride = std::max<int64_t>(p->bnd_stride, 3 * (ho[h + 1] - ho[h] + 1));
            } else {
                p->class_pairs[rescue_class_of(m)] += H;
            }
        }
    }
    p->cells = cells;
    // 3 waves per SIMD of 4-row windows (the few) fill the GPU; more items than
    // that take 16 rows per lane (the many).  us, few / many, by windows of the
    // few: reads of 1,100-2,000 x 1,500-3,000 at 654 811 / 1,160, 2,598 1,018 /
    // 1,319, 3,616 1,157 / 1,419, 5,218 1,446 / 1,528, 7,760 1,837 / 1,951;
    // 1,030-1,100 x 1,200-1,500 at 2,800 676 / 817, 4,000 807 / 940, 6,000 982 /
    // 1,016; 4,000-8,000 x 5,000-9,000 at 2,276 3,769 / 4,609, 6,788 7,755 /
    // 8,283.  With every pair swept again in FP64: 1,044 / 1,078 (2,800), 1,413 /
    // 1,320 (4,000), 1,957 / 1,640 (6,000), 2,143 / 2,152 (5,218), 2,951 / 2,890
    // (7,760).  So the line is on the safe side for FP64 and early, by 4-23% of a
    // call, where nearly all results stay in FP32.
    p->long_few = few_items <= 3072;
    p->windows = max_m / (64 * (p->long_few ? kLongK32Few : kLongK32Many)) + 1;
    p->windows64 = max_m / (64 * kLongK64) + 1;
    p->bnd_stride = (p->bnd_stride + 11) / 12 * 12;
    // the split table travels behind the length map in the same device array
    if (any_split) {
        p->split_at = (int)m2bin.size();
        m2bin.insert(m2bin.end(), split.begin(), split.end());
    }
    Book img{};
    std::vector<PairRec> recs;
    if (opts.plain && !out) return PH_OK;
    if (!opts.plain) {
        const int own_cols = choose_chain_cols(p.get(), nb, rb, hb, ro, ho, m2bin);
        if (!chain_cols) chain_cols = own_cols;
        if (!out) return PH_OK;
        // chains longer than the plan's own choice are swept in pieces of that
        // length (a part of 1e10 cells of a batch of 5.2e10, on its own: tiles of
        // 4,096 columns leave its bins uneven, 10.2 against 9.1 ms for the batch)
        const int piece = std::min(own_cols, chain_cols);
        if (!build_lists(p.get(), rb, hb, ro, ho, out_off, m2bin, split, chain_cols, piece, recs, img))
            return fail(PH_ERR_INVALID, "internal: the work lists do not cover every pair once");
    }
    // small plans (reads of up to 1,023 bases, no option that names a launch)
    std::vector<OneRec> one;
    if (!opts.plain && !opts.force_p && !opts.single_launch && P > 0 && max_m <= kMaxReadLen &&
        one_pair_plan(p.get(), rb, hb, ro, ho)) {
        p->one = true;
        one = one_list(p.get(), recs, img, ro, ho);
        for (const OneRec &r : one) p->one_reads[ro[r.read + 1] - ro[r.read] > 255] = true;
        p->one_max_m = max_m;
    }
    // the first HIP calls (everything above is host work)
    HIPCHK(hipGetDevice(&p->device));
    HIPCHK(hipDeviceGetAttribute(&p->cus, hipDeviceAttributeMultiprocessorCount, p->device));
    std::call_once(g_lut_once, [] { g_lut_status = upload_luts(); });
    HIPCHK(g_lut_status);
    p->bin_grid.assign(nbins, 0);
    for (int b = 0; b < nbins; ++b) {
        // (a chain tile can sit in a split's second bin although no single
        // pair's haplotype reaches the split: bins are launched by tiles)
        if (opts.plain || !p->bin_tiles[b] || b == p->long_bin) continue;
        const TuneEntry &e = p->table[nbins - 1 - b];
        const int64_t tiles = p->bin_tiles[b];
        const int64_t cap = (int64_t)p->cus * fwd32_blocks_per_cu(e.P, e.K);
        p->bin_grid[b] = (int)std::min<int64_t>(tiles, cap);
    }
    // side streams of the bin kernels: the long-read bin first, then the bins
    // longest reads first, round-robin, so that every stream starts with its
    // longest tiles.  (Balancing the streams' estimated work instead, largest
    // first, was 6% slower on the mixed batch.)
    {
        p->launch_order.clear();
        int next = 0;
        if (p->long_pairs) p->launch_order.push_back({p->long_bin, next++ % kSideStreams});
        for (int b = 0; b < nbins; ++b)
            if (p->bin_grid[b]) p->launch_order.push_back({b, next++ % kSideStreams});
    }
    if (p->long_pairs) {
        // work items: a pair's windows, few pairs kLongWaves of them at a time
        const int wv = p->long_few ? kLongWaves : 1;
        p->long_grid = (int)std::min<int64_t>(p->long_pairs * ((p->windows + wv - 1) / wv),
                                              (int64_t)p->cus * long32_blocks_per_cu(p->long_few));
        p->long64_grid = (int)std::min<int64_t>(p->long_pairs * ((p->windows64 + wv - 1) / wv),
                                                (int64_t)p->cus * long64_blocks_per_cu(p->long_few));
    }
    if (opts.single_launch && !opts.plain) {
        bool ok = true;
        int64_t tiles = 0;
        for (int b = 0; b < nbins; ++b) {
            if (!p->bin_tiles[b]) continue;
            const TuneEntry &e = p->table[nbins - 1 - b];
            ok = ok && single_supported(e.P, e.K);
            tiles += p->bin_tiles[b];
        }
        if (ok && tiles > 0) {
            p->single = true;
            p->single_grid = (int)std::min<int64_t>(tiles, (int64_t)p->cus * fwd32_single_blocks_per_cu());
        }
    }
    for (int g = 0; g < kRescueGroups; ++g)
        p->rescue_grid[g] = (int)std::min<int64_t>(rescue_pairs(p->class_pairs, g),
                                                   (int64_t)p->cus * rescue_blocks_per_cu(g, !p->class_pairs[1]));
    p->plain_K = (max_m + 1 + 63) / 64;
    if (p->plain_K < 1) p->plain_K = 1;
    p->plain_grid = (int)std::min<int64_t>(std::max<int64_t>(P, 1), (int64_t)p->cus * plain32_blocks_per_cu(p->plain_K));

    // --- device scratch -------------------------------------------------------
    ph_status st;
    if ((st = dalloc(&p->d_book, 1))) return st;
    if (opts.plain) {
        if ((st = dalloc(&p->d_out_offset, nb + 1))) return st;
        if ((st = dalloc(&p->d_m2bin, m2bin.size()))) return st;
        if ((st = dalloc(&p->d_bin_G, kMaxBins))) return st;
        if ((st = dalloc(&p->d_hist, kMaxKeys))) return st;
        if ((st = dalloc(&p->d_recs, std::max<int64_t>(P, 1)))) return st;
        HIPCHK(hipMemcpy(p->d_out_offset, out_off.data(), (nb + 1) * sizeof(int64_t), hipMemcpyHostToDevice));
        HIPCHK(hipMemcpy(p->d_m2bin, m2bin.data(), m2bin.size() * sizeof(int16_t), hipMemcpyHostToDevice));
        HIPCHK(hipMemcpy(p->d_bin_G, binG.data(), nbins * sizeof(int32_t), hipMemcpyHostToDevice));
    } else if (p->one) {
        if ((st = dalloc(&p->d_one, one.size()))) return st;
        if ((st = dalloc(&p->d_one_rescued, (size_t)P))) return st;
        HIPCHK(hipMemcpy(p->d_one, one.data(), one.size() * sizeof(OneRec), hipMemcpyHostToDevice));
    } else {
        // the lists' records, then (chain tiles) one FP64 record slot per pair
        const int64_t nrecs = (int64_t)recs.size() + (p->chain_tiles ? P : 0);
        if ((st = dalloc(&p->d_recs, std::max<int64_t>(nrecs, 1)))) return st;
        if ((st = dalloc(&p->d_book_img, 1))) return st;
        HIPCHK(hipMemcpy(p->d_book_img, &img, sizeof(Book), hipMemcpyHostToDevice));
        if (!recs.empty())
            HIPCHK(hipMemcpy(p->d_recs, recs.data(), recs.size() * sizeof(PairRec), hipMemcpyHostToDevice));
        if (p->chain_tiles && (st = dalloc(&p->d_chain_codes, (size_t)(ho[nh] + (int64_t)kChainSep * nh))))
            return st;
        if ((st = dalloc(&p->d_rescue, (size_t)kRescueQueues * std::max<int64_t>(P, 1)))) return st;
    }
    if ((st = dalloc(&p->d_bad, 1))) return st;
    if (p->long_pairs) {
        if ((st = dalloc(&p->d_bnd32, (size_t)(p->long_pairs * p->bnd_stride)))) return st;
        if ((st = dalloc(&p->d_bnd64, (size_t)(p->long_pairs * p->bnd_stride)))) return st;
        if ((st = dalloc(&p->d_long_rescue, (size_t)p->long_pairs * 2))) return st;
        if ((st = dalloc(&p->d_progress, (size_t)(p->long_pairs * (p->windows + 2 * p->windows64))))) return st;
    }
    HIPCHK(hipMemset(p->d_book, 0, sizeof(Book)));

    HIPCHK(hipStreamCreateWithFlags(&p->cap, hipStreamNonBlocking));
    for (auto &s : p->side) HIPCHK(hipStreamCreateWithFlags(&s, hipStreamNonBlocking));
    HIPCHK(hipEventCreateWithFlags(&p->fork, hipEventDisableTiming));
    for (auto &e : p->join) HIPCHK(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    for (auto &e : p->ev) HIPCHK(hipEventCreate(&e));
    for (auto &e : p->ev_adj) HIPCHK(hipEventCreate(&e));
    for (auto *c : {&p->fwd[0], &p->fwd[1], &p->adj}) HIPCHK(hipEventCreateWithFlags(&c->ran, hipEventDisableTiming));
    if (nb > 0) {
        p->h_rb.assign(rb, rb + nb + 1);
        p->h_hb.assign(hb, hb + nb + 1);
    }
    p->h_ro.assign(ro, ro + nr + 1);
    p->h_ho.assign(ho, ho + nh + 1);
    p->h_out_off = out_off;
    std::call_once(g_lut_adj_once, [] { g_lut_adj_status = upload_luts_adjoint(); });
    HIPCHK(g_lut_adj_status);
    if (opts.keep_checkpoints) {
        ph_status ast = build_adjoint(p.get());
        if (ast != PH_OK && ast != PH_ERR_UNSUPPORTED) return ast;
    }
    *out = p.release();
    return PH_OK;
}

}  // namespace ph

extern "C" {

ph_status ph_plan_info(const ph_plan *p, int64_t *num_pairs, int64_t *num_cells, int32_t *max_read_len,
                       int32_t *max_hap_len)
{
    if (!p) return fail(PH_ERR_INVALID, "plan is NULL");
    if (num_pairs) *num_pairs = p->P;
    if (num_cells) *num_cells = p->cells;
    if (max_read_len) *max_read_len = p->max_m;
    if (max_hap_len) *max_hap_len = p->max_n;
    return PH_OK;
}

void ph_plan_destroy(ph_plan *p) { free_plan(p); }

}  // extern "C"

namespace {

BinArgs bin_args(ph_plan *p, const ph_problem *pb)
{
    BinArgs a{};
    a.num_pairs = p->P;
    a.num_batches = p->nb;
    a.out_offset = p->d_out_offset;
    a.batch_read_begin = pb->batch_read_begin;
    a.batch_hap_begin = pb->batch_hap_begin;
    a.read_offset = pb->read_offset;
    a.hap_offset = pb->hap_offset;
    a.m2bin = p->d_m2bin;
    a.split = p->split_at >= 0 ? p->d_m2bin + p->split_at : nullptr;
    a.num_bins = (int32_t)p->table.size();
    a.bin_G = p->d_bin_G;
    a.hist = p->d_hist;
    a.recs = p->d_recs;
    a.book = p->d_book;
    return a;
}

SweepArgs sweep_args(ph_plan *p, const ph_problem *pb, const double *lin, double *out, uint8_t *status)
{
    SweepArgs a{};
    a.pb.read_offset = pb->read_offset;
    a.pb.read_bases = pb->read_bases;
    a.pb.bq = pb->base_qual;
    a.pb.iq = pb->ins_qual;
    a.pb.dq = pb->del_qual;
    a.pb.gq = pb->gcp_qual;
    a.pb.hap_offset = pb->hap_offset;
    a.pb.hap_bases = pb->hap_bases;
    a.pb.log10_params = nullptr;
    a.lin_params = lin;
    a.recs = p->d_recs;
    a.book = p->d_book;
    a.out_log10 = out;
    a.out_status = status;
    a.rescue_list = p->d_rescue;
    a.rescue_stride = std::max<int64_t>(p->P, 1);
    a.threshold = p->threshold;
    a.floor64 = std::ldexp(1.0, -1000);
    a.num_bins = (int32_t)p->table.size();
    for (int b = 0; b < a.num_bins; ++b) {
        const TuneEntry &e = p->table[a.num_bins - 1 - b];
        a.bins[b] = {e.P, e.K};
    }
    a.plain_count = (int32_t)p->P;
    a.long_bin = p->long_pairs ? p->long_bin : -1;
    a.bnd_stride = p->bnd_stride;
    a.long_rescue_list = p->d_long_rescue;
    a.long_plain_list = p->d_long_rescue ? p->d_long_rescue + p->long_pairs : nullptr;
    a.chain_codes = p->d_chain_codes;
    a.chain_rec_base = p->chain_rec_base;
    a.chain_recs = p->chain_tiles ? p->d_recs + p->chain_rec_base : nullptr;
    return a;
}

// Enqueue one stage of the forward sequence on stream s:
//   0 = parameter exponentiation (explicit mode) and binning,
//   1 = FP32 sweeps of all bins, 2 = FP64 rescue sweeps.
ph_status enqueue_stage(ph_plan *p, int stage, const ph_problem *pb, const float *log10_params, double *out,
                        uint8_t *status, hipStream_t s, bool viterbi)
{
    const double *lin = log10_params ? p->d_lin : nullptr;
    SweepArgs sa = sweep_args(p, pb, lin, out, status);
    sa.viterbi = viterbi ? 1 : 0;
    if (stage == 0) {
        if (log10_params) HIPCHK(launch_prep_params(log10_params, p->nread_bases, p->d_lin, s));
        if (p->opts.plain) {
            const BinArgs ba = bin_args(p, pb);
            HIPCHK(launch_reset_keys(p->d_hist, ba.num_bins * kBuckets, p->d_book, s));
            HIPCHK(launch_plain_records(ba, s));
        } else {
            // the work lists come from plan creation: the book's bin ranges,
            // zero cursors, and the chain code stream of this call's haplotypes
            HIPCHK(launch_prepare(p->d_book, p->d_book_img, pb->hap_offset, pb->hap_bases, p->nh,
                                  p->chain_tiles ? p->d_chain_codes : nullptr, s));
            if (p->long_pairs)  // no window has written a column
                HIPCHK(launch_zero_f32((float *)p->d_progress, p->long_pairs * (p->windows + 2 * p->windows64), s));
        }
    } else if (stage == 1) {
        if (p->opts.plain) {
            HIPCHK(launch_plain32(sa, p->plain_K, p->plain_grid, s));
        } else if (p->single && !viterbi) {
            HIPCHK(launch_fwd32_single(sa, p->single_grid, s));
        } else {
            // the bins on side streams forked from s, in the plan's launch
            // order
            HIPCHK(hipEventRecord(p->fork, s));
            bool used[kSideStreams] = {};
            for (const auto &bk : p->launch_order) {
                const int b = bk.first, k = bk.second;
                if (!used[k]) {
                    HIPCHK(hipStreamWaitEvent(p->side[k], p->fork, 0));
                    used[k] = true;
                }
                if (b == p->long_bin && p->long_pairs) {
                    SweepArgs la = sa;
                    la.bnd = p->d_bnd32;
                    la.windows = p->windows;
                    la.progress = p->d_progress;
                    HIPCHK(launch_long32(la, p->long_few, p->long_grid, p->side[k]));
                } else {
                    HIPCHK(launch_fwd32(sa, sa.bins[b].P, sa.bins[b].K, b, p->bin_grid[b], p->side[k]));
                }
            }
            for (int k = 0; k < kSideStreams; ++k) {
                if (!used[k]) continue;
                HIPCHK(hipEventRecord(p->join[k], p->side[k]));
                HIPCHK(hipStreamWaitEvent(s, p->join[k], 0));
            }
        }
    } else if (!p->opts.plain) {
        for (int g = 0; g < kRescueGroups; ++g)
            if (p->rescue_grid[g]) HIPCHK(launch_rescue(sa, g, !p->class_pairs[1], p->rescue_grid[g], s));
        if (p->long_pairs) {
            SweepArgs la = sa;
            la.bnd = p->d_bnd64;
            la.windows = p->windows64;
            la.progress = p->d_progress + p->long_pairs * p->windows;
            HIPCHK(launch_long64(la, p->long_few, true, p->long64_grid, s));
            la.progress += p->long_pairs * p->windows64;
            HIPCHK(launch_long64(la, p->long_few, false, p->long64_grid, s));
        }
    }
    return PH_OK;
}

// The adjoint's launch sequence: parameter preparation, zeroing of the
// counters (and of the gradient when some read has no pair; kernels, so that
// the sequence can be captured), the persistent FP32 launches, the FP64 launches of the classes present, then the
// fixed-order sum of the per-pair rows of reads with several pairs.
ph_status enqueue_backward(ph_plan *p, const ph_problem *pb, const float *log10_params,
                           const double *grad_log10L, float *grad_params, hipStream_t s)
{
    if (log10_params) HIPCHK(launch_prep_params(log10_params, p->nread_bases, p->d_lin, s));
    if (p->adj_zero) HIPCHK(launch_zero_f32(grad_params, p->nread_bases * 7, s));
    HIPCHK(launch_zero_i32(p->d_adj_ctr, 2 * kAdj64Classes + (int)p->adj_launches.size(), s));
    AdjArgs a{};
    a.pb.read_offset = pb->read_offset;
    a.pb.read_bases = pb->read_bases;
    a.pb.bq = pb->base_qual;
    a.pb.iq = pb->ins_qual;
    a.pb.dq = pb->del_qual;
    a.pb.gq = pb->gcp_qual;
    a.pb.hap_offset = pb->hap_offset;
    a.pb.hap_bases = pb->hap_bases;
    a.lin_params = log10_params ? p->d_lin : nullptr;
    a.ws = p->d_ws;
    a.grad_in = grad_log10L;
    a.grad_out = grad_params;
    a.grad_pair = p->d_grad_pair;
    a.threshold = p->threshold;
    a.all_recs = p->d_adj_recs;
    a.q64 = p->d_q64;
    a.q64_stride = p->q64_stride;
    a.q64_count = p->d_adj_ctr;
    a.q64_next = p->d_adj_ctr + kAdj64Classes;
    a.ws64 = p->d_ws64;
    a.ws64_stride = p->ws64_stride;
    a.hs_bytes64 = p->hs_bytes64;
    a.floor64 = std::ldexp(1.0, -1000);
    for (size_t k = 0; k < p->adj_launches.size(); ++k) {
        const ph_plan::AdjLaunch &L = p->adj_launches[k];
        for (size_t r = 0; r < L.runs.size(); ++r) a.runs[r] = L.runs[r];
        a.tiles = p->d_adj_tiles + L.tile_begin;
        a.ntiles = L.ntiles;
        a.tile_next = p->d_adj_ctr + 2 * kAdj64Classes + k;
        a.ws_stride = L.ws_stride;
        HIPCHK(launch_adj32(a, L.runs.size() == 1 ? L.runs[0].P : 0, L.runs[0].K, L.lds, L.grid, s));
    }
    // pairs out of the FP32 range
    HIPCHK(launch_adj64(a, p->k64_only, p->k64_max, p->grid64, s));
    HIPCHK(launch_adj_reduce(p->d_red, p->n_red, p->d_grad_pair, grad_params, s));
    return PH_OK;
}

// Whether a call on stream s replays captured launches (graph) or enqueues them
// itself.  The first set of pointers is captured at once, another when it comes twice
// in a row: calls whose buffers alternate, as autograd's do, would capture and
// instantiate a graph each (0.3 ms and more) and wait for the one that it takes the
// place of.  That one is let go only after its last launch has run, which no call
// waits for: until then calls enqueue their launches themselves.
template <typename F>
ph_status use_captured(ph_plan *p, ph_plan::Captured &c, std::vector<const void *> key, hipStream_t s, bool &graph,
                       F enqueue)
{
    graph = false;
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (!p->opts.use_graph) return PH_OK;
    HIPCHK(hipStreamIsCapturing(s, &cs));
    if (cs != hipStreamCaptureStatusNone) {  // the caller's own graph takes the launches
        p->events_captured = true;
        return PH_OK;
    }
    const bool again = c.last.empty() || key == c.last;
    c.last = key;
    if (c.exec && key == c.key) {
        c.marked = false;
        graph = true;
        return PH_OK;
    }
    if (c.exec) {
        if (!c.marked) HIPCHK(hipEventRecord(c.ran, s));
        c.marked = true;
        if (!again) return PH_OK;
        if (hipEventQuery(c.ran) != hipSuccess) {
            (void)hipGetLastError();  // (not ready: no error)
            return PH_OK;
        }
        drop_captured(c);
    }
    if (!again) return PH_OK;
    HIPCHK(hipStreamBeginCapture(p->cap, hipStreamCaptureModeRelaxed));
    const ph_status st = enqueue(p->cap);
    hipGraph_t g = nullptr;
    const hipError_t e = hipStreamEndCapture(p->cap, &g);
    if (st != PH_OK) {
        if (g) (void)hipGraphDestroy(g);
        return st;
    }
    if (e != hipSuccess) return fail(PH_ERR_HIP, "hipStreamEndCapture: %s", hipGetErrorString(e));
    c.graph = g;
    const hipError_t ei = hipGraphInstantiate(&c.exec, g, nullptr, nullptr, 0);
    if (ei != hipSuccess) {
        c.exec = nullptr;
        drop_captured(c);
        return fail(PH_ERR_HIP, "hipGraphInstantiate: %s", hipGetErrorString(ei));
    }
    c.key = std::move(key);
    graph = true;
    return PH_OK;
}

// The forward call and the Viterbi call: the same three stages, with the
// sum (forward) or the maximum (Viterbi) in the sweeps, each mode with its
// own stage graphs.
ph_status run_forward(ph_plan *p, const ph_problem *pb, const float *log10_params, double *out_log10L,
                      uint8_t *out_status, void *stream_v, bool viterbi)
{
    g_err.clear();
    if (!p) return fail(PH_ERR_INVALID, "plan is NULL");
    ph_status st = check_problem(p, pb);
    if (st != PH_OK) return st;
    if (p->P == 0) return PH_OK;
    if (!out_log10L) return fail(PH_ERR_INVALID, "out_log10L is NULL");
    if (!log10_params && (!pb->base_qual || !pb->ins_qual || !pb->del_qual || !pb->gcp_qual))
        return fail(PH_ERR_INVALID, "Phred arrays are NULL and no log10 parameters were given");
    if (viterbi && p->opts.plain) return fail(PH_ERR_UNSUPPORTED, "the Viterbi score needs a binned plan");
    hipStream_t s = (hipStream_t)stream_v;
    if (log10_params && p->lin_cap < p->nread_bases) {
        if (p->d_lin) HIPCHK(hipFree(p->d_lin));
        p->d_lin = nullptr;
        if ((st = dalloc(&p->d_lin, (size_t)p->nread_bases * 8))) return st;
        p->lin_cap = p->nread_bases;
        drop_graphs(p);
    }
    const int v = viterbi ? 1 : 0;

    if (p->one) {
        // a small call: launched directly, one or two kernels
        const double *lin = log10_params ? p->d_lin : nullptr;
        SweepArgs sa = sweep_args(p, pb, lin, out_log10L, out_status);
        sa.viterbi = v;
        OneArgs oa{};
        oa.recs = p->d_one;
        oa.rescued = p->d_one_rescued;
        HIPCHK(hipEventRecord(p->ev[0], s));
        if (log10_params) HIPCHK(launch_prep_params(log10_params, p->nread_bases, p->d_lin, s));
        HIPCHK(launch_one_pairs(sa, oa, p->one_reads, p->one_max_m, (int)p->P, s));
        HIPCHK(hipEventRecord(p->ev[3], s));
        p->last_stream = s;
        p->stages_recorded = true;
        p->forward_done = true;
        return PH_OK;
    }

    // The FP32 stage (one launch per bin, on side streams) is captured into a
    // graph; the stages before and after it are a launch or two.  HIP events
    // recorded on the caller's stream around the stages time them.
    bool graph = false;
    st = use_captured(p, p->fwd[v],
                      {pb->batch_read_begin, pb->batch_hap_begin, pb->read_offset, pb->read_bases, pb->base_qual,
                       pb->ins_qual, pb->del_qual, pb->gcp_qual, pb->hap_offset, pb->hap_bases, log10_params,
                       out_log10L, out_status},
                      s, graph, [&](hipStream_t cs) {
                          return enqueue_stage(p, 1, pb, log10_params, out_log10L, out_status, cs, viterbi);
                      });
    if (st != PH_OK) return st;
    for (int stage = 0; stage < 3; ++stage) {
        HIPCHK(hipEventRecord(p->ev[stage], s));
        if (stage == 1 && graph) {
            HIPCHK(hipGraphLaunch(p->fwd[v].exec, s));
        } else {
            st = enqueue_stage(p, stage, pb, log10_params, out_log10L, out_status, s, viterbi);
            if (st != PH_OK) return st;
        }
    }
    HIPCHK(hipEventRecord(p->ev[3], s));
    p->last_stream = s;
    p->stages_recorded = true;
    p->forward_done = true;
    return PH_OK;
}

}  // namespace

extern "C" {

ph_status ph_forward_batch(ph_plan *p, const ph_problem *pb, const float *log10_params, double *out_log10L,
                           uint8_t *out_status, void *stream_v)
{
    return run_forward(p, pb, log10_params, out_log10L, out_status, stream_v, false);
}

ph_status ph_viterbi_batch(ph_plan *p, const ph_problem *pb, const float *log10_params, double *out_log10V,
                           uint8_t *out_status, void *stream_v)
{
    return run_forward(p, pb, log10_params, out_log10V, out_status, stream_v, true);
}

ph_status ph_backward_batch(ph_plan *p, const ph_problem *pb, const float *log10_params,
                            const double *grad_log10L, float *grad_params, void *stream_v)
{
    g_err.clear();
    if (!p) return fail(PH_ERR_INVALID, "plan is NULL");
    ph_status st = check_problem(p, pb);
    if (st != PH_OK) return st;
    if (p->P == 0) return PH_OK;
    if (!grad_log10L || !grad_params) return fail(PH_ERR_INVALID, "gradient buffers are NULL");
    if (!log10_params && (!pb->base_qual || !pb->ins_qual || !pb->del_qual || !pb->gcp_qual))
        return fail(PH_ERR_INVALID, "Phred arrays are NULL and no log10 parameters were given");
    st = build_adjoint(p);
    if (st != PH_OK) return p->adj_error.empty() ? st : fail(st, "%s", p->adj_error.c_str());
    hipStream_t s = (hipStream_t)stream_v;
    if (log10_params && p->lin_cap < p->nread_bases) {
        if (p->d_lin) HIPCHK(hipFree(p->d_lin));
        p->d_lin = nullptr;
        if ((st = dalloc(&p->d_lin, (size_t)p->nread_bases * 8))) return st;
        p->lin_cap = p->nread_bases;
        drop_graphs(p);
    }
    bool graph = false;
    st = use_captured(p, p->adj,
                      {pb->read_offset, pb->read_bases, pb->base_qual, pb->ins_qual, pb->del_qual, pb->gcp_qual,
                       pb->hap_offset, pb->hap_bases, log10_params, grad_log10L, grad_params},
                      s, graph, [&](hipStream_t cs) {
                          return enqueue_backward(p, pb, log10_params, grad_log10L, grad_params, cs);
                      });
    if (st != PH_OK) return st;
    HIPCHK(hipEventRecord(p->ev_adj[0], s));
    if (graph) {
        HIPCHK(hipGraphLaunch(p->adj.exec, s));
    } else {
        st = enqueue_backward(p, pb, log10_params, grad_log10L, grad_params, s);
        if (st != PH_OK) return st;
    }
    HIPCHK(hipEventRecord(p->ev_adj[1], s));
    p->adj_recorded = true;
    return PH_OK;
}

ph_status ph_validate(ph_plan *p, const ph_problem *pb, void *stream_v)
{
    g_err.clear();
    if (!p) return fail(PH_ERR_INVALID, "plan is NULL");
    ph_status st = check_problem(p, pb);
    if (st != PH_OK) return st;
    hipStream_t s = (hipStream_t)stream_v;
    DevProblem d{};
    d.read_bases = pb->read_bases;
    d.hap_bases = pb->hap_bases;
    // a counter of its own: the forward's bookkeeping (rescue counts, bin
    // ranges) stays as the last forward call left it
    HIPCHK(hipMemsetAsync(p->d_bad, 0, sizeof(int32_t), s));
    HIPCHK(launch_validate(d, p->nread_bases, p->nhap_bases, p->d_bad, s));
    int32_t bad = 0;
    HIPCHK(hipMemcpyAsync(&bad, p->d_bad, sizeof(bad), hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    if (bad) return fail(PH_ERR_INVALID, "%d base codes outside 0..4", bad);
    return PH_OK;
}

ph_status ph_plan_stage_ms(ph_plan *p, float ms[4])
{
    if (!p || !ms) return fail(PH_ERR_INVALID, "NULL argument");
    if (!p->stages_recorded && !p->adj_recorded) return fail(PH_ERR_STATE, "no forward or backward call recorded");
    for (int i = 0; i < 4; ++i) ms[i] = 0.0f;
    if (p->stages_recorded) {
    HIPCHK(hipEventSynchronize(p->ev[3]));
    if (p->one) {  // one launch: no binning, and the FP64 sweeps are part of it
        HIPCHK(hipEventElapsedTime(&ms[1], p->ev[0], p->ev[3]));
    } else {
    HIPCHK(hipEventElapsedTime(&ms[0], p->ev[0], p->ev[1]));
    HIPCHK(hipEventElapsedTime(&ms[1], p->ev[1], p->ev[2]));
    HIPCHK(hipEventElapsedTime(&ms[2], p->ev[2], p->ev[3]));
    }
    }
    if (p->adj_recorded) {
        HIPCHK(hipEventSynchronize(p->ev_adj[1]));
        HIPCHK(hipEventElapsedTime(&ms[3], p->ev_adj[0], p->ev_adj[1]));
    }
    return PH_OK;
}

ph_status ph_plan_rescued(ph_plan *p, int64_t *count)
{
    if (!p || !count) return fail(PH_ERR_INVALID, "NULL argument");
    if (!p->forward_done) return fail(PH_ERR_STATE, "no forward call recorded");
    HIPCHK(hipEventSynchronize(p->ev[3]));
    if (p->one) {
        std::vector<uint8_t> went((size_t)p->P);
        HIPCHK(hipMemcpy(went.data(), p->d_one_rescued, went.size(), hipMemcpyDeviceToHost));
        *count = 0;
        for (uint8_t w : went) *count += w;
        return PH_OK;
    }
    int32_t c[kRescueQueues], lc = 0, lp = 0, passed = 0;
    HIPCHK(hipMemcpy(c, p->d_book->rescue_count, sizeof(c), hipMemcpyDeviceToHost));
    HIPCHK(hipMemcpy(&lc, &p->d_book->long_rescue_count, sizeof(lc), hipMemcpyDeviceToHost));
    HIPCHK(hipMemcpy(&lp, &p->d_book->long_plain_count, sizeof(lp), hipMemcpyDeviceToHost));
    HIPCHK(hipMemcpy(&passed, &p->d_book->rescue_passed, sizeof(passed), hipMemcpyDeviceToHost));
    // pairs of reads longer than 1023 bases (windowed FP64 sweeps) and both sets of
    // queues, less those that a rescaled sweep passed on (counted twice)
    *count = (int64_t)lc + lp - passed;
    for (int i = 0; i < kRescueQueues; ++i) *count += c[i];
    return PH_OK;
}

}  // extern "C"

// ---------------------------------------------------------------------------
// Allocation-free forward (ph_forward_batch_noalloc): the scratch of the
// binning, the FP32 sweeps and the FP64 rescue lives in one fixed device
// array of this library instead of plan-owned buffers.  Its layout, at
// 256-byte aligned offsets: the bookkeeping (Book), the key histogram, the
// read-length -> bin map, the pairs per tile of each bin, the batch output
// offsets, the pair records, the FP64 queues and (explicit parameters) the
// linear parameters of every read base.
// ---------------------------------------------------------------------------
namespace {

constexpr int64_t kNaMaxPairs = (int64_t)1 << 16;
constexpr int32_t kNaMaxBatches = 1 << 14;
constexpr int64_t kNaMaxParamBases = (int64_t)1 << 16;  // explicit parameters: read bases
constexpr size_t na_align(size_t x) { return (x + 255) & ~(size_t)255; }
constexpr size_t kNaBook = 0;
constexpr size_t kNaHist = na_align(kNaBook + sizeof(Book));
constexpr size_t kNaM2bin = na_align(kNaHist + (size_t)kMaxKeys * sizeof(int32_t));
constexpr size_t kNaBinG = na_align(kNaM2bin + (size_t)(kMaxReadLen + 2) * sizeof(int16_t));
constexpr size_t kNaOutOff = na_align(kNaBinG + (size_t)kMaxBins * sizeof(int32_t));
constexpr size_t kNaRecs = na_align(kNaOutOff + (size_t)(kNaMaxBatches + 1) * sizeof(int64_t));
constexpr size_t kNaRescue = na_align(kNaRecs + (size_t)kNaMaxPairs * sizeof(PairRec));
constexpr size_t kNaLin = na_align(kNaRescue + (size_t)kRescueQueues * kNaMaxPairs * sizeof(int32_t));
constexpr size_t kNaBytes = na_align(kNaLin + (size_t)kNaMaxParamBases * 8 * sizeof(double));

}  // namespace

// One copy per GPU, held until the process ends.  In host code this name
// is only a stand-in for the symbol: device addresses come from
// hipGetSymbolAddress (NaDevice::base).
static __device__ __align__(256) unsigned char scratch[kNaBytes];

namespace {

constexpr int kNaMaxDevices = 64;

// Per-device state of the allocation-free forward, set up by the first call
// on that device.
struct NaDevice {
    bool ready = false;
    unsigned char *base = nullptr;  // device address of `scratch` on this device
    int cus = 0;
    int fwd32_cap[kMaxBins] = {};   // persistent grid cap of each built-in bin (bin order)
    int rescue_cap[kRescueGroups][2] = {};  // [1: no read of 128 to 255 bases]
};

std::mutex g_na_mu;
NaDevice g_na[kNaMaxDevices];
TuneEntry g_na_table[kMaxBins];  // the built-in table, shortest reads first
int g_na_bins = 0;

ph_status na_device_setup(int dev, NaDevice *&out)
{
    std::lock_guard<std::mutex> lk(g_na_mu);
    NaDevice &d = g_na[dev];
    if (!d.ready) {
        if (!g_na_bins) g_na_bins = builtin_table(g_na_table);
        // the constant tables of the sweeps (per device) and the address of
        // this device's copy of the scratch array
        HIPCHK(upload_luts());
        void *ptr = nullptr;
        HIPCHK(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        HIPCHK(hipDeviceGetAttribute(&d.cus, hipDeviceAttributeMultiprocessorCount, dev));
        for (int b = 0; b < g_na_bins; ++b) {
            const TuneEntry &e = g_na_table[g_na_bins - 1 - b];
            d.fwd32_cap[b] = d.cus * std::max(1, fwd32_blocks_per_cu(e.P, e.K));
        }
        for (int g = 0; g < kRescueGroups; ++g)
            for (int u = 0; u < 2; ++u) d.rescue_cap[g][u] = d.cus * std::max(1, rescue_blocks_per_cu(g, u));
        d.base = (unsigned char *)ptr;
        d.ready = true;
    }
    out = &d;
    return PH_OK;
}

}  // namespace

extern "C" {

ph_status ph_forward_batch_noalloc(const ph_shape *shape, const ph_problem *pb, const float *log10_params,
                                   double *out_log10L, uint8_t *out_status, void *stream_v)
{
    g_err.clear();
    if (!shape || !pb) return fail(PH_ERR_INVALID, "shape or problem is NULL");
    const int32_t nb = shape->num_batches, nr = shape->num_reads, nh = shape->num_haps;
    if (nb < 0 || nr < 0 || nh < 0) return fail(PH_ERR_INVALID, "negative counts");
    if (pb->num_batches != nb || pb->num_reads != nr || pb->num_haps != nh)
        return fail(PH_ERR_PLAN_MISMATCH, "problem has %d batches, %d reads, %d haplotypes; shape has %d, %d, %d",
                    pb->num_batches, pb->num_reads, pb->num_haps, nb, nr, nh);
    if (nb > kNaMaxBatches)
        return fail(PH_ERR_UNSUPPORTED, "%d batches exceed the allocation-free maximum of %d", nb, kNaMaxBatches);
    if (nb > 0 && (!shape->batch_read_begin || !shape->batch_hap_begin))
        return fail(PH_ERR_INVALID, "batch arrays are NULL");
    if (!shape->read_offset || !shape->hap_offset) return fail(PH_ERR_INVALID, "offset arrays are NULL");
    const int32_t *rb = shape->batch_read_begin, *hb = shape->batch_hap_begin;
    const int64_t *ro = shape->read_offset, *ho = shape->hap_offset;
    if (ro[0] != 0 || ho[0] != 0) return fail(PH_ERR_INVALID, "read_offset[0] and hap_offset[0] must be 0");
    for (int32_t r = 0; r < nr; ++r) {
        const int64_t m = ro[r + 1] - ro[r];
        if (m < 1) return fail(PH_ERR_INVALID, "read %d has length %lld", r, (long long)m);
        if (m > kMaxReadLen)
            return fail(PH_ERR_UNSUPPORTED, "read %d has length %lld: the allocation-free forward takes reads up to %d",
                        r, (long long)m, kMaxReadLen);
    }
    for (int32_t h = 0; h < nh; ++h) {
        const int64_t n = ho[h + 1] - ho[h];
        if (n < 1) return fail(PH_ERR_INVALID, "haplotype %d has length %lld", h, (long long)n);
        if (n > (1 << 30)) return fail(PH_ERR_UNSUPPORTED, "haplotype %d is too long", h);
    }
    if (nb > 0 && (rb[0] != 0 || hb[0] != 0)) return fail(PH_ERR_INVALID, "batch ranges must start at 0");
    int64_t P = 0;
    for (int32_t q = 0; q < nb; ++q) {
        if (rb[q + 1] < rb[q] || hb[q + 1] < hb[q] || rb[q + 1] > nr || hb[q + 1] > nh)
            return fail(PH_ERR_INVALID, "batch %d has a bad read or haplotype range", q);
        P += (int64_t)(rb[q + 1] - rb[q]) * (hb[q + 1] - hb[q]);
    }
    if (P > kNaMaxPairs)
        return fail(PH_ERR_UNSUPPORTED, "%lld pairs exceed the allocation-free maximum of %lld", (long long)P,
                    (long long)kNaMaxPairs);
    const int64_t nbases = ro[nr];
    if (log10_params && nbases > kNaMaxParamBases)
        return fail(PH_ERR_UNSUPPORTED, "%lld read bases with explicit parameters exceed the allocation-free maximum of %lld",
                    (long long)nbases, (long long)kNaMaxParamBases);
    if (P == 0) return PH_OK;
    if (!out_log10L) return fail(PH_ERR_INVALID, "out_log10L is NULL");
    if (!pb->batch_read_begin || !pb->batch_hap_begin || !pb->read_offset || !pb->hap_offset ||
        !pb->read_bases || !pb->hap_bases)
        return fail(PH_ERR_INVALID, "problem has a NULL array");
    if (!log10_params && (!pb->base_qual || !pb->ins_qual || !pb->del_qual || !pb->gcp_qual))
        return fail(PH_ERR_INVALID, "Phred arrays are NULL and no log10 parameters were given");

    int dev = 0;
    HIPCHK(hipGetDevice(&dev));
    if (dev < 0 || dev >= kNaMaxDevices) return fail(PH_ERR_UNSUPPORTED, "device %d: too many devices", dev);
    NaDevice *d = nullptr;
    ph_status st = na_device_setup(dev, d);
    if (st != PH_OK) return st;
    const int nbins = g_na_bins;

    // pairs per bin and per FP64 class, from the host shape
    int64_t bin_pairs[kMaxBins] = {}, class_pairs[kRescueClasses] = {}, bin_cols[kMaxBins] = {};
    int64_t bin_steps[kMaxBins] = {};  // of every pair
    int64_t steps = 0, row_steps = 0, n_max = 0, long_pairs = 0;  // of one-pair tiles
    int m_max = 0;
    for (int32_t q = 0; q < nb; ++q) {
        const int64_t R = rb[q + 1] - rb[q], H = hb[q + 1] - hb[q], cols = ho[hb[q + 1]] - ho[hb[q]];
        if (R == 0 || H == 0) continue;
        int64_t n_longest = 0, K_sum = 0, long_reads = 0;
        for (int32_t h = hb[q]; h < hb[q + 1]; ++h) n_longest = std::max(n_longest, ho[h + 1] - ho[h]);
        for (int32_t r = rb[q]; r < rb[q + 1]; ++r) {
            const int m = (int)(ro[r + 1] - ro[r]), b = nbins - 1 - builtin_entry(m);
            bin_pairs[b] += H;
            bin_steps[b] += cols + kBinnedSteps * H;
            bin_cols[b] = std::max(bin_cols[b], n_longest);
            class_pairs[rescue_class_of(m)] += H;
            K_sum += (m + 64) >> 6;
            long_reads += m > 255;
            m_max = std::max(m_max, m);
        }
        steps += R * (cols + kOneSteps * H);
        row_steps += K_sum * (cols + kOneSteps * H);
        n_max = std::max(n_max, n_longest);
        long_pairs += long_reads * H;
    }
    const double one = one_pair_ns(P, (double)steps, (double)row_steps, n_max, m_max, long_pairs);
    const bool one_reads[2] = {long_pairs < P, long_pairs > 0};  // some read of up to 255 bases, some longer one
    // the binned launches run one after the other here
    const double few = (double)std::min<int64_t>(P, kFreeFurther);
    double launches = kFreeNs - kNextBinNs + kFreePairNs * few + kFreeFurtherNs * ((double)P - few) + kFreeBatchNs * nb;
    double sum = 0, ends = 0;
    for (int b = 0; b < nbins; ++b) {
        const TuneEntry &e = g_na_table[nbins - 1 - b];
        if (!bin_pairs[b]) continue;
        launches += kNextBinNs;
        sum += bin_ns((double)bin_steps[b] * e.P / 64, e.P, e.K);
        ends += tile_ns(bin_cols[b], e.P, e.K);
    }

    unsigned char *base = d->base;
    Book *book = (Book *)(base + kNaBook);
    int32_t *hist = (int32_t *)(base + kNaHist);
    int16_t *m2bin = (int16_t *)(base + kNaM2bin);
    int32_t *binG = (int32_t *)(base + kNaBinG);
    int64_t *out_off = (int64_t *)(base + kNaOutOff);
    PairRec *recs = (PairRec *)(base + kNaRecs);
    int32_t *rescue = (int32_t *)(base + kNaRescue);
    double *lin = (double *)(base + kNaLin);
    hipStream_t s = (hipStream_t)stream_v;

    BinTable tab{};
    tab.num_bins = nbins;
    for (int e = 0; e < nbins; ++e) {
        tab.max_m[e] = (int16_t)g_na_table[e].max_m;
        tab.P[e] = (int8_t)g_na_table[e].P;
    }
    SweepArgs sa{};
    sa.pb.read_offset = pb->read_offset;
    sa.pb.read_bases = pb->read_bases;
    sa.pb.bq = pb->base_qual;
    sa.pb.iq = pb->ins_qual;
    sa.pb.dq = pb->del_qual;
    sa.pb.gq = pb->gcp_qual;
    sa.pb.hap_offset = pb->hap_offset;
    sa.pb.hap_bases = pb->hap_bases;
    sa.lin_params = log10_params ? lin : nullptr;
    sa.recs = recs;
    sa.book = book;
    sa.out_log10 = out_log10L;
    sa.out_status = out_status;
    sa.rescue_list = rescue;
    sa.rescue_stride = P;
    sa.threshold = 1e-28;
    sa.floor64 = std::ldexp(1.0, -1000);
    sa.num_bins = nbins;
    for (int b = 0; b < nbins; ++b) sa.bins[b] = {g_na_table[nbins - 1 - b].P, g_na_table[nbins - 1 - b].K};
    sa.plain_count = (int32_t)P;
    sa.long_bin = -1;

    if (within_binned(one, launches, sum, ends)) {
        // a small call: no binning, one pair per wave; the first pair of every
        // batch travels in the kernel's arguments, or is summed up on the
        // device where there are too many batches for that
        OneArgs oa{};
        oa.num_batches = nb;
        oa.batch_read_begin = pb->batch_read_begin;
        oa.batch_hap_begin = pb->batch_hap_begin;
        if (log10_params) HIPCHK(launch_prep_params(log10_params, nbases, lin, s));
        if (nb <= kOneBatches) {
            int32_t first = 0;
            for (int32_t q = 0; q < nb; ++q) {
                oa.first[q] = first;
                first += (rb[q + 1] - rb[q]) * (hb[q + 1] - hb[q]);
            }
        } else {
            HIPCHK(launch_na_setup(pb->batch_read_begin, pb->batch_hap_begin, nb, out_off, m2bin, binG, tab, s));
            oa.out_offset = out_off;
        }
        HIPCHK(launch_one_pairs(sa, oa, one_reads, m_max, (int)P, s));
        return PH_OK;
    }
    // binning (the set-up kernel writes what a plan uploads at creation;
    // kernels only, so that a caller may capture the sequence)
    if (log10_params) HIPCHK(launch_prep_params(log10_params, nbases, lin, s));
    HIPCHK(launch_reset_keys(hist, nbins * kBuckets, book, s));
    HIPCHK(launch_na_setup(pb->batch_read_begin, pb->batch_hap_begin, nb, out_off, m2bin, binG, tab, s));
    BinArgs ba{};
    ba.num_pairs = P;
    ba.num_batches = nb;
    ba.out_offset = out_off;
    ba.batch_read_begin = pb->batch_read_begin;
    ba.batch_hap_begin = pb->batch_hap_begin;
    ba.read_offset = pb->read_offset;
    ba.hap_offset = pb->hap_offset;
    ba.m2bin = m2bin;
    ba.num_bins = nbins;
    ba.bin_G = binG;
    ba.hist = hist;
    ba.recs = recs;
    ba.book = book;
    HIPCHK(launch_bin_count(ba, s));
    HIPCHK(launch_bin_scan(ba, s));
    HIPCHK(launch_bin_scatter(ba, s));

    // FP32 sweeps, longest bin first, then the FP64 rescue (all on `s`)
    for (int b = 0; b < nbins; ++b) {
        if (!bin_pairs[b]) continue;
        const int G = 64 / sa.bins[b].P;
        const int grid = (int)std::min<int64_t>((bin_pairs[b] + G - 1) / G, d->fwd32_cap[b]);
        HIPCHK(launch_fwd32(sa, sa.bins[b].P, sa.bins[b].K, b, grid, s));
    }
    for (int g = 0; g < kRescueGroups; ++g) {
        const int64_t pairs = rescue_pairs(class_pairs, g);
        const bool upto127 = !class_pairs[1];
        if (pairs)
            HIPCHK(launch_rescue(sa, g, upto127, (int)std::min<int64_t>(pairs, d->rescue_cap[g][upto127]), s));
    }
    return PH_OK;
}

}  // extern "C"
