// Internal declarations shared by the source files of libgoodroute (gfx950).
// The public interface and the time model are in goodroute.h.
//
// Closed form used throughout.  Let instance g hold N requests with remaining
// lengths R_i and contexts c_i.  Under continuous batching with step time
// alpha + beta*B + gamma*C, the time of its next L steps is
//     W_g(L) = alpha*L + beta*sum_i min(R_i,L) + gamma*sum_i [c_i*min(R_i,L) + tri(min(R_i,L))]
// with tri(x) = x(x-1)/2, because request i is in the batch for min(R_i,L) of
// those steps and its context at its s-th step is c_i + s - 1.  With the
// requests sorted by R and k = #{i : R_i <= L} this is
//     W_g(L) = alpha*L + beta*(Y_k + (N-k)*L) + gamma*(X_k + L*S_{k+1} + (N-k)*tri(L))
//     Y_k = sum_{i<=k} R_i,  X_k = sum_{i<=k} (c_i*R_i + tri(R_i)),  S_{k+1} = sum_{i>k} c_i,
// three integer prefix sums, exact in 64-bit.  A request r routed to g is one
// more batch member with R = L, so Eq. 2 reads
//     T(r,g) = q_g + delta*c0 + W_g(L) + beta*L + gamma*(c0*L + tri(L))
//            = E_g(L) + c0 * kappa_g(L),
//     E_g(L)     = q_g + W_g(L) + beta*L + gamma*tri(L)      (instance and length only)
//     kappa_g(L) = delta + gamma*L.
// On the segment R_k <= L < R_{k+1}, with n = N - k requests still running:
//     E_g(L) = [q_g + beta*Y_k + gamma*X_k] + L*[alpha + beta*(n+1) + gamma*S_{k+1}] + tri(L)*gamma*(n+1).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <vector>

#include "goodroute.h"

namespace gr {

constexpr int kBlock = 256;
constexpr int kWave = 64;
constexpr int kSimds = 1024;       // 256 compute units of four
constexpr int kMaxEntries = 2048;
constexpr int kMaxClasses = 64;
constexpr int kMaxLen = 32767;     // lengths and row numbers are kept in 16 bits
constexpr int kAllAlike = 1 << 30; // with the entries of an instance (gr_fleet::instK): its segments all have the same (Gq, H) and no curvature
constexpr int kMemoU = 256;        // distinct lengths per block of the table of a scoring pass
constexpr int kDirectMax = 4096;   // most requests of a batch that a caller has scored pair by pair
constexpr int64_t kDirectPairs = int64_t(1) << 19;   // pairs of a batch that is where the sizes decide (see pair_by_pair),
constexpr int64_t kDirectLanes = int64_t(3) << 18;   // and pairs that its lanes go through
constexpr int64_t kDirectInfinite = int64_t(1) << 18;   // pairs (of whole 128 instances) up to which infinite latencies count there
constexpr int kDirectSpan = 4096;  // instances that one workgroup takes of a request scored pair by pair
constexpr int kFeedInst = 512;     // most instances of a fleet whose feedback routing is a launch a round, or one for all
constexpr int kDirectParts = 16384;  // room for the selections of such parts
constexpr int64_t kDenseValues = int64_t(1) << 22;   // values of a table that has a row for every length
constexpr int kMemoP = 16;         // positions of a run of the class order
constexpr int kRanges = 4;         // ranges of prompt lengths that a length's possible least latencies are looked up for
constexpr int kRestParts = 64;     // lists of requests that those do not decide
constexpr int kRestStride = 16;    // ints from one list's counter to the next: a cache line each
constexpr int kRestItems = 2;      // requests per thread that append to a list
constexpr int kRestRuns = 1024;    // most runs of a fleet whose requests are decided that way
constexpr int64_t kTurnedBytes = int64_t(64) << 20;   // room for rows of the table over the instances, where 256 rows fit

// Splitters of an instance's sorted lengths, by table size (strides of 8, 8, 16, 32, 32, 64 lengths).
constexpr int split_count(int cap) { return cap <= 64 ? 8 : cap <= 512 ? 16 : 32; }

// Where the pair (Gq, H) of instance g's segment k = 0 .. cap is kept: segment 1, the first of the
// sorted entries, at a multiple of 16 bytes.
__host__ __device__ constexpr size_t gh_at(int g, int k, int cap) { return (size_t)g * (cap + 2) + 1 + k; }

struct ClassCoef {
    double delta, alpha, beta, gamma;
};

// Where a batch of requests comes from: the caller's arrays (routing) or the
// flagged active requests (migration).
struct ReqSrc {
    const int *ctx0, *pred_len;
    const float* budget;
    const int* exclude;
    const int *act_prompt, *act_gen, *act_rem, *act_inst;
    const uint8_t* flag;
    const float* act_budget;
    const int* act_off;
    int64_t n;
};

struct ScoreOut {
    int* inst;
    float* slack;
    uint8_t* fallback;   // may be null
    float* T;            // may be null: every pair's latency
    int* n_selected;     // may be null: number of requests scored
};

// Alg. 1's two selections over a share of the instances.
struct DirectPart {
    uint32_t any_T, any_g;      // least latency (as an integer of the same order) and its instance; all ones: none
    uint32_t d_hi, d_lo;        // d_g of the feasible choice as an integer that falls with d_g; all ones: none
    uint32_t g, T;              // the feasible choice and its latency
};

// Feedback routing: the sums behind an instance's table as it was built last.
struct FeedBase {
    double ctx, q_ctx;      // of all contexts, of those that are prefilled first
    int n, listed, room;    // entries; requests of its list among them; the most of those that there is room for
    int pad;
};

__host__ __device__ constexpr int feed_groups(int n_inst) { return (n_inst + 3) / 4; }

// Words that the workgroups of a feedback routing in one launch leave for each other (see k_feedback_rounds).
struct FeedWords {
    unsigned long long *least = nullptr, *own = nullptr;   // [2][feed_groups][kWave], [2][M][4]; behind them as many for a part of the workgroups
    uint32_t *gate = nullptr, *team = nullptr;             // workgroups that have started, and at the end how many shared the work
    int n = 0;                                             // all of them, in words of 8 bytes, from `least` on
    __host__ __device__ FeedWords of(bool part, int n_inst) const
    {
        FeedWords w = *this;
        if (part) { w.least += set(n_inst); w.own += set(n_inst); }
        return w;
    }
    __host__ __device__ static constexpr int set(int n_inst) { return 2 * feed_groups(n_inst) * kWave + 2 * n_inst * 4; }
};
// and where they put away what has come to an instance since its table was built, 32 requests at a time
struct FeedBlocks {
    double2* yx = nullptr;     // [M][cap] sums of R, c*R + tri(R) up to each of the 32, in order of length
    double* c = nullptr;       // [M][cap] of contexts
    uint16_t* R = nullptr;     // [M][cap] the lengths
};

enum KernelId {
    kBuild = 0, kRank, kMarkRoute, kScanRoute, kMemoRoute, kClassRoute, kLinesRoute, kSelectRoute,
    kScanMigrate, kMemoMigrate, kClassMigrate, kLinesMigrate, kSelectMigrate, kHitsRoute, kPairsRoute, kDirect, kDirectMerge, kFeedback,
    kNumKernels
};

struct Profiler {
    bool on = false;
    uint64_t mask = ~0ull;           // bit k: launches of kernel id k are timed
    std::vector<hipEvent_t> events;  // pairs: start, stop
    std::vector<int> ids;            // kernel id of each recorded pair
};

struct StatusIn {
    const int *act_off, *act_prompt, *act_gen, *act_rem;
    const int *q_off, *q_prompt, *q_len;
    const float* act_budget;  // null unless flags are wanted
    int64_t n_active, n_queued;
    float *out_act_finish, *out_q_finish;
    double* out_d;
    int* out_rank;
    uint8_t* out_flag;
    int mark = 0;             // with flags: leave the lengths of flagged requests for the table pass
    int use_pending = 0;      // count the requests routed since the caller's status (feedback routing)
    int only_touched = 0;     // rebuild only the instances that have been given requests since the last build
    // a chunk just decided, to be taken into the lists by the build (see BuildArgs); 0: none
    int chunk_n = 0;
    const int *chunk_inst = nullptr, *chunk_ctx0 = nullptr, *chunk_len = nullptr;
};

// What is known of the instance tables at a call.
struct TableView {
    bool current = false;    // every instance's table is from the last inputs, blend weight and caps
    bool ordered = false;    // the class order belongs to the d_g (else the next scoring pass makes it)
    bool blended = false;    // the tables may hold a blend with the smoothed status
};

}  // namespace gr

struct gr_fleet {
    gr::Profiler prof;
    int n_inst = 0, n_class = 0, max_entries = 0, max_len = 0;
    int64_t max_requests = 0;
    int64_t max_active = 0;
    int64_t req_cap = 0;   // requests one scoring pass may hold
    int epl = 0;           // sort words per lane of the status build: 1, 2, 4 .. 32
    int cap = 0;           // 64 * epl >= max_entries: table entries per instance
    int n_split = 0;       // splitters per instance: 8 (cap 64), 16 (to 512), 32
    int m_pad = 0;         // instances rounded up to a multiple of 128, for the size of a small batch (gr_set_small_batch_pairs)
    int m_pos = 0;         // positions of the class order: every class rounded up to whole runs of kMemoP
    int n_run = 0;         // m_pos / kMemoP
    int run_pad = 0;       // n_run rounded up to whole runs of kMemoP: row length of grp_min
    int class_shift = 0;   // n_class rounded up to 2, 4, 8 or 16, as a power of two: row length of class_least
    int bins = 0;          // max_len + 1
    int most_of_class = 0; // instances of the largest class
    int64_t row_cap = 0;   // rows of the memo table, rounded up to whole blocks of kMemoU
    int device = 0;
    bool has_status = false;
    // smoothed black-box status (Sec. 3.3) and the weight it is blended in with
    double lam = 0.0;        // as set; takes effect at the next status build
    bool have_q = false, have_p = false, have_d = false;
    double *emaQ = nullptr, *emaP = nullptr, *emaD = nullptr;   // [M] each
    // device memory: fleet description
    gr::ClassCoef* cls = nullptr;
    int* inst_class = nullptr;
    // per-instance tables written by the status build
    // E_g(L) = Gq + L*H + tri(L)*gamma*(n+1) on the segment after the k shortest requests (n still running)
    uint16_t* tabR = nullptr; // [M][cap] remaining lengths, ascending; 0xFFFF past the last entry (and room for a wave's reads behind it)
    float2* tabGH = nullptr;  // [M][cap + 2] (Gq, H) of segment k, see gh_at (and room for a wave's reads behind it); segment 0 is (q_g, alpha + beta*(N+1) + gamma*sum of contexts)
    double* hD = nullptr;    // [M] d_g
    // [M] what a pair needs of its instance besides the tables: (delta, gamma) of the latency's prefill
    // part T = E + c0 * (delta + gamma * L), blended as the tables are; the curvature gamma of E; entries (int bits, see entries_of)
    float4* instK = nullptr;
    uint16_t* tabS = nullptr; // [M][n_split] every (cap / n_split)-th of the sorted lengths: the first step of a search
    // Class order: the instances class by class, every class padded to whole runs of kMemoP positions,
    // inside a class in capability order (largest d_g first, equal d_g by index).  Without a blend the
    // instances of a run then share the prefill part of T(r, g), and which of them is least or
    // feasible depends on E alone.
    float2* clsK = nullptr;       // [n_class] (delta, gamma) as single precision
    int* slot_inst = nullptr;     // [m_pos] the instances class by class in index order, -1: padding
    int* slot_of = nullptr;       // [M] slot of each instance
    unsigned long long* slot_key = nullptr;   // [m_pos] d_g of each slot's instance as an integer that falls with it
    int2* run_cls = nullptr;      // [n_run] first position of the run's class, instances of the class
    int2* cls_run = nullptr;      // [n_class] first run of the class, runs of the class
    int* order = nullptr;         // [m_pos] instance at each position, -1: padding
    int* pos_of = nullptr;        // [M] position of each instance
    float2* posK = nullptr;       // [m_pos] (delta, gamma) of the instance at each position
    unsigned long long* posKey = nullptr;   // [m_pos] d_g as an integer that falls with it
    uint4* run_head = nullptr;    // [n_run] the first position of each run: its key (low, high word), instance
    int* act_inst = nullptr; // [max_active] instance of each active request
    // feedback routing: the caller's last status inputs, and the requests routed since, per instance
    gr::StatusIn last_in{};
    int* pend_cnt = nullptr;      // [M]
    int* commit_mark = nullptr;   // [M] 1: chosen by a request of the chunk being committed (all zero between commits)
    int* pend_prompt = nullptr;   // [M][cap]
    int* pend_len = nullptr;      // [M][cap]
    float* scratch_finish = nullptr;  // [max_active + kBlock * kRestItems] finish times of rebuilds nobody asked to see
    int* batch_cap = nullptr;     // [M] requests that may decode together on each instance
    bool has_cap = false;
    int* counters = nullptr; // [2] GR_DEV_* bits, FeedWords::team
    // scoring workspace
    uint8_t* seen = nullptr;  // [bins, to 16] 1: some request of the batch has the length; all zero between calls
    int* late_cnt = nullptr;  // [4][M] flagged requests, counted by the build (late_parts counts per instance)
    int late_parts = 0;
    int* row_len = nullptr;   // [row_cap] the distinct lengths ("rows"), ascending
    uint16_t* len_row = nullptr;  // [bins + 1] rows shorter than each length = its row if it has one; 0xFFFF (past every row) at the end
    int* dense_totals = nullptr;   // [2] -, bins: the rows of a table that has one for every length
    int* totals = nullptr;    // [4] -, distinct lengths, 1: flags that the risk scan's build has not set (zero between calls)
    float* memo = nullptr;       // [row_cap / kMemoU][n_run][kMemoU][kMemoP] E per distinct length and position
    float* grp_min = nullptr;    // [row_cap][run_pad] least E of each run, per row (see runs_at)
    float* row_min = nullptr;    // [row_cap][run_pad] (behind grp_min) the same row by row, of a routing batch whose classes are looked at first; null where none can be
    uint32_t* run_rank = nullptr;   // [n_run] runs whose first instance is more capable than the run's first
    int* run_at = nullptr;          // [n_run] the run of each rank
    uint32_t* pos_thr = nullptr;    // [m_pos] runs whose first instance is more capable than the position's
    float4* run_k = nullptr;     // [n_run] least delta of the run, gamma, largest delta, lowest instance (int bits)
    uint32_t* cls_rank = nullptr;   // [n_class] run_rank of each class's first run
    float4* lines = nullptr;     // [row_cap][kRanges][2] with a blend: the instances that can have the least latency, see k_lines
    int* rest_cnt = nullptr;     // [kRestParts][kRestStride] length of each list (the lists themselves: scratch_finish)
    float* turned = nullptr;     // [turned_rows][M] a part of memo with a row's values together, for out_T
    int turned_rows = 0;         // multiple of kMemoU
    uint2* class_least = nullptr; // [bins][1 << class_shift] by length: least E of each class (bits), the instance that has it and how near the next is; null on more than 16 classes
    // What the host knows of the tables.  A call that is being recorded runs nothing, and what it records
    // changes the tables at every replay without the host: calls of a capture keep an account of their
    // own (`rec`, of capture `rec_id`), and once one of them may change the tables, or what they are made
    // from, the direct calls no longer rely on theirs (`recorded`; `blend_recorded`: one with a blend).
    gr::TableView now, rec;
    unsigned long long rec_id = ~0ull;
    bool recorded = false, blend_recorded = false;
    int* pend_touched = nullptr;   // [M] 1: given requests since its table was built
    int64_t small_batch_pairs = -1;   // largest batch, in pairs, scored pair by pair; -1: by the sizes (see pair_by_pair)
    // feedback routing, a launch a round or one for all (null on fleets of more than kFeedInst instances, and where one wave takes an instance), two of each in turn: what
    // every instance offers the requests of a chunk
    char* feed_parts = nullptr;             // (all of this)
    uint32_t* feed_T = nullptr;             // [2][M][kWave] latency as an integer of the same order; all ones: not allowed
    unsigned long long* feed_met = nullptr; // [2][M] bit j: request j's deadline is met
    unsigned long long* feed_key = nullptr; // [2][M] d_g as an integer that falls with it
    // the sums behind the tables (Y_k, X_k and the contexts of the k shortest), by segment, and those of whole instances
    double2* feed_yx = nullptr;             // [M][cap + 1]
    double* feed_c = nullptr;               // [M][cap + 1]
    gr::FeedBase* feed_base = nullptr;      // [M]
    gr::FeedWords feed_words;
    gr::FeedBlocks feed_blocks;
    int feed_polls = 64, feed_team = INT32_MAX;   // see gr_set_feedback_wait, gr_set_feedback_team
    int feed_per_unit = 0;                  // workgroups of k_feedback_rounds that a compute unit runs at once
    int units = 0, feed_units = INT32_MAX;  // compute units of the device; see gr_set_feedback_units
    gr::DirectPart* direct_part = nullptr;       // [kDirectParts] selections of the parts of a wide fleet, scored pair by pair
};

namespace gr {

// Brackets one kernel launch with a pair of events when timing is switched on.
struct ProfScope {
    Profiler& p;
    hipStream_t s;
    size_t slot = SIZE_MAX;
    ProfScope(gr_fleet* f, int id, hipStream_t stream) : p(f->prof), s(stream)
    {
        if (!p.on || !((p.mask >> id) & 1ull) || (p.ids.size() + 1) * 2 > p.events.size()) return;
        slot = p.ids.size();
        p.ids.push_back(id);
        (void)hipEventRecord(p.events[2 * slot], s);
    }
    ~ProfScope()
    {
        if (slot != SIZE_MAX) (void)hipEventRecord(p.events[2 * slot + 1], s);
    }
};


// The account of the tables that a call on stream `s` reads and keeps up to date (see gr_fleet).
struct TableAccount {
    bool ok = true;          // false: the stream may not be asked (a default stream next to a capture)
    bool capturing = false;
    TableView* v;

    TableAccount(gr_fleet* f, hipStream_t s) : v(&f->now)
    {
        hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
        unsigned long long id = 0;
        ok = hipStreamGetCaptureInfo(s, &status, &id) == hipSuccess;
        if (!ok) { (void)hipGetLastError(); return; }
        capturing = status != hipStreamCaptureStatusNone;
        if (!capturing) return;
        if (f->rec_id != id) { f->rec_id = id; f->rec = view(f); }
        v = &f->rec;
    }

    // what may be relied upon
    TableView view(const gr_fleet* f) const
    {
        if (v == &f->rec) return {v->current, false, v->blended};      // (replayed after whatever: the order is made)
        return {v->current && !f->recorded, v->ordered && !f->recorded, v->blended || f->blend_recorded};
    }
};

// What the class order needs (see gr_fleet).
struct OrderArgs {
    const unsigned long long* key;    // [m_pos] d_g as an integer that falls with it, by slot
    const float4* instK;    // [M] see gr_fleet
    const int* slot_inst;
    const int2* run_cls;
    int *order, *pos_of;
    float2* posK;
    unsigned long long* posKey;
    uint4* run_head;
    int m_pos;
};

// status.hip
int status_prepare();
int feedback_prepare(gr_fleet* f);
int launch_ranks(gr_fleet* f, int* out_rank, hipStream_t s);
int launch_status(gr_fleet* f, const StatusIn& in, hipStream_t s);
// A whole feedback routing in chunks of up to kWave requests, a launch a round (see k_feedback) or one for all (k_feedback_rounds).  `in`: the status inputs to
// rebuild from; `current`: instances that are given nothing keep their tables.
struct FeedbackIn {
    int64_t n;
    int chunk;
    const int *ctx0, *pred_len, *exclude;
    const float* budget;
    int* out_inst;
    float* out_slack;
    uint8_t* out_fallback;
    bool current;
};
// Waves that share an instance of a fleet of M whose tables take epl sort words per lane of one wave (without caps):
// fewer instances than the chip takes waves at four per SIMD, several waves per instance (measured on 1 024
// instances x 1 000 requests: 19.8 us with one wave each, 17.7 with two, 16.0 with four, 18.0 with eight, 29 with
// sixteen; on 256 x 512: 9.2, 8.5, 7.7-8.2, 8.1)
inline int waves_per_instance(int epl, int M)
{
    const int room = 4 * kSimds / M;
    return epl >= 4 && room >= 4 ? 4 : epl >= 2 && room >= 2 ? 2 : 1;
}

bool feedback_by_round(const gr_fleet* f, int64_t chunk);
int launch_feedback(gr_fleet* f, const StatusIn& in, const FeedbackIn& r, hipStream_t s);
int launch_commit(gr_fleet* f, int64_t n, const int* inst, const int* ctx0, const int* pred_len, hipStream_t s);
int launch_ema(gr_fleet* f, double w, const float* s_q, const float* s_p, const float* s_d, hipStream_t s);

// score.hip
int launch_score(gr_fleet* f, const ReqSrc& src, bool migrate, const ScoreOut& out, hipStream_t s,
                 bool small_batch_ok = false);
bool classes_first(const gr_fleet* f, bool migrate, int64_t n);
bool needs_marks(const gr_fleet* f, int64_t n);      // a risk scan's table pass makes a list of lengths
bool pair_by_pair(const gr_fleet* f, int64_t n);
int launch_direct(gr_fleet* f, const ReqSrc& src, const ScoreOut& out, hipStream_t s);
int launch_hits(gr_fleet* f, const ReqSrc& src, const int* hit_off, const int* hit_inst, const int* hit_len,
                int64_t n_hits, const ScoreOut& out, hipStream_t s);

// ------------------------------------------------------------------ wave helpers
// A launch's arguments come from memory, a line of 64 bytes at a time, and what the compiler reads where it is first
// used is waited for there.  This has all of a kernel's lines on their way together, at its start: for kernels that are a
// chain of reads.  Whole calls, us, without it in the one kernel / with it:
//   feedback routing  33 launches of 64 requests 333.5 / 307.3, 101 launches of one 766 / 665
//   builds            status of 256 x 512 9.1 / 8.75, 1 024 x 1 000 16.1 / 15.9, 1 024 x 200 and 40 queued under caps 32.6 / 31.8
//                     (eight words a lane and two or four waves spill two to four registers for it, 12 to 20 bytes a
//                     lane, and gain all the same: 600 x 1 500 19.4 / 18.9, 1 024 x 2 000 24.2 / 23.9, 2 000 x 1 000 22.65 / 22.7)
//   table             a row per length: step of 256 x 512 with 65 536 requests 45.0 / 44.6; with a list it loses (scan of 4 096 x 512
//                     109.0 / 110.8), as the selections by class do
//   pair by pair      64 instances x 12 000 requests 9.3 / 9.15, 16 x 40 000 7.2 / 7.05, 1 024 x 500 11.0 / 11.1
//   k_select          1 024 instances x 8 000 18.6 / 18.3, x 100 000 29.9 / 29.6, 4 096 x 400 20.8 / 20.7
// No difference in k_select_lanes (that step 45.6 / 45.5), k_scan and k_hits, which do without.
template <typename Args>
__device__ __forceinline__ void fetch_args()
{
    const auto* p = (const __attribute__((address_space(4))) uint32_t*)__builtin_amdgcn_kernarg_segment_ptr();
    uint32_t x = 0;
#pragma unroll
    for (unsigned i = 0; i < sizeof(Args); i += 64) x |= p[i / 4];
    asm volatile("" :: "s"(x));
}

__device__ inline int lane_id() { return threadIdx.x & (kWave - 1); }

template <typename T>
__device__ inline T wave_sum(T v)
{
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) v += __shfl_xor(v, d, kWave);
    return v;
}

// Inclusive prefix sum of a 32-bit value over the wave without going through
// LDS: inside each row of 16 lanes by shifts of 1, 2, 4, 8 (a lane without a
// source adds 0), then lane 15 of rows 0 and 2 onto rows 1 and 3, then lane 31
// onto rows 2 and 3.
__device__ inline int wave_incl_scan_i32(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2, 3
    return v;
}

template <int kCtrl, int kRowMask>
__device__ inline uint32_t min_dpp(uint32_t v)      // (all ones where the lane has no source)
{
    return min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, kCtrl, kRowMask, 0xf, false));
}

// The least value over the wave, or over the lane's row of 16 (kRow), for every lane.
template <bool kRow>
__device__ inline uint32_t min_over(uint32_t v)
{
    if constexpr (kRow) {
        v = min_dpp<0x128, 0xf>(v);      // row_ror 8, 4, 2, 1
        v = min_dpp<0x124, 0xf>(v);
        v = min_dpp<0x122, 0xf>(v);
        return min_dpp<0x121, 0xf>(v);
    } else {
        v = min_dpp<0x111, 0xf>(v);      // row_shr 1, 2, 4, 8
        v = min_dpp<0x112, 0xf>(v);
        v = min_dpp<0x114, 0xf>(v);
        v = min_dpp<0x118, 0xf>(v);
        v = min_dpp<0x142, 0xa>(v);      // row_bcast 15 into rows 1 and 3, 31 into rows 2 and 3
        v = min_dpp<0x143, 0xc>(v);
        return (uint32_t)__builtin_amdgcn_readlane((int)v, kWave - 1);
    }
}

// a double as an unsigned integer of the opposite order (both zeros alike, NaNs have a place too)
__device__ inline unsigned long long falling_bits(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v + 0.0);
    return ~(b ^ ((b >> 63) ? ~0ull : 0x8000000000000000ull));
}

// Of the eight 16-bit lengths in `w` those that are at most L (up to 32 767), in two counts of 16 bits: a saturating
// difference from L + 1, cut to one, for two lengths at a time (12 instructions; compared one by one 20).
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

__device__ inline uint32_t count_upto2(const uint4& w, uint32_t L)
{
    const u16x2 one = {1, 1}, next = __builtin_bit_cast(u16x2, (L + 1) * 0x10001u);
    u16x2 c = {0, 0};
    for (const uint32_t x : {w.x, w.y, w.z, w.w})
        c += __builtin_elementwise_min(__builtin_elementwise_sub_sat(next, __builtin_bit_cast(u16x2, x)), one);
    return __builtin_bit_cast(uint32_t, c);
}

__device__ inline int both_counts(uint32_t c) { return (int)((c & 0xFFFFu) + (c >> 16)); }

__device__ inline int count_upto(const uint4& w, uint32_t L) { return both_counts(count_upto2(w, L)); }

// a float as an unsigned integer of the same order
__device__ inline uint32_t ordered_bits(float v)
{
    const uint32_t b = __float_as_uint(v);
    return b ^ ((b >> 31) ? 0xFFFFFFFFu : 0x80000000u);
}

__device__ inline float from_ordered_bits(uint32_t u)
{
    return __uint_as_float(u ^ ((u >> 31) ? 0x80000000u : 0xFFFFFFFFu));
}

__device__ inline int entries_of(const float4& K) { return __float_as_int(K.w) & ~kAllAlike; }
__device__ inline bool all_alike(const float4& K) { return (__float_as_int(K.w) & kAllAlike) != 0; }

// kappa = delta + gamma * L, the same instruction wherever a pair's latency is formed
__device__ inline float kappa_of(float2 dg, float Lf) { return fmaf(dg.y, Lf, dg.x); }

__device__ inline DirectPart no_selection() { return DirectPart{~0u, ~0u, ~0u, ~0u, ~0u, ~0u}; }

__device__ inline void take_better(DirectPart& b, const DirectPart& o)
{
    // (values, not references: a choice between two structs' members keeps both in memory)
    const uint32_t oT = o.any_T, og = o.any_g, oh = o.d_hi, ol = o.d_lo, ofg = o.g, ofT = o.T;
    const uint32_t bT = b.any_T, bg = b.any_g, bh = b.d_hi, bl = b.d_lo, bfg = b.g, bfT = b.T;
    const bool less = oT < bT || (oT == bT && og < bg);
    const bool better = oh < bh || (oh == bh && (ol < bl || (ol == bl && ofg < bfg)));
    b = DirectPart{less ? oT : bT, less ? og : bg, better ? oh : bh, better ? ol : bl, better ? ofg : bfg, better ? ofT : bfT};
}

constexpr int kRankPer = 8;      // instances that kRankWaves waves rank together
constexpr int kRankWaves = 4;
static_assert(kMemoP % kRankPer == 0, "the instances ranked together are of one class");

// Workgroup `wg` of kThreads threads of the class order: the ranks of kThreads / 256 runs of kRankPer
// instances among those of their class,
//   rank_g = #{h : d_h > d_g} + #{h < g : d_h = d_g},
// which place each instance behind its class's first position.  Four waves share the instances
// and split the competitors, a lane per competitor, each lane with its own counts, added up over the
// wave and then through LDS.  The time is that of the reads (the status build has just written d, so
// each XCD fetches it from memory): a wave reads its share of the competitors in one batch.
// Every thread of the workgroup must call it.  `sums`: kThreads / 64 * kRankPer ints of LDS.
template <int kThreads>
__device__ inline void order_block(const OrderArgs& a, int wg, int* sums)
{
    constexpr int kRuns = kThreads / (kRankWaves * kWave);
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int quarter = wave % kRankWaves, s0 = (wg * kRuns + wave / kRankWaves) * kRankPer;
    const int s = s0 + lane;
    int first = 0, cnt = 0, g = -1;
    float4 k{};
    unsigned long long own = 0;
    if (s0 < a.m_pos) {
        const int2 rc = a.run_cls[s0 / kMemoP];
        first = rc.x; cnt = rc.y;
        if (quarter == 0 && lane < kRankPer && s < first + cnt) { g = a.slot_inst[s]; k = a.instK[g]; own = a.key[s]; }
        unsigned long long dg[kRankPer];
        int r[kRankPer] = {};
#pragma unroll
        for (int j = 0; j < kRankPer; ++j) dg[j] = a.key[s0 + j];
        constexpr int kAhead = 8;
        const int per = ((cnt + kRankWaves - 1) / kRankWaves + kWave - 1) / kWave * kWave;
        const int h_end = min((quarter + 1) * per, cnt), mine = s0 - first;
        for (int h0 = quarter * per; h0 < h_end; h0 += kAhead * kWave) {
            unsigned long long dh[kAhead];
#pragma unroll
            for (int k = 0; k < kAhead; ++k) dh[k] = a.key[first + min(h0 + k * kWave + lane, h_end - 1)];
#pragma unroll
            for (int k = 0; k < kAhead; ++k) {
                const int h = h0 + k * kWave + lane;
#pragma unroll
                for (int j = 0; j < kRankPer; ++j)
                    r[j] += h < h_end && (dh[k] < dg[j] || (dh[k] == dg[j] && h < mine + j));
            }
        }
#pragma unroll
        for (int j = 0; j < kRankPer; ++j) {
            const int all = wave_incl_scan_i32(r[j]);
            if (lane == kWave - 1) sums[wave * kRankPer + j] = all;
        }
    }
    __syncthreads();
    if (quarter != 0 || lane >= kRankPer || s >= a.m_pos) return;
    if (s < first + cnt) {
        int p = first;
#pragma unroll
        for (int q = 0; q < kRankWaves; ++q) p += sums[(wave + q) * kRankPer + lane];
        a.pos_of[g] = p;
        a.order[p] = g;
        a.posK[p] = make_float2(k.x, k.y);
        a.posKey[p] = own;
        if (p % kMemoP == 0) a.run_head[p / kMemoP] = make_uint4((uint32_t)own, (uint32_t)(own >> 32), (uint32_t)g, 0u);
    } else {
        a.order[s] = -1;     // positions past the last instance of the class
        a.posK[s] = make_float2(__builtin_inff(), 0.f);
        a.posKey[s] = ~0ull;
    }
}

// Workgroups of kThreads threads that place every instance (and fill the padded positions).
constexpr int order_blocks(int m_pos, int threads)
{
    const int per = threads / (kRankWaves * kWave) * kRankPer;
    return (m_pos + per - 1) / per;
}

}  // namespace gr
