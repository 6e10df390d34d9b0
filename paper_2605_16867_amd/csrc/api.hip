// Host entry points of libgoodroute: the fleet handle, argument checks and the
// order in which the kernels of status.hip and score.hip are queued.
#include <algorithm>
#include <new>
#include <type_traits>

#include "common.h"

namespace gr {
namespace {

const char* const kKernelNames[kNumKernels] = {
    "k_build", "k_rank",
    "k_mark<route>", "k_scan<route>", "k_memo<route>", "k_class<route>", "k_lines<route>", "k_select<route>",
    "k_scan<migrate>", "k_memo<migrate>", "k_class<migrate>", "k_lines<migrate>", "k_select<migrate>",
    "k_hits<route>", "k_pairs<route>", "k_direct", "k_direct_merge", "k_feedback"};

template <typename T>
bool dev_alloc(T** p, size_t n)
{
    return hipMalloc(reinterpret_cast<void**>(p), (n ? n : 1) * sizeof(T)) == hipSuccess;
}

// The fleet as the kernels read it: coefficients, classes, and the instances class by class, every
// class padded to whole runs of kMemoP positions (see gr_fleet).
struct FleetTables {
    std::vector<ClassCoef> coef;
    std::vector<float2> coef32;
    std::vector<int2> cls_run, run_cls;
    std::vector<int> slot, slot_of;
};

bool make_tables(FleetTables& t, int n_inst, int n_class, const double* delta, const double* alpha, const double* beta,
                 const double* gamma, const int32_t* inst_class) noexcept
{
    try {
        std::vector<int> per_class(n_class, 0), next(n_class), by_step(n_class);
        for (int g = 0; g < n_inst; ++g) ++per_class[inst_class[g]];
        for (int c = 0; c < n_class; ++c) {
            t.coef.push_back(ClassCoef{delta[c], alpha[c], beta[c], gamma[c]});
            t.coef32.push_back(make_float2((float)delta[c], (float)gamma[c]));
            by_step[c] = c;
        }
        // classes of slow steps first: their instances are the just-enough choices, and a search that
        // meets them first passes over most of the others (any order gives the same answers)
        std::stable_sort(by_step.begin(), by_step.end(), [&](int x, int y) { return alpha[x] > alpha[y]; });
        t.cls_run.resize(n_class);
        for (const int c : by_step) {
            const int run = (int)t.run_cls.size(), runs = (per_class[c] + kMemoP - 1) / kMemoP;
            t.cls_run[c] = make_int2(run, runs);
            t.run_cls.insert(t.run_cls.end(), runs, make_int2(run * kMemoP, per_class[c]));
            next[c] = run * kMemoP;
        }
        t.slot.assign(t.run_cls.size() * kMemoP, -1);
        t.slot_of.resize(n_inst);
        for (int g = 0; g < n_inst; ++g) {
            t.slot_of[g] = next[inst_class[g]]++;
            t.slot[t.slot_of[g]] = g;
        }
        return true;
    } catch (...) {
        return false;
    }
}

bool status_args_ok(const gr_fleet* f, const int32_t* act_off, const int32_t* act_prompt,
                    const int32_t* act_gen, const int32_t* act_rem, int64_t n_active,
                    const int32_t* q_off, const int32_t* q_prompt, const int32_t* q_len, int64_t n_queued,
                    int* rc)
{
    *rc = GR_ERR_INVALID_ARG;
    if (!f || !act_off || !q_off || n_active < 0 || n_queued < 0) return false;
    if (n_active > 0 && (!act_prompt || !act_gen || !act_rem)) return false;
    if (n_queued > 0 && (!q_prompt || !q_len)) return false;
    *rc = GR_ERR_TOO_LARGE;
    if (n_active > f->max_active || n_queued > f->max_active) return false;
    *rc = GR_OK;
    return true;
}

}  // namespace
}  // namespace gr

using namespace gr;

extern "C" {

int gr_create(gr_fleet** out, int32_t n_inst, int32_t n_class,
              const double* delta, const double* alpha, const double* beta, const double* gamma,
              const int32_t* inst_class, int32_t max_entries_per_inst, int32_t max_len,
              int64_t max_requests)
{
    if (!out) return GR_ERR_INVALID_ARG;
    *out = nullptr;
    if (n_inst <= 0 || n_class <= 0 || !delta || !alpha || !beta || !gamma || !inst_class ||
        max_entries_per_inst < 0 || max_len < 1 || max_requests < 0)
        return GR_ERR_INVALID_ARG;
    if (n_class > kMaxClasses || max_entries_per_inst > kMaxEntries || max_len > kMaxLen ||
        max_requests > (int64_t(1) << 30) || n_inst > (1 << 20))
        return GR_ERR_TOO_LARGE;
    for (int c = 0; c < n_class; ++c)
        if (!(delta[c] >= 0) || !(alpha[c] >= 0) || !(beta[c] >= 0) || !(gamma[c] >= 0))
            return GR_ERR_INVALID_ARG;
    for (int g = 0; g < n_inst; ++g)
        if (inst_class[g] < 0 || inst_class[g] >= n_class) return GR_ERR_INVALID_ARG;
    if ((int64_t)n_inst * max_entries_per_inst > (int64_t(1) << 30)) return GR_ERR_TOO_LARGE;

    FleetTables tab_h;
    if (!make_tables(tab_h, n_inst, n_class, delta, alpha, beta, gamma, inst_class)) return GR_ERR_NOMEM;
    gr_fleet* f = new (std::nothrow) gr_fleet;
    if (!f) return GR_ERR_NOMEM;
    f->n_inst = n_inst; f->n_class = n_class;
    f->max_entries = max_entries_per_inst; f->max_len = max_len; f->max_requests = max_requests;
    f->max_active = (int64_t)n_inst * max_entries_per_inst;
    f->req_cap = f->max_active > max_requests ? f->max_active : max_requests;
    f->epl = 1;
    while (kWave * f->epl < max_entries_per_inst) f->epl *= 2;
    f->cap = kWave * f->epl;
    f->n_split = split_count(f->cap);
    f->m_pad = ((n_inst + 2 * kWave - 1) / (2 * kWave)) * (2 * kWave);
    f->n_run = (int)tab_h.run_cls.size();
    f->m_pos = f->n_run * kMemoP;
    f->run_pad = (f->n_run + kMemoP - 1) / kMemoP * kMemoP;
    f->class_shift = 1;
    while ((1 << f->class_shift) < n_class) ++f->class_shift;
    f->bins = max_len + 1;
    for (const int2 r : tab_h.run_cls) f->most_of_class = std::max(f->most_of_class, r.y);
    f->row_cap = f->req_cap < f->bins ? f->req_cap : f->bins;
    f->row_cap = (f->row_cap + kMemoU - 1) / kMemoU * kMemoU;
    if (f->row_cap < kMemoU) f->row_cap = kMemoU;
    f->turned_rows = (int)std::min<int64_t>(f->row_cap, std::max<int64_t>(kTurnedBytes / ((int64_t)n_inst * 4 * kMemoU), 1) * kMemoU);
    if (hipGetDevice(&f->device) != hipSuccess) { delete f; return GR_ERR_HIP; }

    const size_t tab = (size_t)n_inst * f->cap, segments = (size_t)n_inst * (f->cap + 1), seen_bytes = (size_t)(f->bins + 15) / 16 * 16;
    const bool by_row = classes_first(f, false, max_requests), by_round = n_inst <= kFeedInst && waves_per_instance(f->epl, n_inst) > 1;
    const size_t words = 2 * (size_t)FeedWords::set(n_inst) + 1;
    // (parts of one allocation: each takes its time, 8 us)
    const auto feedback_parts = [&](auto part) {
        part(&f->feed_base, (size_t)n_inst);
        part(&f->feed_yx, segments); part(&f->feed_c, segments);
        part(&f->feed_blocks.yx, tab); part(&f->feed_blocks.c, tab); part(&f->feed_blocks.R, tab);
        part(&f->feed_words.least, words);
        part(&f->feed_T, (size_t)2 * n_inst * kWave); part(&f->feed_met, (size_t)2 * n_inst); part(&f->feed_key, (size_t)2 * n_inst);
    };
    const auto bytes_of = [](size_t each, size_t n) { return (each * n + 255) / 256 * 256; };
    size_t feed_bytes = 0;
    if (by_round) feedback_parts([&](auto** p, size_t n) { feed_bytes += bytes_of(sizeof **p, n); });
    const bool ok =
        dev_alloc(&f->cls, n_class) && dev_alloc(&f->inst_class, n_inst) &&
        dev_alloc(&f->tabR, tab + kWave) && dev_alloc(&f->tabGH, (size_t)n_inst * (f->cap + 2) + kWave) &&
        dev_alloc(&f->hD, n_inst) &&
        dev_alloc(&f->emaQ, n_inst) && dev_alloc(&f->emaP, n_inst) && dev_alloc(&f->emaD, n_inst) &&
        dev_alloc(&f->instK, n_inst) && dev_alloc(&f->tabS, (size_t)n_inst * f->n_split) &&
        dev_alloc(&f->clsK, n_class) && dev_alloc(&f->slot_inst, f->m_pos) && dev_alloc(&f->slot_of, n_inst) && dev_alloc(&f->slot_key, f->m_pos) && dev_alloc(&f->run_cls, f->n_run) && dev_alloc(&f->cls_run, n_class) &&
        dev_alloc(&f->order, f->m_pos) && dev_alloc(&f->pos_of, n_inst) && dev_alloc(&f->posK, f->m_pos) && dev_alloc(&f->posKey, f->m_pos) && dev_alloc(&f->run_head, f->n_run) &&
        dev_alloc(&f->act_inst, f->max_active) && dev_alloc(&f->counters, 2) &&
        dev_alloc(&f->pend_cnt, n_inst) && dev_alloc(&f->commit_mark, n_inst) && dev_alloc(&f->pend_touched, n_inst) && dev_alloc(&f->pend_prompt, tab) && dev_alloc(&f->pend_len, tab) &&
        dev_alloc(&f->scratch_finish, f->max_active + kBlock * kRestItems) && dev_alloc(&f->batch_cap, n_inst) &&
        dev_alloc(&f->seen, seen_bytes) && dev_alloc(&f->late_cnt, (size_t)n_inst * 4) &&
        dev_alloc(&f->row_len, f->row_cap) && dev_alloc(&f->len_row, f->bins + 1) && dev_alloc(&f->totals, 4) && dev_alloc(&f->dense_totals, 2) &&
        dev_alloc(&f->memo, (size_t)f->row_cap * f->m_pos) && dev_alloc(&f->grp_min, (size_t)f->row_cap * f->run_pad * (by_row ? 2 : 1)) &&
        dev_alloc(&f->run_k, f->n_run) && dev_alloc(&f->run_rank, f->n_run) && dev_alloc(&f->run_at, f->n_run) && dev_alloc(&f->pos_thr, f->m_pos) &&
        dev_alloc(&f->cls_rank, n_class) && (n_class > kMemoP || dev_alloc(&f->class_least, (size_t)f->bins << f->class_shift)) &&
        dev_alloc(&f->rest_cnt, kRestParts * kRestStride) && dev_alloc(&f->lines, (size_t)f->row_cap * kRanges * 2) && dev_alloc(&f->turned, (size_t)f->turned_rows * n_inst) && dev_alloc(&f->direct_part, (size_t)kDirectParts) &&
        (!by_round || dev_alloc(&f->feed_parts, feed_bytes));
    if (!ok) { gr_destroy(f); return GR_ERR_NOMEM; }
    if (by_row) f->row_min = f->grp_min + (size_t)f->row_cap * f->run_pad;
    if (by_round) {
        char* at = f->feed_parts;
        feedback_parts([&](auto** p, size_t n) {
            *p = reinterpret_cast<std::remove_reference_t<decltype(*p)>>(at);
            at += bytes_of(sizeof **p, n);
        });
        f->feed_words.own = f->feed_words.least + 2 * feed_groups(n_inst) * kWave;
        f->feed_words.gate = reinterpret_cast<uint32_t*>(f->feed_words.least + words - 1);
        f->feed_words.team = reinterpret_cast<uint32_t*>(f->counters + 1);
        f->feed_words.n = (int)words;
    }

    bool sent = true;
    const auto send = [&](void* to, const void* from, size_t bytes) {
        sent = sent && hipMemcpy(to, from, bytes, hipMemcpyHostToDevice) == hipSuccess;
    };
    const auto clear = [&](void* p, size_t bytes) { sent = sent && hipMemset(p, 0, bytes) == hipSuccess; };
    send(f->cls, tab_h.coef.data(), sizeof(ClassCoef) * n_class);
    send(f->clsK, tab_h.coef32.data(), sizeof(float2) * n_class);
    send(f->cls_run, tab_h.cls_run.data(), sizeof(int2) * n_class);
    send(f->run_cls, tab_h.run_cls.data(), sizeof(int2) * f->n_run);
    send(f->slot_inst, tab_h.slot.data(), sizeof(int) * f->m_pos);
    send(f->slot_of, tab_h.slot_of.data(), sizeof(int) * n_inst);
    const int dense[2] = {0, f->bins};
    send(f->dense_totals, dense, sizeof dense);
    send(f->inst_class, inst_class, sizeof(int) * n_inst);
    clear(f->counters, 2 * sizeof(int));
    clear(f->seen, seen_bytes);
    clear(f->slot_key, sizeof(unsigned long long) * f->m_pos);
    clear(f->totals, sizeof(int) * 4);
    // tables without an entry, as far as the reads go: a status build may be recorded first, and a direct call
    // come before its first replay
    sent = sent && hipMemset(f->tabR, 0xFF, (tab + kWave) * sizeof(uint16_t)) == hipSuccess &&
           hipMemset(f->len_row + f->bins, 0xFF, sizeof(uint16_t)) == hipSuccess &&
           hipMemset(f->tabS, 0xFF, (size_t)n_inst * f->n_split * sizeof(uint16_t)) == hipSuccess;
    clear(f->tabGH, ((size_t)n_inst * (f->cap + 2) + kWave) * sizeof(float2));
    clear(f->instK, sizeof(float4) * n_inst);
    clear(f->hD, sizeof(double) * n_inst);
    clear(f->pend_cnt, sizeof(int) * n_inst);
    clear(f->pend_touched, sizeof(int) * n_inst);
    clear(f->commit_mark, sizeof(int) * n_inst);
    if (!sent || hipDeviceSynchronize() != hipSuccess) {
        gr_destroy(f);
        return GR_ERR_HIP;
    }
    if (status_prepare() != GR_OK || (by_round && feedback_prepare(f) != GR_OK)) { gr_destroy(f); return GR_ERR_HIP; }
    *out = f;
    return GR_OK;
}

int gr_destroy(gr_fleet* f)
{
    if (!f) return GR_OK;
    (void)hipDeviceSynchronize();
    void* ptrs[] = {f->cls, f->inst_class, f->tabR, f->tabGH, f->hD, f->emaQ, f->emaP, f->emaD, f->instK, f->tabS,
                    f->clsK, f->slot_inst, f->slot_of, f->slot_key, f->run_cls, f->cls_run, f->order, f->pos_of, f->posK, f->posKey, f->run_head, f->act_inst, f->pend_cnt, f->commit_mark, f->pend_touched, f->pend_prompt, f->pend_len,
                    f->scratch_finish, f->batch_cap, f->counters, f->seen, f->late_cnt, f->row_len,
                    f->len_row, f->totals, f->dense_totals, f->memo, f->grp_min, f->run_k, f->run_rank, f->run_at, f->pos_thr, f->cls_rank, f->class_least, f->rest_cnt, f->lines, f->turned, f->feed_parts, f->direct_part};
    int rc = GR_OK;
    for (void* p : ptrs)
        if (p && hipFree(p) != hipSuccess) rc = GR_ERR_HIP;
    for (hipEvent_t e : f->prof.events) (void)hipEventDestroy(e);
    delete f;
    return rc;
}

int gr_build_status(gr_fleet* f, const int32_t* act_off, const int32_t* act_prompt,
                    const int32_t* act_gen, const int32_t* act_rem, int64_t n_active,
                    const int32_t* q_off, const int32_t* q_prompt, const int32_t* q_len,
                    int64_t n_queued, float* out_act_finish, float* out_q_finish,
                    double* out_d, int32_t* out_rank, void* hip_stream)
{
    int rc;
    if (!status_args_ok(f, act_off, act_prompt, act_gen, act_rem, n_active, q_off, q_prompt, q_len,
                        n_queued, &rc))
        return rc;
    if (n_active > 0 && !out_act_finish) return GR_ERR_INVALID_ARG;
    StatusIn in{};
    in.act_off = act_off; in.act_prompt = act_prompt; in.act_gen = act_gen; in.act_rem = act_rem;
    in.q_off = q_off; in.q_prompt = q_prompt; in.q_len = q_len;
    in.n_active = n_active; in.n_queued = n_queued;
    in.out_act_finish = out_act_finish; in.out_q_finish = out_q_finish;
    in.out_d = out_d; in.out_rank = out_rank;
    return launch_status(f, in, static_cast<hipStream_t>(hip_stream));
}

namespace {
// gr_score_route; `small_batch_ok`: a batch of a few requests may be scored pair by pair,
// which leaves no table of per-length values behind
int score_route(gr_fleet* f, int64_t n_req, const int32_t* ctx0, const int32_t* pred_len,
                const float* budget, const int32_t* exclude_inst, int32_t* out_inst,
                float* out_slack, uint8_t* out_fallback, float* out_T, void* hip_stream, bool small_batch_ok)
{
    if (!f || n_req < 0) return GR_ERR_INVALID_ARG;
    if (!f->has_status) return GR_ERR_NO_STATUS;
    if (n_req == 0) return GR_OK;
    if (!ctx0 || !pred_len || !budget || !out_inst || !out_slack) return GR_ERR_INVALID_ARG;
    if (n_req > f->max_requests) return GR_ERR_TOO_LARGE;
    ReqSrc src{};
    src.ctx0 = ctx0; src.pred_len = pred_len; src.budget = budget; src.exclude = exclude_inst;
    src.n = n_req;
    ScoreOut o{};
    o.inst = out_inst; o.slack = out_slack; o.fallback = out_fallback; o.T = out_T;
    return launch_score(f, src, false, o, static_cast<hipStream_t>(hip_stream), small_batch_ok);
}
}  // namespace

int gr_score_route(gr_fleet* f, int64_t n_req, const int32_t* ctx0, const int32_t* pred_len,
                   const float* budget, const int32_t* exclude_inst, int32_t* out_inst,
                   float* out_slack, uint8_t* out_fallback, float* out_T, void* hip_stream)
{
    return score_route(f, n_req, ctx0, pred_len, budget, exclude_inst, out_inst, out_slack, out_fallback, out_T,
                       hip_stream, true);
}

int gr_score_route_noalloc(gr_fleet* f, int64_t n_req, const int32_t* ctx0, const int32_t* pred_len,
                           const float* budget, const int32_t* exclude_inst, int32_t* out_inst,
                           float* out_slack, uint8_t* out_fallback, void* hip_stream)
{
    if (!f || n_req < 0) return GR_ERR_INVALID_ARG;
    if (n_req > GR_NOALLOC_MAX_REQUESTS) return GR_ERR_TOO_LARGE;
    if (!f->has_status) return GR_ERR_NO_STATUS;
    if (n_req == 0) return GR_OK;
    if (!ctx0 || !pred_len || !budget || !out_inst || !out_slack) return GR_ERR_INVALID_ARG;
    ReqSrc src{};
    src.ctx0 = ctx0; src.pred_len = pred_len; src.budget = budget; src.exclude = exclude_inst;
    src.n = n_req;
    ScoreOut o{};
    o.inst = out_inst; o.slack = out_slack; o.fallback = out_fallback;
    return launch_direct(f, src, o, static_cast<hipStream_t>(hip_stream));
}

int gr_score_route_cached(gr_fleet* f, int64_t n_req, const int32_t* ctx0, const int32_t* pred_len,
                          const float* budget, const int32_t* exclude_inst,
                          const int32_t* hit_off, const int32_t* hit_inst, const int32_t* hit_len,
                          int64_t n_hits, int32_t* out_inst, float* out_slack, uint8_t* out_fallback,
                          float* out_T, void* hip_stream)
{
    if (n_hits < 0 || (n_req > 0 && !hit_off) || (n_hits > 0 && (!hit_inst || !hit_len)))
        return GR_ERR_INVALID_ARG;
    // (the correction below reads the per-length table)
    const int rc = score_route(f, n_req, ctx0, pred_len, budget, exclude_inst, out_inst, out_slack,
                               out_fallback, out_T, hip_stream, false);
    if (rc != GR_OK || n_req == 0) return rc;
    ReqSrc src{};
    src.ctx0 = ctx0; src.pred_len = pred_len; src.budget = budget; src.exclude = exclude_inst;
    src.n = n_req;
    ScoreOut o{};
    o.inst = out_inst; o.slack = out_slack; o.fallback = out_fallback; o.T = out_T;
    return launch_hits(f, src, hit_off, hit_inst, hit_len, n_hits, o, static_cast<hipStream_t>(hip_stream));
}

int gr_route_feedback(gr_fleet* f, int64_t n_req, int64_t chunk, const int32_t* ctx0,
                      const int32_t* pred_len, const float* budget, const int32_t* exclude_inst,
                      int32_t* out_inst, float* out_slack, uint8_t* out_fallback, void* hip_stream)
{
    if (!f || n_req < 0 || chunk < 1) return GR_ERR_INVALID_ARG;
    if (!f->has_status) return GR_ERR_NO_STATUS;
    if (n_req == 0) return GR_OK;
    if (!ctx0 || !pred_len || !budget || !out_inst || !out_slack) return GR_ERR_INVALID_ARG;
    if (chunk > f->max_requests) chunk = f->max_requests;
    if (chunk < 1) return GR_ERR_TOO_LARGE;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    // rebuilds start from the caller's last status inputs; what they report goes to scratch
    StatusIn in = f->last_in;
    in.use_pending = 1;
    in.act_budget = nullptr; in.out_flag = nullptr;
    in.out_act_finish = f->scratch_finish; in.out_q_finish = nullptr; in.out_d = nullptr; in.out_rank = nullptr;
    // Instances that were given nothing keep their tables, unless those may be from an earlier blend
    // weight or earlier caps: then the first rebuild takes every instance.
    bool current = TableAccount(f, s).view(f).current;
    if (feedback_by_round(f, std::min(chunk, n_req))) {
        FeedbackIn r{};
        r.n = n_req; r.chunk = (int)std::min(chunk, n_req);
        r.ctx0 = ctx0; r.pred_len = pred_len; r.exclude = exclude_inst; r.budget = budget;
        r.out_inst = out_inst; r.out_slack = out_slack; r.out_fallback = out_fallback;
        r.current = current;
        return launch_feedback(f, in, r, s);
    }
    for (int64_t s0 = 0; s0 < n_req; s0 += chunk) {
        const int64_t n = n_req - s0 < chunk ? n_req - s0 : chunk;
        ReqSrc src{};
        src.ctx0 = ctx0 + s0; src.pred_len = pred_len + s0; src.budget = budget + s0;
        src.exclude = exclude_inst ? exclude_inst + s0 : nullptr;
        src.n = n;
        ScoreOut o{};
        o.inst = out_inst + s0; o.slack = out_slack + s0; o.fallback = out_fallback ? out_fallback + s0 : nullptr;
        int rc = launch_score(f, src, false, o, s, true);
        // the chunk's requests join the queues: in the build itself where a wave holds the chunk (the
        // build under caps is a kernel of its own and does not)
        const bool in_build = n <= kWave && !f->has_cap;
        in.chunk_n = in_build ? (int)n : 0;
        in.chunk_inst = out_inst + s0; in.chunk_ctx0 = ctx0 + s0; in.chunk_len = pred_len + s0;
        if (rc == GR_OK && !in_build) rc = launch_commit(f, n, out_inst + s0, ctx0 + s0, pred_len + s0, s);
        in.only_touched = current ? 1 : 0;
        if (rc == GR_OK) rc = launch_status(f, in, s);
        if (rc != GR_OK) return rc;
        current = true;
    }
    return GR_OK;
}

int gr_risk_scan(gr_fleet* f, const int32_t* act_off, const int32_t* act_prompt,
                 const int32_t* act_gen, const int32_t* act_rem_refreshed, int64_t n_active,
                 const int32_t* q_off, const int32_t* q_prompt, const int32_t* q_len,
                 int64_t n_queued, const float* act_budget, uint8_t* out_flag, float* out_finish,
                 int32_t* out_target, float* out_target_slack, int32_t* out_n_flagged,
                 void* hip_stream)
{
    int rc;
    if (!status_args_ok(f, act_off, act_prompt, act_gen, act_rem_refreshed, n_active, q_off, q_prompt,
                        q_len, n_queued, &rc))
        return rc;
    if (n_active > 0 && (!act_budget || !out_flag || !out_finish || !out_target || !out_target_slack))
        return GR_ERR_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    StatusIn in{};
    in.act_off = act_off; in.act_prompt = act_prompt; in.act_gen = act_gen; in.act_rem = act_rem_refreshed;
    in.q_off = q_off; in.q_prompt = q_prompt; in.q_len = q_len;
    in.act_budget = act_budget;
    in.n_active = n_active; in.n_queued = n_queued;
    in.out_act_finish = out_finish; in.out_flag = out_flag;
    in.mark = needs_marks(f, n_active);
    rc = launch_status(f, in, s);
    if (rc != GR_OK) return rc;
    ReqSrc src{};
    src.act_prompt = act_prompt; src.act_gen = act_gen; src.act_rem = act_rem_refreshed;
    src.act_inst = f->act_inst; src.flag = out_flag; src.act_budget = act_budget;
    src.act_off = act_off;
    src.n = n_active;
    ScoreOut o{};
    o.inst = out_target; o.slack = out_target_slack; o.n_selected = out_n_flagged;
    return launch_score(f, src, true, o, s, true);
}

int gr_observe(gr_fleet* f, double weight, const float* obs_wait, const float* obs_prefill,
               const float* obs_decode, void* hip_stream)
{
    if (!f || !(weight >= 0.0 && weight <= 1.0)) return GR_ERR_INVALID_ARG;
    if (!obs_wait && !obs_prefill && !obs_decode) return GR_OK;
    const TableAccount account(f, static_cast<hipStream_t>(hip_stream));
    account.v->current = false;      // (a blended table holds the smoothed status)
    f->recorded |= account.capturing;
    return launch_ema(f, weight, obs_wait, obs_prefill, obs_decode, static_cast<hipStream_t>(hip_stream));
}

int gr_set_blend(gr_fleet* f, double black_box_weight)
{
    if (!f || !(black_box_weight >= 0.0 && black_box_weight <= 1.0)) return GR_ERR_INVALID_ARG;
    if (black_box_weight > 0.0 && !(f->have_q && f->have_p && f->have_d)) return GR_ERR_NO_STATUS;
    f->lam = black_box_weight;
    f->now.current = f->rec.current = false;
    return GR_OK;
}

int gr_set_small_batch_pairs(gr_fleet* f, int64_t max_pairs)
{
    if (!f || max_pairs < 0) return GR_ERR_INVALID_ARG;
    f->small_batch_pairs = max_pairs;
    return GR_OK;
}

int gr_set_feedback_wait(gr_fleet* f, int32_t looks)
{
    if (!f || looks < 0) return GR_ERR_INVALID_ARG;
    f->feed_polls = looks;
    return GR_OK;
}

int gr_set_feedback_team(gr_fleet* f, int32_t workgroups)
{
    if (!f || workgroups < 1) return GR_ERR_INVALID_ARG;
    f->feed_team = workgroups;
    return GR_OK;
}

int gr_feedback_team(gr_fleet* f, int32_t* out_workgroups)
{
    if (!f || !out_workgroups) return GR_ERR_INVALID_ARG;
    *out_workgroups = 0;
    if (!f->feed_words.team) return GR_OK;
    return hipDeviceSynchronize() == hipSuccess &&
           hipMemcpy(out_workgroups, f->feed_words.team, sizeof(int32_t), hipMemcpyDeviceToHost) == hipSuccess ? GR_OK : GR_ERR_HIP;
}

int gr_set_feedback_units(gr_fleet* f, int32_t units)
{
    if (!f || units < 0) return GR_ERR_INVALID_ARG;
    f->feed_units = units;
    return GR_OK;
}

int gr_set_batch_cap(gr_fleet* f, const int32_t* cap)
{
    if (!f) return GR_ERR_INVALID_ARG;
    f->now.current = f->rec.current = false;
    if (!cap) { f->has_cap = false; return GR_OK; }
    for (int g = 0; g < f->n_inst; ++g)
        if (cap[g] < 1) return GR_ERR_INVALID_ARG;
    if (hipDeviceSynchronize() != hipSuccess) return GR_ERR_HIP;
    if (hipMemcpy(f->batch_cap, cap, sizeof(int) * f->n_inst, hipMemcpyHostToDevice) != hipSuccess) return GR_ERR_HIP;
    f->has_cap = true;
    return GR_OK;
}

int gr_device_status(gr_fleet* f, int32_t* out_bits)
{
    if (!f || !out_bits) return GR_ERR_INVALID_ARG;
    if (hipDeviceSynchronize() != hipSuccess) return GR_ERR_HIP;
    int v = 0;
    if (hipMemcpy(&v, f->counters, sizeof(int), hipMemcpyDeviceToHost) != hipSuccess) return GR_ERR_HIP;
    *out_bits = v;
    return GR_OK;
}

int gr_profile_enable(gr_fleet* f, int32_t max_launches)
{
    if (!f || max_launches < 0) return GR_ERR_INVALID_ARG;
    Profiler& p = f->prof;
    if (hipDeviceSynchronize() != hipSuccess) return GR_ERR_HIP;
    p.ids.clear();
    p.on = max_launches > 0;
    p.ids.reserve((size_t)max_launches);
    while (p.events.size() < (size_t)max_launches * 2) {
        hipEvent_t e;
        if (hipEventCreate(&e) != hipSuccess) { p.on = false; return GR_ERR_HIP; }
        p.events.push_back(e);
    }
    return GR_OK;
}

int gr_profile_select(gr_fleet* f, uint64_t kernel_mask)
{
    if (!f) return GR_ERR_INVALID_ARG;
    f->prof.mask = kernel_mask;
    return GR_OK;
}

int gr_profile_read(gr_fleet* f, int32_t n_kernels, double* total_ms, int64_t* launches)
{
    if (!f || n_kernels < 0 || (n_kernels > 0 && (!total_ms || !launches))) return GR_ERR_INVALID_ARG;
    if (hipDeviceSynchronize() != hipSuccess) return GR_ERR_HIP;
    Profiler& p = f->prof;
    for (int k = 0; k < n_kernels; ++k) { total_ms[k] = 0.0; launches[k] = 0; }
    for (size_t i = 0; i < p.ids.size(); ++i) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, p.events[2 * i], p.events[2 * i + 1]) != hipSuccess) return GR_ERR_HIP;
        if (p.ids[i] < n_kernels) { total_ms[p.ids[i]] += ms; launches[p.ids[i]] += 1; }
    }
    p.ids.clear();
    return GR_OK;
}

int gr_profile_read_launches(gr_fleet* f, int32_t max_launches, int32_t* kernel_id, float* ms, int32_t* n_launches)
{
    if (!f || max_launches < 0 || !n_launches || (max_launches > 0 && (!kernel_id || !ms))) return GR_ERR_INVALID_ARG;
    if (hipDeviceSynchronize() != hipSuccess) return GR_ERR_HIP;
    Profiler& p = f->prof;
    const size_t n = p.ids.size() < (size_t)max_launches ? p.ids.size() : (size_t)max_launches;
    for (size_t i = 0; i < n; ++i) {
        if (hipEventElapsedTime(&ms[i], p.events[2 * i], p.events[2 * i + 1]) != hipSuccess) return GR_ERR_HIP;
        kernel_id[i] = p.ids[i];
    }
    *n_launches = (int32_t)n;
    p.ids.clear();
    return GR_OK;
}

int32_t gr_profile_kernel_count(void) { return kNumKernels; }

const char* gr_profile_kernel_name(int32_t id)
{
    return id >= 0 && id < kNumKernels ? kKernelNames[id] : "";
}

const char* gr_strerror(int code)
{
    switch (code) {
        case GR_OK: return "ok";
        case GR_ERR_INVALID_ARG: return "invalid argument";
        case GR_ERR_TOO_LARGE: return "size exceeds what the handle was created for or a hard limit";
        case GR_ERR_HIP: return "HIP runtime error";
        case GR_ERR_NO_STATUS: return "no status yet: gr_build_status / gr_risk_scan (or gr_observe) must come first";
        case GR_ERR_NOMEM: return "out of memory";
        default: return "unknown error";
    }
}

}  // extern "C"
