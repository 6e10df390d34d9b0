// Status build (step 1 of the path): per instance, a sort of the remaining
// lengths, three exact prefix sums over the sorted order, and from them the
// finish time of every held request (Sec. 3.4's "expected finish time"), q_g
// and d_g of Eq. 2, and the instance table used for scoring; then the
// capability order of Alg. 1's argmax d_g.
//
// One wave per instance (two or four when the fleet has fewer instances than
// the chip takes waves), everything in registers: a wave holds 64 * kEPL sort
// words (remaining length in the high bits, entry index in the low bits, so
// all words differ and the order is stable), kEPL consecutive positions of the
// sorted order per lane.  A bitonic network sorts them: exchanges inside a lane
// are a min/max pair, exchanges between lanes fetch the partner's word (through
// the register file or the LDS crossbar, see kShortChain) and keep the smaller
// or the larger of the two, mostly with one median-of-three against 0 or 0xFFFFFFFF.  No atomics; barriers only between the waves that
// share an instance.
#include <algorithm>
#include <cfloat>
#include <type_traits>

#include "common.h"

namespace gr {
namespace {

struct BuildArgs {
    const int *act_off, *act_prompt, *act_gen, *act_rem;
    const int *q_off, *q_prompt, *q_len;
    const float* act_budget;  // null unless flags are wanted
    float *out_act_finish, *out_q_finish;
    double* out_d;
    uint8_t* out_flag;
    const ClassCoef* cls;
    const int* inst_class;
    uint16_t* tabR;
    float2* tabGH;
    int* unset;          // 1: some running entry's flag is not set here (read by k_scan)
    double* hD;
    int* act_inst;
    float4* instK;
    uint16_t* tabS;
    const int* slot_of;
    unsigned long long* slot_key;
    int* counters;
    int64_t n_active, n_queued;
    int n_inst, max_entries, max_len;
    // for the migration pass of a risk scan: which lengths flagged requests have, and how many are flagged
    uint8_t* seen;       // null: nobody asks for the lengths
    int* late_cnt;
    // requests routed since the caller's status (feedback routing): per instance, queued behind the queue
    int* pend_cnt;
    int *pend_prompt, *pend_len;
    int use_pending;     // 0: a fresh status from the caller, the lists are emptied
    int* pend_touched;   // 1: given requests since its table was built
    int only_touched;    // leave the instances with a 0 there as they are
    // a chunk of up to kWave requests that has just been decided and joins the lists in this build
    // (0: no such chunk, or its requests are in the lists already); those not chosen count as not touched
    int chunk_n;
    const int *chunk_inst, *chunk_ctx0, *chunk_len;
    const int* batch_cap;   // per instance: requests that may decode together; null = no bound
    // blend with the smoothed black-box status (Sec. 3.3): weight lam on it, 0 = none
    double lam;
    const double *emaQ, *emaP, *emaD;
};

// The coefficients of a pair's latency that depend on the instance alone (see gr_fleet::instK);
// `bp`: its smoothed prefill seconds per token.
__device__ __forceinline__ float4 inst_coef(const BuildArgs& a, const ClassCoef& cc, double bp, int n)
{
    const double keep = 1.0 - a.lam;
    const float gam = (float)keep * (float)cc.gamma;
    // the smoothed status alone: every segment is the same (as long as no sum of the white-box part is infinite)
    if (keep == 0.0 && cc.delta + cc.alpha + cc.beta + cc.gamma < 1e100) n |= kAllAlike;
    return a.lam != 0.0 ? make_float4((float)(keep * cc.delta + a.lam * bp), (float)(keep * cc.gamma), gam, __int_as_float(n))
                        : make_float4((float)cc.delta, (float)cc.gamma, gam, __int_as_float(n));
}

// Median of three; the compiler turns this shape into one v_med3_u32.
__device__ __forceinline__ uint32_t med3_u32(uint32_t a, uint32_t b, uint32_t c)
{
    return min(max(a, b), max(min(a, b), c));
}

template <int kCtrl>
__device__ __forceinline__ uint32_t dpp_move(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, kCtrl, 0xf, 0xf, false);
}

__device__ __forceinline__ void order2(uint32_t& lo, uint32_t& hi)
{
    const uint32_t a = lo, b = hi;
    lo = a < b ? a : b;
    hi = a < b ? b : a;
}

// How a lane gets its partner's word.  What bounds a build decides.  With up to two words a lane several waves share an instance and a
// SIMD hardly has a wave to run meanwhile: an exchange is a step of a chain, and stays in the
// register file, whose step is shorter than the crossbar's.  With more words the vector ALU is what the waves of a SIMD wait for,
// and the fetches that no single pattern does are left to the crossbar.  Whole calls, us, everywhere like that / as here: refresh of 256 x 512 and
// one request 8.77 / 8.42, step of 32 x 256 20.43 / 20.00 (of 4 x 64: no difference that timing shows).  (All fetches through
// the crossbar: 8.85, 20.2; status of 4 096 x 512 21.3 / 21.0, but its scan 108.6 / 109.6; scan of 1 024 x 1 000 60.4 / 59.9 to 60.6.)
// Under caps an instance has one wave, whose sort is a chain between the turns of others': in the register file at every size.  Status
// under caps, crossbar / here: 1 024 x (56 + 7) 11.45 / 11.10, (110 + 13) 14.83 / 14.87, (224 + 28) 23.8 / 23.7, (450 + 56) 40.1 / 40.8 (long tails
// 27.7 / 27.7), (900 + 112) 78.5 / 77.1 (47.7 / 46.1), (1 820 + 227) 138.2 / 136.4 (88.5 / 85.1); 4 096 x 450 38.4 / 38.2, x (450 + 56) 90.8 / 92.3
// (61.0 / 60.7), x (900 + 112) 276 / 272 (154 / 149); 64 x 1 820 the same.
template <int kEPL>
constexpr bool kShortChain = kEPL <= 2;

// The copy of x held by lane (lane ^ kMask); lane4 = 4 * lane.
template <bool kChain, int kMask>
__device__ __forceinline__ uint32_t fetch_xor(uint32_t x, int lane4)
{
    if constexpr (kMask == 1) return dpp_move<0xB1>(x);       // quad_perm [1,0,3,2]
    else if constexpr (kMask == 2) return dpp_move<0x4E>(x);       // quad_perm [2,3,0,1]
    else if constexpr (kMask == 3) return dpp_move<0x1B>(x);       // quad_perm [3,2,1,0]
    else if constexpr (kMask == 7) return dpp_move<0x141>(x);      // row_half_mirror
    else if constexpr (kMask == 8 && kChain) return dpp_move<0x128>(x);      // row_ror:8
    else if constexpr (kMask == 15) return dpp_move<0x140>(x);     // row_mirror
    else return (uint32_t)__builtin_amdgcn_ds_bpermute(lane4 ^ (kMask << 2), (int)x);
}

// Words of lanes kMask apart in order, the lesser one in the lower lane, without the crossbar: shifts inside a row of which either half
// of the lanes takes one, or the halves of two registers changed over and back.
template <int kMask>
__device__ __forceinline__ void order_lanes(uint32_t& a, uint32_t& b)
{
    static_assert(kMask == 4 || kMask == 16 || kMask == 32);
    if constexpr (kMask == 4) {
        const auto both = [](uint32_t x) {
            const uint32_t lower = min((uint32_t)__builtin_amdgcn_update_dpp(-1, (int)x, 0x104, 0xf, 0x5, false), x);      // row_shl:4
            return max((uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xa, false), lower);                   // row_shr:4
        };
        a = both(a);
        b = both(b);
    } else {
        const auto change = [](uint32_t& x, uint32_t& y) {
            const auto v = kMask == 16 ? __builtin_amdgcn_permlane16_swap(x, y, false, false)
                                       : __builtin_amdgcn_permlane32_swap(x, y, false, false);
            x = v[0];
            y = v[1];
        };
        change(a, b);
        order2(a, b);
        change(a, b);
    }
}

// Ascending bitonic sort of 64 * kEPL words, word v = lane * kEPL + r in key[r].
// Level K merges sorted runs of K/2 into runs of K: first v against its mirror
// image v ^ (K-1) in the run, then distances K/4, K/8, .. 1; the lower position
// always keeps the smaller word.  Levels and distances are template parameters
// (the network is straight-line code with every register named at compile
// time; as loops over K and the distance the larger sizes were left rolled,
// with registers addressed indirectly).
template <bool kChain, int kEPL, int K>
__device__ __forceinline__ void bitonic_mirror(uint32_t (&key)[kEPL], int lane, int lane4)
{
    if constexpr (K <= kEPL) {
#pragma unroll
        for (int r = 0; r < kEPL; ++r)
            if (r < (r ^ (K - 1))) order2(key[r], key[r ^ (K - 1)]);
    } else {
        constexpr int lm = K / kEPL - 1;
        const uint32_t bound = (lane & (K / kEPL / 2)) ? 0xFFFFFFFFu : 0u;   // upper partner keeps the larger
        uint32_t p[kEPL];
#pragma unroll
        for (int r = 0; r < kEPL; ++r) p[r] = fetch_xor<kChain, lm>(key[kEPL - 1 - r], lane4);
#pragma unroll
        for (int r = 0; r < kEPL; ++r) key[r] = med3_u32(key[r], p[r], bound);
    }
}

template <bool kChain, int kEPL, int J>
__device__ __forceinline__ void bitonic_distances(uint32_t (&key)[kEPL], int lane, int lane4)
{
    if constexpr (J >= 1) {
        if constexpr (J < kEPL) {
#pragma unroll
            for (int r = 0; r < kEPL; ++r)
                if ((r & J) == 0) order2(key[r], key[r | J]);
        } else {
            constexpr int lm = J / kEPL;
            if constexpr (kChain && (lm == 4 || lm >= 16)) {
                uint32_t same = key[0];      // (one word a lane: two registers alike come to the same)
#pragma unroll
                for (int r = 0; r < kEPL; r += 2) order_lanes<lm>(key[r], kEPL > 1 ? key[r + 1 < kEPL ? r + 1 : r] : same);
            } else {
                const uint32_t bound = (lane & lm) ? 0xFFFFFFFFu : 0u;
#pragma unroll
                for (int r = 0; r < kEPL; ++r) key[r] = med3_u32(key[r], fetch_xor<kChain, lm>(key[r], lane4), bound);
            }
        }
        bitonic_distances<kChain, kEPL, J / 2>(key, lane, lane4);
    }
}

template <bool kChain, int kEPL, int K, int kMost = kWave * kEPL>
__device__ __forceinline__ void bitonic_levels(uint32_t (&key)[kEPL], int lane, int lane4)
{
    if constexpr (K <= kMost) {
        bitonic_mirror<kChain, kEPL, K>(key, lane, lane4);
        bitonic_distances<kChain, kEPL, K / 4>(key, lane, lane4);
        bitonic_levels<kChain, kEPL, 2 * K, kMost>(key, lane, lane4);
    }
}

template <bool kChain, int kEPL>
__device__ __forceinline__ void bitonic_sort(uint32_t (&key)[kEPL], int lane)
{
    bitonic_levels<kChain, kEPL, 2>(key, lane, lane << 2);
}

// The same network over the kSplit waves that share an instance (word v = (part * 64 + lane) *
// kEPL + r): each wave sorts its own words as above, and the levels that span waves fetch the
// partner's words through LDS -- word r of lane l of wave w sits at buf[(w * kEPL + r) * 64 + l],
// so every access is consecutive over the lanes, mirrored or not.  One workgroup barrier per
// exchange: consecutive exchanges alternate between two buffers, and a wave reaches the barrier
// of the next exchange only after it has read what it needed of this one.
template <int kEPL, bool kMirrored>
__device__ __forceinline__ void bitonic_exchange(uint32_t (&key)[kEPL], int lane, int part, int partner, bool upper,
                                                 uint32_t* buf)
{
#pragma unroll
    for (int r = 0; r < kEPL; ++r) buf[(part * kEPL + r) * kWave + lane] = key[r];
    __syncthreads();
    const uint32_t bound = upper ? 0xFFFFFFFFu : 0u;      // the upper partner keeps the larger word
#pragma unroll
    for (int r = 0; r < kEPL; ++r) {
        const uint32_t p = kMirrored ? buf[(partner * kEPL + (kEPL - 1 - r)) * kWave + (kWave - 1 - lane)]
                                     : buf[(partner * kEPL + r) * kWave + lane];
        key[r] = med3_u32(key[r], p, bound);
    }
}

template <int kEPL, int kSplit>
__device__ __forceinline__ void bitonic_sort_split(uint32_t (&key)[kEPL], int lane, int part, uint32_t* xch)
{
    static_assert(kSplit >= 2 && (kSplit & (kSplit - 1)) == 0, "a power of two of waves per instance");
    constexpr int kWords = kWave * kEPL, kCap = kWords * kSplit;
    const int lane4 = lane << 2;
    bitonic_levels<kShortChain<kEPL>, kEPL, 2>(key, lane, lane4);
    int flip = 0;
#pragma unroll
    for (int span = 2; span <= kSplit; span *= 2) {
        // runs of `span` waves: the mirror image across the run, then the same position span/4, .. 1
        // waves away, then the distances inside the wave
        bitonic_exchange<kEPL, true>(key, lane, part, part ^ (span - 1), part & (span / 2), xch + flip * kCap);
        flip ^= 1;
#pragma unroll
        for (int d = span / 4; d >= 1; d /= 2) {
            bitonic_exchange<kEPL, false>(key, lane, part, part ^ d, part & d, xch + flip * kCap);
            flip ^= 1;
        }
        bitonic_distances<kShortChain<kEPL>, kEPL, kWords / 2>(key, lane, lane4);
    }
}

// Sorted length number `v` of instance g, `len`, if it is one of the splitters of a search (every
// (kCap / splitters)-th; a lane's share of consecutive lengths never spans more than one stride).
template <int kCap>
__device__ __forceinline__ void store_splitter(uint16_t* tabS, int g, int v, uint16_t len)
{
    constexpr int kSplit = split_count(kCap), kStride = kCap / kSplit;
    if ((v + 1) % kStride == 0) tabS[(size_t)g * kSplit + v / kStride] = len;
}

// v of the lane `ctrl` names (0 where there is none or the row is masked out), both halves
template <int kCtrl, int kRowMask>
__device__ __forceinline__ long long dpp_or_zero_i64(long long v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, (int)v, kCtrl, kRowMask, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), kCtrl, kRowMask, 0xf, false);
    return ((long long)hi << 32) | (unsigned)lo;
}

// Inclusive prefix sum over the lanes of a wave (see wave_incl_scan_i32 for the pattern).
__device__ __forceinline__ long long wave_incl_scan_i64(long long v)
{
    v += dpp_or_zero_i64<0x111, 0xf>(v);   // row_shr:1
    v += dpp_or_zero_i64<0x112, 0xf>(v);   // row_shr:2
    v += dpp_or_zero_i64<0x114, 0xf>(v);   // row_shr:4
    v += dpp_or_zero_i64<0x118, 0xf>(v);   // row_shr:8
    v += dpp_or_zero_i64<0x142, 0xa>(v);   // row_bcast:15 into rows 1, 3
    v += dpp_or_zero_i64<0x143, 0xc>(v);   // row_bcast:31 into rows 2, 3
    return v;
}

// The last lane's value: of a prefix sum, the total.
__device__ __forceinline__ long long last_lane_i64(long long v)
{
    const int lo = __builtin_amdgcn_readlane((int)v, kWave - 1), hi = __builtin_amdgcn_readlane((int)(v >> 32), kWave - 1);
    return ((long long)hi << 32) | (unsigned)lo;
}

__device__ __forceinline__ long long wave_sum_i64(long long v) { return last_lane_i64(wave_incl_scan_i64(v)); }

// Exclusive prefix over the lanes of a wave, and the total.
__device__ __forceinline__ long long wave_excl_scan(long long v, long long& total)
{
    const long long incl = wave_incl_scan_i64(v);
    total = last_lane_i64(incl);
    return incl - v;
}

constexpr int kBuildWaves = kBlock / kWave;

constexpr int log2_of(int v) { return v <= 1 ? 0 : 1 + log2_of(v / 2); }

// The build under batch caps (a kernel of its own: the event loop's registers would cost the
// plain build, k_build_lean below, a wave per SIMD).  The loop over the events is one chain, so what
// bounds the kernel is the length of a turn: the next departure is found and the sums are formed
// without leaving the registers (DPP; through the LDS crossbar each step of a reduction waited
// for the one before it, and a turn had thirty-six), finish times go to LDS and reach the caller's
// arrays in entry order at the end, where a budget is also read (in the loop its read stood in
// the chain).  And as long as
// nobody can be admitted nothing is played at all.  1 024 instances of 200 running and 40 queued
// requests, caps of 120 to 288: 94 us, 54 with the shorter turns, 33 without the turns before the
// first admission, 30.5 with a turn's reductions side by side (one chain of DPP steps fills the waits of another),
// 27.9 where a turn of one departure and one admission has no sums over the lanes: the newcomer's context is read from LDS, the
// other's off its lane; an entry's context when it leaves is known beforehand, and one that has left is
// marked, so that the minimum needs no comparison with the step.  1 000 x (1 000 + 125) 167 -> 136, 4 096 x (400 + 50) 103 -> 89.
// (Less is won than prepared where one or two wait in tables of 513 to 1 024 entries: 64 x (1 000 + 1) 31.6 -> 32.1, + 2 32.0 -> 32.0, + 8 36.4 -> 35.2.)
// An instance without a queue plays no turn, and what the turns need is not prepared for it: 64 x 1 000 24.2 -> 22.8 us,
// 4 096 x 900 95.5 -> 91, 1 024 x 1 820 60.7 -> 56.6.
constexpr int kLowBits = 24;     // a lane's sum of contexts is added up over the wave in two parts of 32 bits
constexpr long long kLowMask = (1ll << kLowBits) - 1;

template <int kEPL>
__global__ __launch_bounds__(kBlock, 1) void k_build_capped(BuildArgs a)
{
    fetch_args<BuildArgs>();
    extern __shared__ uint32_t smem[];
    constexpr int kCap = kWave * kEPL;
    constexpr int kIdxBits = log2_of(kCap);
    constexpr uint32_t kIdxMask = (1u << kIdxBits) - 1u;
    const int lane = lane_id(), wave = threadIdx.x / kWave;
    const int g = blockIdx.x * kBuildWaves + wave;
    if (g >= a.n_inst) return;
    {   // feedback routing: an instance that has been given nothing since its table was built keeps it
        const bool touched = a.pend_touched[g] != 0;
        if (lane == 0 && touched) a.pend_touched[g] = 0;
        if (a.only_touched && !touched) return;
    }
    // this wave's entries, by index: white-box finish times (none yet: -1), and contexts (once the
    // events have been played, as they are when a newcomer would be admitted)
    double* fin_lds = reinterpret_cast<double*>(smem) + wave * kCap;
    int* ctx = reinterpret_cast<int*>(reinterpret_cast<double*>(smem) + kBuildWaves * kCap) + wave * kCap;
    constexpr double kNoFinish = -1.0;

    const ClassCoef cc = a.cls[a.inst_class[g]];
    // offsets are clamped into the arrays, so broken CSR data cannot index outside them
    const int a0 = (int)min((int64_t)max(a.act_off[g], 0), a.n_active);
    const int q0 = (int)min((int64_t)max(a.q_off[g], 0), a.n_queued);
    int A = (int)max(min((int64_t)a.act_off[g + 1], a.n_active) - a0, (int64_t)0);
    int Q = (int)max(min((int64_t)a.q_off[g + 1], a.n_queued) - q0, (int64_t)0);
    int status = 0;
    if (A > a.max_entries) { A = a.max_entries; status |= GR_DEV_ENTRIES_DROPPED; }
    if (Q > a.max_entries - A) { Q = a.max_entries - A; status |= GR_DEV_ENTRIES_DROPPED; }
    int P = a.use_pending ? min(a.pend_cnt[g], kCap) : 0;
    if (P > a.max_entries - A - Q) { P = a.max_entries - A - Q; status |= GR_DEV_ENTRIES_DROPPED; }
    const int N = A + Q + P;
    const int* pp = a.pend_prompt + (size_t)g * kCap;
    const int* pl = a.pend_len + (size_t)g * kCap;

    // load, entry i = 64 r + lane.  First every entry's three words, from wherever its kind keeps
    // them (running, queued, routed since the status), so that all loads are in flight together;
    // then one sort word per entry = (remaining length << kIdxBits) | i.
    int rem_in[kEPL], c_in[kEPL], gen_in[kEPL];
#pragma unroll
    for (int r = 0; r < kEPL; ++r) {
        const int i = r * kWave + lane;
        const int* p_rem = a.act_rem + a0 + i;
        const int* p_ctx = a.act_prompt + a0 + i;
        if (i >= A + Q) { p_rem = pl + (i - A - Q); p_ctx = pp + (i - A - Q); }
        else if (i >= A) { p_rem = a.q_len + q0 + (i - A); p_ctx = a.q_prompt + q0 + (i - A); }
        rem_in[r] = i < N ? *p_rem : 0;
        c_in[r] = i < N ? *p_ctx : 0;
        gen_in[r] = i < A ? a.act_gen[a0 + i] : 0;
    }
    uint32_t key[kEPL];
    long long qsum = 0;
#pragma unroll
    for (int r = 0; r < kEPL; ++r) {
        const int i = r * kWave + lane;
        uint32_t word = 0xFFFFFFFFu;        // past the last entry: sorts to the end
        if (i < N) {
            int rem = rem_in[r];
            const int c = c_in[r] + gen_in[r];
            if (i >= A) qsum += c;
            if (rem < 0 || rem > a.max_len) { rem = min(max(rem, 0), a.max_len); status |= GR_DEV_LEN_CLAMPED; }
            word = ((uint32_t)rem << kIdxBits) | (uint32_t)i;
            c_in[r] = c;
        }
        ctx[i] = c_in[r];
        fin_lds[i] = kNoFinish;
        key[r] = word;
    }
    // the instance of each running request, for the migration pass of a risk scan
    // (stores on their own: a store between two uses of loaded words would make the second wait for it)
    if (a.act_budget) {
#pragma unroll
        for (int r = 0; r < kEPL; ++r)
            if (r * kWave + lane < A) a.act_inst[a0 + r * kWave + lane] = g;
    }
    if (status) atomicOr(&a.counters[0], status);
    if (a.act_budget && (status & GR_DEV_ENTRIES_DROPPED)) *a.unset = 1;
    if (Q + P > 0) qsum = wave_sum_i64(qsum);   // Q and P are the same in every lane
    double q = cc.delta * (double)qsum;

    // with a blend, every estimate below is keep * (white-box value) + lam * (Eq. 2 with the smoothed status)
    const bool blended = a.lam != 0.0;
    const double keep = 1.0 - a.lam;
    const double bq = blended ? a.emaQ[g] : 0.0, bp = blended ? a.emaP[g] : 0.0, bd = blended ? a.emaD[g] : 0.0;
    // what a request of the instance is told, at the end and in entry order
    const auto report_all = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        int n_late = 0;
#pragma unroll 4
        for (int r = 0; r < kEPL; ++r) {
            const int i = r * kWave + lane;
            double fin = fin_lds[i];
            if (a.act_budget && i < A && fin == kNoFinish) *a.unset = 1;      // (no token left to decode)
            if (i >= A + Q || fin == kNoFinish) continue;
            // (length and prompt as given are read again: kept through the events they would spill)
            const float bud = a.act_budget && i < A ? a.act_budget[a0 + i] : 0.f;
            int rem = 0;
            if (a.act_budget || blended) rem = min(max(i < A ? a.act_rem[a0 + i] : a.q_len[q0 + i - A], 0), a.max_len);
            if (blended)   // black-box finish: d per remaining token; a queued request also waits and prefills
                fin = keep * fin + a.lam * (i < A ? bd * (double)rem
                                                  : (bq + bp * (double)a.q_prompt[q0 + i - A]) + bd * (double)rem);
            if (i < A) {
                a.out_act_finish[a0 + i] = (float)fin;
                if (a.act_budget) {
                    const bool late = fin > (double)bud;
                    a.out_flag[a0 + i] = late;
                    if (late) { if (a.seen) a.seen[rem] = 1; ++n_late; }
                }
            } else if (a.out_q_finish) {
                a.out_q_finish[q0 + i - A] = (float)fin;
            }
        }
        if (a.act_budget) {
            n_late = wave_incl_scan_i32(n_late);
            if (lane == kWave - 1) a.late_cnt[g] = n_late;
        }
    };

    // ---- batch cap (Sec. 3.1: concurrency bounded by memory).  With room for everybody and a
    // newcomer nothing changes.  Otherwise, while there is a queue, the instance is played forward
    // event by event (the queue's head is admitted whenever the batch has room; between two
    // departures the batch is fixed and its time is a closed form); requests that leave meanwhile
    // get their finish time here.  Once the queue is empty only departures are left: if the batch
    // has room now, a newcomer is admitted now (q_g = now, and the closed form below is built on
    // what is running); if not, it is admitted after the departure that makes room, which the
    // closed form itself gives (further down).
    const int cap_g = max(a.batch_cap[g], 1);
    const bool capped = cap_g <= N;
    int Nrun = N;
    double d_first = -1.0;
    if (capped && A < N) {
        // decode step at which the entry leaves (kNever and more: not in yet, gone, none), steps it stays once it is admitted,
        // its context when it leaves
        constexpr uint32_t kNever = 0x7fffffffu;
        uint32_t fstep[kEPL], stays[kEPL];
        int ctx_end[kEPL];
#pragma unroll
        for (int r = 0; r < kEPL; ++r) {
            const int i = r * kWave + lane;
            const uint32_t len0 = i < N ? key[r] >> kIdxBits : 0u;
            stays[r] = len0 ? len0 : kNever;
            fstep[r] = i < A ? stays[r] : kNever;
            ctx_end[r] = ctx[i] + (int)len0;
        }
        long long C = 0;
#pragma unroll
        for (int r = 0; r < kEPL; ++r) C += r * kWave + lane < A ? ctx[r * kWave + lane] : 0;
        C = wave_sum_i64(C);
        int n = A, s = 0, next_q = A;     // batch size, steps done, next entry of the queue
        double t = 0.0;
        // More running than the cap allows: nobody is admitted until enough of them have left, and up to
        // then every finish time is the closed form over the sorted lengths: the turns of the loop
        // below start with the first admission.  (An entry without a token left is the loop's business.)
        if (A >= cap_g) {
            uint32_t run[kEPL];
#pragma unroll
            for (int r = 0; r < kEPL; ++r) run[r] = r * kWave + lane < A ? key[r] : 0xFFFFFFFFu;
            bitonic_sort<true, kEPL>(run, lane);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            int R[kEPL], cx[kEPL];
            long long yl = 0, xl = 0, cl = 0;
#pragma unroll
            for (int r = 0; r < kEPL; ++r) {
                const bool valid = lane * kEPL + r < A;
                R[r] = valid ? (int)(run[r] >> kIdxBits) : 0;
                cx[r] = valid ? ctx[run[r] & kIdxMask] : 0;
                yl += R[r];
                xl += (long long)cx[r] * R[r] + (long long)(R[r] * (R[r] - 1) / 2);
                cl += cx[r];
            }
            if (__builtin_amdgcn_readfirstlane(R[0]) > 0) {
                long long Y, X, Pc, Ctot;
                Y = wave_excl_scan(yl, Ctot); X = wave_excl_scan(xl, Ctot); Pc = wave_excl_scan(cl, Ctot);
                const int leave = A - cap_g + 1;      // departures until there is room
                int step = 0;
#pragma unroll
                for (int r = 0; r < kEPL; ++r)
                    if (lane * kEPL + r == leave - 1) step = R[r];
                step = __shfl(step, (leave - 1) / kEPL, kWave);
                double t_at = 0.0;
                int gone = 0;
                long long goneC = 0;
#pragma unroll
                for (int r = 0; r < kEPL; ++r) {
                    const int v = lane * kEPL + r;
                    const long long Rr = R[r], triR = (long long)(R[r] * (R[r] - 1) / 2);
                    Y += Rr; X += (long long)cx[r] * Rr + triR; Pc += cx[r];
                    if (v < A && R[r] <= step) {
                        const double n_after = (double)(A - v - 1), S_next = (double)(Ctot - Pc), Rd = (double)Rr;
                        const double I1 = (double)Y + n_after * Rd;
                        const double I2 = (double)X + Rd * S_next + n_after * (double)triR;
                        const double fin = fma(cc.gamma, I2, fma(cc.beta, I1, cc.alpha * Rd));
                        fin_lds[run[r] & kIdxMask] = fin;
                        if (v == leave - 1) t_at = fin;
                        ++gone;
                        goneC += cx[r];
                    }
                }
                d_first = fma(cc.gamma, (double)C, fma(cc.beta, (double)n, cc.alpha));
                t = __shfl(t_at, (leave - 1) / kEPL, kWave);
                s = step;
                n -= (int)wave_sum_i64(gone);
                C += (long long)n * s - wave_sum_i64(goneC);
            }
        }
        // (the wave's own contexts in LDS)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int r = 0; r < kEPL; ++r) fstep[r] = fstep[r] > (uint32_t)s ? fstep[r] : kNever;
        double Cd = (double)C;        // (an integer below 2^53, as all that is added to it)
        long long left = 0;           // this lane's contexts that left with the last departure, where several did: not taken off Cd yet
        bool several = false;
        for (int guard = 0; guard <= 2 * N + 2; ++guard) {
            // admit entries next_q .. next_q + k - 1: prefill, then into the batch; and the next departure.  Nearly always
            // one leaves and one comes, which needs no sum over the lanes; else the sums and the minimum are formed side by side
            // (each alone is a chain of steps that wait for one another)
            const int k = max(min(cap_g - n, N - next_q), 0);
            uint32_t smin = kNever;
            if (k <= 1 && !several) {
                if (k) {
                    const double in = (double)ctx[next_q];
                    t += cc.delta * in;
                    Cd += in;
#pragma unroll
                    for (int r = 0; r < kEPL; ++r) fstep[r] = lane - next_q == -r * kWave ? (uint32_t)s + stays[r] : fstep[r];
                }
#pragma unroll
                for (int r = 0; r < kEPL; ++r) smin = min(smin, fstep[r]);
                smin = min_over<false>(smin);
            } else {
                long long in_l = 0;
#pragma unroll
                for (int r = 0; r < kEPL; ++r) {
                    const bool admitted = (uint32_t)(r * kWave + lane - next_q) < (uint32_t)k;
                    fstep[r] = admitted ? (uint32_t)s + stays[r] : fstep[r];
                    in_l += admitted ? ctx_end[r] - (stays[r] == kNever ? 0 : (int)stays[r]) : 0;
                    smin = min(smin, fstep[r]);
                }
                const long long dc_l = in_l - (several ? left : 0ll);
                const int in_lo = wave_incl_scan_i32((int)(in_l & kLowMask)), in_hi = wave_incl_scan_i32((int)(in_l >> kLowBits));
                const int dc_lo = wave_incl_scan_i32((int)(dc_l & kLowMask)), dc_hi = wave_incl_scan_i32((int)(dc_l >> kLowBits));
                smin = min_over<false>(smin);
                const auto total = [](int lo, int hi) {
                    return (double)(((long long)__builtin_amdgcn_readlane(hi, kWave - 1) << kLowBits) + __builtin_amdgcn_readlane(lo, kWave - 1));
                };
                if (k > 0) t += cc.delta * total(in_lo, in_hi);
                Cd += total(dc_lo, dc_hi);
            }
            n += k; next_q += k;
            if (next_q == N) break;        // the queue is empty: what follows is departures only (below)
            if (smin >= kNever) break;           // (nobody is running: cannot be, the batch has room then)
            const double step_now = fma(cc.gamma, Cd, fma(cc.beta, (double)n, cc.alpha));
            if (d_first < 0.0) d_first = step_now;
            const int ks = (int)smin - s;      // (no more than the longest length)
            // ks steps of a fixed batch: contexts grow by one per member and step
            t += (double)ks * step_now + cc.gamma * ((double)n * (double)(ks * (ks - 1) / 2));
            Cd += (double)(n * ks);
            s = (int)smin;
            int gone = 0, ctx_gone = 0, at = 0;
            unsigned long long lanes = 0;
            bool leaves[kEPL];
#pragma unroll
            for (int r = 0; r < kEPL; ++r) {
                leaves[r] = fstep[r] == smin;
                const unsigned long long m = __ballot(leaves[r]);
                gone += __popcll(m);
                lanes |= m;
                ctx_gone = leaves[r] ? ctx_end[r] : ctx_gone;
                at = leaves[r] ? r * kWave + lane : at;
                fstep[r] = leaves[r] ? kNever : fstep[r];
            }
            several = gone > 1;
            if (!several) {
                if ((lanes >> lane) & 1ull) fin_lds[at] = t;
                Cd -= (double)__builtin_amdgcn_readlane(ctx_gone, __ffsll((long long)lanes) - 1);
            } else {
                left = 0;
#pragma unroll
                for (int r = 0; r < kEPL; ++r)
                    if (leaves[r]) {
                        left += ctx_end[r];
                        fin_lds[r * kWave + lane] = t;
                    }
            }
            n -= gone;
        }
        // what is left, as of now: the sort words and contexts the closed form is built from
        q = t;
        Nrun = n;
#pragma unroll
        for (int r = 0; r < kEPL; ++r) {
            const int i = r * kWave + lane;
            const bool running = fstep[r] < kNever;
            key[r] = running ? ((fstep[r] - (uint32_t)s) << kIdxBits) | (uint32_t)i : 0xFFFFFFFFu;
            if (running) ctx[i] = ctx_end[r] - (int)(fstep[r] - (uint32_t)s);
        }
    } else if (capped) {      // nobody waits: what is running is left as it is (one without a token is not)
#pragma unroll
        for (int r = 0; r < kEPL; ++r) key[r] = key[r] >> kIdxBits ? key[r] : 0xFFFFFFFFu;
    }

    bitonic_sort<true, kEPL>(key, lane);

    // the wave's own LDS writes above must be visible to its reads below
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

    // sorted position v = lane * kEPL + r; entries first, in order of remaining length
    int R[kEPL], cx[kEPL], idx[kEPL];
    long long yl = 0, xl = 0, cl = 0;       // this lane's sums of R, c*R + tri(R), c
#pragma unroll
    for (int r = 0; r < kEPL; ++r) {
        const bool valid = lane * kEPL + r < Nrun;
        idx[r] = (int)(key[r] & kIdxMask);
        R[r] = valid ? (int)(key[r] >> kIdxBits) : 0;
        cx[r] = valid ? ctx[idx[r]] : 0;
        yl += R[r];
        xl += (long long)cx[r] * R[r] + (long long)(R[r] * (R[r] - 1) / 2);
        cl += cx[r];
    }
    long long Ytot, Xtot, Ctot;
    long long Y = wave_excl_scan(yl, Ytot), X = wave_excl_scan(xl, Xtot), Pc = wave_excl_scan(cl, Ctot);

    // ---- a full batch with an empty queue: a newcomer is admitted when the kstar-th of the running
    // requests has left.  Until then nobody joins, so everybody's finish time is the closed form
    // as it stands, the admission time q_g is the finish time of that request (s steps from now),
    // and the table describes the others as they are then: s steps shorter, contexts s longer.
    // With R' = R - s, c' = c + s over the survivors (positions vstar.. of the sorted order):
    //   sum R' = sum R - m s,   sum (c' R' + tri(R')) = sum (c R + tri(R)) - s sum c - m tri(s),
    //   sum c' = sum c + m s    (m terms each; all integers, exact)
    {
        if (capped && Nrun >= cap_g) {
            const int kstar = Nrun - cap_g + 1;
            long long Y1 = Y, X1 = X, P1 = Pc;
            double q_adm = 0.0;
            int sstar = 0;
#pragma unroll
            for (int r = 0; r < kEPL; ++r) {
                const int v = lane * kEPL + r;
                const long long Rr = R[r], triR = (long long)(R[r] * (R[r] - 1) / 2);
                Y1 += Rr; X1 += (long long)cx[r] * Rr + triR; P1 += cx[r];
                if (v < Nrun) {
                    const double n_after = (double)(Nrun - v - 1), S_next = (double)(Ctot - P1), Rd = (double)Rr;
                    const double I1 = (double)Y1 + n_after * Rd;
                    const double I2 = (double)X1 + Rd * S_next + n_after * (double)triR;
                    const double fin = q + fma(cc.gamma, I2, fma(cc.beta, I1, cc.alpha * Rd));
                    fin_lds[idx[r]] = fin;
                    if (v == kstar - 1) { q_adm = fin; sstar = R[r]; }
                }
            }
            const int owner = (kstar - 1) / kEPL;
            q_adm = __shfl(q_adm, owner, kWave);
            sstar = __shfl(sstar, owner, kWave);
            // those that have left by then (equal lengths leave together)
            long long gone = 0, yg = 0, xg = 0, cg = 0;
#pragma unroll
            for (int r = 0; r < kEPL; ++r)
                if (lane * kEPL + r < Nrun && R[r] <= sstar) {
                    ++gone; yg += R[r]; cg += cx[r];
                    xg += (long long)cx[r] * R[r] + (long long)(R[r] * (R[r] - 1) / 2);
                }
            const int vstar = (int)wave_sum_i64(gone);
            const long long Ystar = wave_sum_i64(yg), Xstar = wave_sum_i64(xg), Pstar = wave_sum_i64(cg);
            const int Nleft = Nrun - vstar;
            const long long s64 = sstar, tri_s = s64 * (s64 - 1) / 2;
            Y1 = Y; X1 = X; P1 = Pc;
            uint16_t* dstR = a.tabR + (size_t)g * kCap;
            uint16_t* dstS = a.tabS + (size_t)g * split_count(kCap);
            constexpr int kStride = kCap / split_count(kCap);
            float2* dstGH = a.tabGH + gh_at(g, 1, kCap);
            const auto put_R = [&](int slot, uint16_t len) {
                dstR[slot] = len;
                if ((slot + 1) % kStride == 0) dstS[slot / kStride] = len;
            };
#pragma unroll
            for (int r = 0; r < kEPL; ++r) {
                const int v = lane * kEPL + r;
                const long long Rr = R[r];
                Y1 += Rr; X1 += (long long)cx[r] * Rr + (long long)(R[r] * (R[r] - 1) / 2); P1 += cx[r];
                if (v >= vstar && v < Nrun) {
                    const int w = v - vstar;                      // position among the survivors
                    const long long m = w + 1;
                    const double Ys = (double)((Y1 - Ystar) - m * s64);
                    const double Xs = (double)((X1 - Xstar) - s64 * (P1 - Pstar) - m * tri_s);
                    const double n_after = (double)(Nleft - w - 1);
                    const double S_next = (double)((Ctot - P1) + (long long)(Nleft - w - 1) * s64);
                    double Gq = q_adm + (cc.beta * Ys + cc.gamma * Xs);
                    double Hs = cc.alpha + (cc.beta * (n_after + 1.0) + cc.gamma * S_next);
                    if (blended) { Gq = keep * Gq + a.lam * bq; Hs = keep * Hs + a.lam * bd; }
                    put_R(w, (uint16_t)(R[r] - sstar));
                    dstGH[w] = make_float2((float)Gq, (float)Hs);
                } else {                                          // the slots behind the survivors
                    const int slot = v < Nrun ? Nleft + v : v;
                    put_R(slot, (uint16_t)0xFFFFu);
                    dstGH[slot] = make_float2(0.f, 0.f);
                }
            }
            report_all();
            if (lane == 0) {
                const double Cd = (double)((Ctot - Pstar) + (long long)Nleft * s64);
                double Gq0 = q_adm, H0 = cc.alpha + (cc.beta * (double)(Nleft + 1) + cc.gamma * Cd);
                if (blended) { Gq0 = keep * Gq0 + a.lam * bq; H0 = keep * H0 + a.lam * bd; }
                a.tabGH[gh_at(g, 0, kCap)] = make_float2((float)Gq0, (float)H0);
                a.instK[g] = inst_coef(a, cc, bp, Nleft);
                if (!a.use_pending) a.pend_cnt[g] = 0;
                // the next decode step that runs: the first one played above, else the batch as it stands
                double d = d_first >= 0.0 ? d_first
                                          : fma(cc.gamma, (double)Ctot, fma(cc.beta, (double)Nrun, cc.alpha));
                if (blended) d = keep * d + a.lam * bd;
                a.hD[g] = d;
                a.slot_key[a.slot_of[g]] = falling_bits(d);
                if (a.out_d) a.out_d[g] = d;
            }
            return;
        }
    }

    // table entry v describes the segment after the v+1 shortest requests, n of them still running:
    //   E_g(L) = Gq + L * H + tri(L) * gamma * (n + 1)
    //   Gq = q + beta * Y + gamma * X,   H = alpha + beta * (n + 1) + gamma * S
    uint16_t tR[kEPL];
    float2 tGH[kEPL];
#pragma unroll
    for (int r = 0; r < kEPL; ++r) {
        const int v = lane * kEPL + r;
        const bool valid = v < Nrun;
        const long long Rr = R[r], triR = (long long)(R[r] * (R[r] - 1) / 2);
        Y += Rr;
        X += (long long)cx[r] * Rr + triR;
        Pc += cx[r];
        const double n_after = (double)(Nrun - v - 1), S_next = (double)(Ctot - Pc);
        const double Yd = (double)Y, Xd = (double)X, Rd = (double)Rr;
        tR[r] = valid ? (uint16_t)R[r] : (uint16_t)0xFFFFu;
        double Gq = q + (cc.beta * Yd + cc.gamma * Xd);
        double Hs = cc.alpha + (cc.beta * (n_after + 1.0) + cc.gamma * S_next);
        if (blended) { Gq = keep * Gq + a.lam * bq; Hs = keep * Hs + a.lam * bd; }
        tGH[r] = make_float2((float)Gq, (float)Hs);
        if (valid) {
            // every product below is an integer below 2^53: exact
            const double I1 = Yd + n_after * Rd;
            const double I2 = Xd + Rd * S_next + n_after * (double)triR;
            const double fin = q + fma(cc.gamma, I2, fma(cc.beta, I1, cc.alpha * Rd));
            fin_lds[idx[r]] = fin;
        }
    }
    {
        uint16_t* dstR = a.tabR + (size_t)g * kCap + lane * kEPL;
        float2* dstGH = a.tabGH + gh_at(g, 1, kCap) + lane * kEPL;
        if constexpr (kEPL >= 8) {
#pragma unroll
            for (int r = 0; r < kEPL; r += 8) {
                uint4 w;
                w.x = tR[r] | ((uint32_t)tR[r + 1] << 16); w.y = tR[r + 2] | ((uint32_t)tR[r + 3] << 16);
                w.z = tR[r + 4] | ((uint32_t)tR[r + 5] << 16); w.w = tR[r + 6] | ((uint32_t)tR[r + 7] << 16);
                *reinterpret_cast<uint4*>(dstR + r) = w;
            }
        } else {
#pragma unroll
            for (int r = 0; r < kEPL; ++r) dstR[r] = tR[r];
        }
        if constexpr (kEPL >= 2) {
#pragma unroll
            for (int r = 0; r < kEPL; r += 2)
                *reinterpret_cast<float4*>(dstGH + r) = make_float4(tGH[r].x, tGH[r].y, tGH[r + 1].x, tGH[r + 1].y);
        } else {
            dstGH[0] = tGH[0];
        }
        store_splitter<kCap>(a.tabS, g, lane * kEPL + kEPL - 1, tR[kEPL - 1]);
    }
    report_all();
    if (lane == 0) {
        const double Cd = (double)Ctot;
        double Gq0 = q, H0 = cc.alpha + (cc.beta * (double)(Nrun + 1) + cc.gamma * Cd);
        if (blended) { Gq0 = keep * Gq0 + a.lam * bq; H0 = keep * H0 + a.lam * bd; }
        a.tabGH[gh_at(g, 0, kCap)] = make_float2((float)Gq0, (float)H0);
        a.instK[g] = inst_coef(a, cc, bp, Nrun);
        if (!a.use_pending) a.pend_cnt[g] = 0;
        // the next decode step that runs: the first one played above, else the batch as it stands
        double d = d_first >= 0.0 ? d_first : fma(cc.gamma, Cd, fma(cc.beta, (double)Nrun, cc.alpha));
        if (blended) d = keep * d + a.lam * bd;
        a.hD[g] = d;
        a.slot_key[a.slot_of[g]] = falling_bits(d);
        if (a.out_d) a.out_d[g] = d;
    }
}

// ---- the build without batch caps: the same results from fewer instructions.
//
// The instance's running requests are read and their results written through buffer
// descriptors that span exactly the instance's slice of the caller's arrays: an offset past
// the slice reads zero and stores nothing, so there is no address arithmetic and no branch per
// entry.  The three prefix sums run in double precision (every term and every sum is an
// integer below 2^53, so they are exact), first along the lane's own consecutive positions,
// then across the lanes by DPP shifts, and the table and finish times come out of them with
// fused multiply-adds, without any integer-to-double conversion of a 64-bit sum.

// x of the lane `ctrl` names (0.0 where there is none or the row is masked out), both halves
template <int kCtrl, int kRowMask>
__device__ __forceinline__ double dpp_or_zero(double x)
{
    const long long b = __builtin_bit_cast(long long, x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, kCtrl, kRowMask, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), kCtrl, kRowMask, 0xf, false);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

// Inclusive prefix sum over the lanes of a wave (see wave_incl_scan_i32 for the pattern).
__device__ __forceinline__ double wave_incl_scan_f64(double v)
{
    v += dpp_or_zero<0x111, 0xf>(v);   // row_shr:1
    v += dpp_or_zero<0x112, 0xf>(v);   // row_shr:2
    v += dpp_or_zero<0x114, 0xf>(v);   // row_shr:4
    v += dpp_or_zero<0x118, 0xf>(v);   // row_shr:8
    v += dpp_or_zero<0x142, 0xa>(v);   // row_bcast:15 into rows 1, 3
    v += dpp_or_zero<0x143, 0xc>(v);   // row_bcast:31 into rows 2, 3
    return v;
}

__device__ __forceinline__ double readlane_f64(double v, int lane)
{
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_readlane((int)b, lane), hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

constexpr int kBufferDwords = 0x00020000;   // descriptor word 3: raw buffer of 32-bit elements

// 32-bit words of LDS per instance of the plain build: contexts, budgets / finish times, flag bytes
constexpr int lean_inst_words(int cap) { return 2 * cap + cap / 4; }

// T of a request on segment k of an instance, as k_direct forms it
__device__ __forceinline__ float latency_at(float c0, int L, const float4& K, const float2& gh, int k)
{
    const float Lf = (float)L, tri = Lf * (Lf - 1.0f) * 0.5f;
    const int N = entries_of(K);
    const float E = fmaf(tri, K.z * (float)(N - k + 1), fmaf(Lf, gh.y, gh.x));
    return fmaf(c0, kappa_of(make_float2(K.x, K.y), Lf), E);
}

struct InstanceIn {
    int g, a0, q0, A, Q, P, status;     // the instance, its slices of the caller's arrays and their lengths, GR_DEV_* bits
    int pend;                           // entries in its list, not counting those of the chunk
    unsigned long long joins;           // requests of the chunk that were sent here
};

// What the instance offers a request of the next decision round, a lane each (see k_feedback).
struct Offer {
    int L;
    float c0, T;
    unsigned long long key;     // d_g as an integer that falls with it
    // the sums that the table is made from, kept for the rounds to come (null: not asked for), see gr_fleet
    double2* sums_yx;
    double* sums_c;
    FeedBase* base;
};

// kEPL sort words per lane; kSplit waves share an instance (kSplit = 1: a workgroup is four instances, a wave each; 2 or 4:
// a workgroup is one instance): wave `part` reads entries part * 64 * kEPL onwards, the sort's
// last levels and the totals of the prefix sums cross the waves through LDS, and the wave ends
// up with sorted positions part * 64 * kEPL onwards.  The results are the same bit for bit (the
// sums are exact); a fleet with fewer instances than the chip has SIMDs gets shorter dependent
// chains and more waves to overlap them.
//
// The work is that of kEPL * 64 * kSplit words; the tables have room for kTab >= that many entries.
//
// kQuiet: nobody asks for finish times or flags.  With an `offer` (of the instance's first wave) the latency of its
// request is formed from the new table, as k_direct would.
template <int kEPL, int kSplit, int kTab, bool kQuiet, bool kOffer = false, bool kSums = false>
__device__ __forceinline__ void build_instance(const BuildArgs& a, const InstanceIn& in, int wave, uint32_t* smem, Offer* offer = nullptr)
{
    const bool risk = !kQuiet && a.act_budget;
    constexpr int kWords = kWave * kEPL;         // sort words of a wave
    constexpr int kCap = kWords * kSplit;        // of the instance
    constexpr int kIdxBits = log2_of(kCap);
    constexpr uint32_t kIdxMask = (1u << kIdxBits) - 1u;
    const int lane = lane_id();
    const int g = in.g;
    const int part = kSplit == 1 ? 0 : wave;
    const int first = part * kWords;             // this wave's first entry, and its first sorted position
    // LDS of an instance, all by entry index: contexts; budgets on the way in and finish times on the
    // way out (the caller's arrays are read and written in their own order, 64 consecutive entries
    // per instruction; the sorted order reaches them through LDS); flags, a byte each
    constexpr int kInstWords = lean_inst_words(kCap);
    uint32_t* const mine_lds = smem + (kSplit == 1 ? wave * kInstWords : 0);
    int* ctx = reinterpret_cast<int*>(mine_lds);
    float* stage = reinterpret_cast<float*>(mine_lds + kCap);
    uint8_t* flag_lds = reinterpret_cast<uint8_t*>(mine_lds + 2 * kCap);
    uint32_t* xch = smem + kInstWords;                                              // (split) two exchange buffers
    double* sums = reinterpret_cast<double*>(smem + kInstWords + 2 * kCap);         // (split) four totals per wave

    const ClassCoef cc = a.cls[a.inst_class[g]];
    // (used at the very end.  Read here it need not be waited for there, which is what a round of feedback routing gains by;
    // a plain build has other waves to run meanwhile, and reads it and forms the instance's own figures in one lane at the end:
    // status of 4 096 instances x 512 21.5 us the other way, 21.2 like this)
    const int slot = kQuiet ? a.slot_of[g] : 0;
    const int a0 = in.a0, q0 = in.q0, A = in.A, Q = in.Q, P = in.P, N = A + Q + P;
    int status = in.status;

    // the instance's slice of each array of running requests (A entries from a0 on)
    const auto slice = [&](const void* base, size_t elem) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(static_cast<const char*>(base)) + (size_t)a0 * elem,
                                                 0, A * (int)elem, kBufferDwords);
    };
    const __amdgpu_buffer_rsrc_t b_rem = slice(a.act_rem, 4), b_prompt = slice(a.act_prompt, 4),
                                 b_gen = slice(a.act_gen, 4), b_fin = slice(a.out_act_finish, 4);
    __amdgpu_buffer_rsrc_t b_bud = b_fin, b_flag = b_fin;
    if (risk) { b_bud = slice(a.act_budget, 4); b_flag = slice(a.out_flag, 1); }

    // load, entry i = first + 64 r + lane: all loads in flight together
    const int lane4 = lane * 4;
    int rem_in[kEPL], c_in[kEPL], gen_in[kEPL], bud_in[kEPL];
#pragma unroll
    for (int r = 0; r < kEPL; ++r) {
        rem_in[r] = __builtin_amdgcn_raw_buffer_load_b32(b_rem, lane4, (first + r * kWave) * 4, 0);
        c_in[r] = __builtin_amdgcn_raw_buffer_load_b32(b_prompt, lane4, (first + r * kWave) * 4, 0);
        gen_in[r] = __builtin_amdgcn_raw_buffer_load_b32(b_gen, lane4, (first + r * kWave) * 4, 0);
    }
    if (risk) {
#pragma unroll
        for (int r = 0; r < kEPL; ++r)
            bud_in[r] = __builtin_amdgcn_raw_buffer_load_b32(b_bud, lane4, (first + r * kWave) * 4, 0);
    }
    long long qsum = 0;
    if (Q + P > 0) {     // queued requests, and those routed since the status (feedback routing)
        const int* pp = a.pend_prompt + (size_t)g * kTab;
        const int* pl = a.pend_len + (size_t)g * kTab;
        const int listed = A + Q + min(in.pend, P);      // entries before those of the chunk
        int join_ctx = 0, join_len = 0;                  // lane j: the j-th request of the chunk that was sent here
        if (in.joins) {
            const bool mine = (in.joins >> lane) & 1ull;
            const int nth = __popcll(in.joins & ((1ull << lane) - 1ull));
            const int ctx0 = a.chunk_ctx0[min(lane, a.chunk_n - 1)], len = a.chunk_len[min(lane, a.chunk_n - 1)];
            // (the others send to the last lane, which nobody looks at unless every lane is `mine`)
            join_ctx = __builtin_amdgcn_ds_permute((mine ? nth : kWave - 1) * 4, ctx0);
            join_len = __builtin_amdgcn_ds_permute((mine ? nth : kWave - 1) * 4, len);
            if (mine && part == 0 && in.pend + nth < kTab) {
                a.pend_prompt[(size_t)g * kTab + in.pend + nth] = ctx0;
                a.pend_len[(size_t)g * kTab + in.pend + nth] = len;
            }
        }
#pragma unroll
        for (int r = 0; r < kEPL; ++r) {
            const int i = first + r * kWave + lane;
            int jc = 0, jl = 0;
            if (in.joins) {
                jc = __builtin_amdgcn_ds_bpermute((i - listed) * 4, join_ctx);
                jl = __builtin_amdgcn_ds_bpermute((i - listed) * 4, join_len);
            }
            if (i >= A && i < N) {
                const bool queued = i < A + Q;
                rem_in[r] = i >= listed ? jl : queued ? a.q_len[q0 + i - A] : pl[i - A - Q];
                c_in[r] = i >= listed ? jc : queued ? a.q_prompt[q0 + i - A] : pp[i - A - Q];
                qsum += c_in[r];
            }
        }
        qsum = wave_sum_i64(qsum);
    }

    // one sort word per entry = (remaining length << kIdxBits) | i; past the last entry all ones
    uint32_t key[kEPL];
    bool bad = false;
#pragma unroll
    for (int r = 0; r < kEPL; ++r) {
        const int i = first + r * kWave + lane;
        const int rem = min(max(rem_in[r], 0), a.max_len);
        bad |= rem != rem_in[r];
        key[r] = i < N ? ((uint32_t)rem << kIdxBits) | (uint32_t)i : 0xFFFFFFFFu;
        ctx[i] = c_in[r] + gen_in[r];          // (zero past the last entry: the loads returned zeros)
    }
    if (risk) {
#pragma unroll
        for (int r = 0; r < kEPL; ++r) stage[first + r * kWave + lane] = __int_as_float(bud_in[r]);
    }
    if (__ballot(bad)) status |= GR_DEV_LEN_CLAMPED;
    if (status && lane == 0) {
        atomicOr(&a.counters[0], status);
        if (risk && (status & GR_DEV_ENTRIES_DROPPED)) *a.unset = 1;
    }
    if (risk) {      // the instance of each running request, for the migration pass of a risk scan
        const __amdgpu_buffer_rsrc_t b_inst = slice(a.act_inst, 4);
#pragma unroll
        for (int r = 0; r < kEPL; ++r) __builtin_amdgcn_raw_buffer_store_b32(g, b_inst, lane4, (first + r * kWave) * 4, 0);
    }

    if constexpr (kSplit == 1) {
        bitonic_sort<kShortChain<kEPL>, kEPL>(key, lane);
        // the wave's own LDS writes above must be visible to its reads below
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        bitonic_sort_split<kEPL, kSplit>(key, lane, part, xch);     // (its barriers also publish the contexts)
    }

    // sorted position v = first + lane * kEPL + r; per lane the sums of R, c*R + tri(R), c
    int idx[kEPL], Ri[kEPL], ci[kEPL];
    const int mine = N - first - lane * kEPL;    // positions of this lane that hold an entry
    // an entry's terms of the three sums, as doubles (formed twice, here and below, rather than kept)
    const auto terms = [&](int r, double& Rd, double& cd, double& td, double& xe) {
        Rd = (double)Ri[r];
        cd = (double)ci[r];
        td = (double)(Ri[r] * (Ri[r] - 1) / 2);
        xe = fma(cd, Rd, td);
    };
    double yl = 0.0, xl = 0.0, cl = 0.0;
#pragma unroll
    for (int r = 0; r < kEPL; ++r) {
        idx[r] = (int)(key[r] & kIdxMask);
        Ri[r] = r < mine ? (int)(key[r] >> kIdxBits) : 0;
        // (a position without an entry carries index kCap - 1, an entry that does not exist either: zero)
        ci[r] = ctx[idx[r]];
    }
#pragma unroll
    for (int r = 0; r < kEPL; ++r) {
        double Rd, cd, td, xe;
        terms(r, Rd, cd, td, xe);
        yl += Rd; xl += xe; cl += cd;
    }
#pragma unroll
    for (int r = 0; r < kEPL; ++r) asm volatile("" : "+v"(Ri[r]), "+v"(ci[r]));   // (so that the terms are not kept in registers)
    const double yi = wave_incl_scan_f64(yl), xi = wave_incl_scan_f64(xl), pi = wave_incl_scan_f64(cl);
    double Ctot = readlane_f64(pi, kWave - 1);
    double Y = yi - yl, X = xi - xl, Pc = pi - cl;
    double qtot = (double)qsum;
    if constexpr (kSplit > 1) {      // the waves before this one, and everybody's total
        if (lane == kWave - 1) {
            sums[part * 4 + 0] = yi; sums[part * 4 + 1] = xi; sums[part * 4 + 2] = pi; sums[part * 4 + 3] = qtot;
        }
        __syncthreads();
        Ctot = 0.0; qtot = 0.0;
#pragma unroll
        for (int w = 0; w < kSplit; ++w) {
            const double yw = sums[w * 4 + 0], xw = sums[w * 4 + 1], pw = sums[w * 4 + 2];
            if (w < part) { Y += yw; X += xw; Pc += pw; }
            Ctot += pw;
            qtot += sums[w * 4 + 3];
        }
    }
    const double q = cc.delta * qtot;

    // with a blend, every estimate below is keep * (white-box value) + lam * (Eq. 2 with the smoothed status)
    const bool blended = a.lam != 0.0;
    const double keep = 1.0 - a.lam;
    const double bq = blended ? a.emaQ[g] : 0.0, bp = blended ? a.emaP[g] : 0.0, bd = blended ? a.emaD[g] : 0.0;

    // table entry v describes the segment after the v+1 shortest requests, n of them still running:
    //   E_g(L) = Gq + L * H + tri(L) * gamma * (n + 1)
    //   Gq = q + beta * Y + gamma * X,   H = alpha + beta * (n + 1) + gamma * S
    // and the request at position v finishes at q + alpha R + beta (Y + n R) + gamma (X + R S + n tri(R)).
    uint16_t tR[kEPL];
    float2 tGH[kEPL];
    float fin32[kEPL], bud[kEPL];
    unsigned late = 0;                           // bit r: the request at position r finishes after its budget
    if (risk) {
#pragma unroll
        for (int r = 0; r < kEPL; ++r) bud[r] = stage[idx[r]];
    }
    double n_here = (double)mine;                // requests still running from this position on, itself included
#pragma unroll
    for (int r = 0; r < kEPL; ++r) {
        double Rd, cd, td, xe;
        terms(r, Rd, cd, td, xe);
        Y += Rd; X += xe; Pc += cd;
        const double n_after = n_here - 1.0, S_next = Ctot - Pc;
        double Gq = fma(cc.gamma, X, fma(cc.beta, Y, q));
        double Hs = fma(cc.gamma, S_next, fma(cc.beta, n_here, cc.alpha));
        double fin = fma(cc.gamma, fma(n_after, td, fma(Rd, S_next, X)),
                         fma(cc.beta, fma(n_after, Rd, Y), fma(cc.alpha, Rd, q)));
        n_here = n_after;
        if (blended) {
            Gq = keep * Gq + a.lam * bq;
            Hs = keep * Hs + a.lam * bd;
            // black-box finish: d per remaining token; a queued request also waits and prefills
            fin = keep * fin + a.lam * (idx[r] < A ? bd * Rd : (bq + bp * cd) + bd * Rd);
        }
        if constexpr (kSums) {      // of the segment after this position
            const size_t at = (size_t)g * (kTab + 1) + first + lane * kEPL + r + 1;
            offer->sums_yx[at] = make_double2(Y, X);
            offer->sums_c[at] = Pc;
        }
        fin32[r] = (float)fin;
        if (risk) late |= (unsigned)(fin > (double)bud[r]) << r;     // decided in double precision
        tR[r] = r < mine ? (uint16_t)Ri[r] : (uint16_t)0xFFFFu;
        tGH[r] = make_float2((float)Gq, (float)Hs);
    }
    // Finish times and flags go back to entry order through LDS: the lane that read an entry's budget
    // from its slot is the one that writes its finish time there.  (A position without an entry
    // carries index kCap - 1 >= N: a slot past the slice, of which nothing is stored.)
    if constexpr (!kQuiet) {
#pragma unroll
        for (int r = 0; r < kEPL; ++r) stage[idx[r]] = fin32[r];
    }
    if (risk) {
#pragma unroll
        for (int r = 0; r < kEPL; ++r) flag_lds[idx[r]] = (uint8_t)((late >> r) & 1u);
        // the lengths of flagged requests, for the migration pass (a byte each; of equal neighbours in
        // the sorted order one is enough), and how many there are
        unsigned mig = 0;
#pragma unroll
        for (int r = 0; r < kEPL; ++r) mig |= (unsigned)(r < mine && idx[r] < A) << r;
        mig &= late;
        if (a.seen) {
#pragma unroll
            for (int r = 0; r < kEPL; ++r) {
                const bool again = r + 1 < kEPL && ((mig >> (r + 1)) & 1u) && Ri[r + 1 < kEPL ? r + 1 : r] == Ri[r];
                if (((mig >> r) & 1u) && !again) a.seen[Ri[r]] = 1;
            }
        }
        const int n_late = wave_incl_scan_i32(__popc(mig));
        if (lane == kWave - 1) a.late_cnt[part * a.n_inst + g] = n_late;
    }
    if constexpr (!kQuiet) {
        if constexpr (kSplit == 1) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        } else {
            __syncthreads();
        }
#pragma unroll
        for (int r = 0; r < kEPL; ++r)
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(stage[first + r * kWave + lane]), b_fin, lane4,
                                                  (first + r * kWave) * 4, 0);
        if (risk) {
#pragma unroll
            for (int r = 0; r < kEPL; ++r)
                __builtin_amdgcn_raw_buffer_store_b8(flag_lds[first + r * kWave + lane], b_flag, lane, first + r * kWave, 0);
        }
        if (Q > 0 && a.out_q_finish) {
#pragma unroll
            for (int r = 0; r < kEPL; ++r)
                if (r < mine && idx[r] >= A && idx[r] < A + Q) a.out_q_finish[q0 + idx[r] - A] = fin32[r];
        }
    }
    {
        uint16_t* dstR = a.tabR + (size_t)g * kTab + first + lane * kEPL;
        float2* dstGH = a.tabGH + gh_at(g, 1, kTab) + first + lane * kEPL;
        if constexpr (kEPL >= 8) {
#pragma unroll
            for (int r = 0; r < kEPL; r += 8) {
                uint4 w;
                w.x = tR[r] | ((uint32_t)tR[r + 1] << 16); w.y = tR[r + 2] | ((uint32_t)tR[r + 3] << 16);
                w.z = tR[r + 4] | ((uint32_t)tR[r + 5] << 16); w.w = tR[r + 6] | ((uint32_t)tR[r + 7] << 16);
                *reinterpret_cast<uint4*>(dstR + r) = w;
            }
        } else {
#pragma unroll
            for (int r = 0; r < kEPL; ++r) dstR[r] = tR[r];
        }
        if constexpr (kEPL >= 2) {
#pragma unroll
            for (int r = 0; r < kEPL; r += 2)
                *reinterpret_cast<float4*>(dstGH + r) = make_float4(tGH[r].x, tGH[r].y, tGH[r + 1].x, tGH[r + 1].y);
        } else {
            dstGH[0] = tGH[0];
        }
        store_splitter<kTab>(a.tabS, g, first + lane * kEPL + kEPL - 1, tR[kEPL - 1]);
        if constexpr (kTab > kCap) {      // the lengths past these words: none, 16 bytes at a time
            constexpr int kStep = kTab / split_count(kTab);
            const uint4 none = make_uint4(~0u, ~0u, ~0u, ~0u);
            for (int v = kCap + (part * kWave + lane) * 8; v < kTab; v += kSplit * kWave * 8) {
                *reinterpret_cast<uint4*>(a.tabR + (size_t)g * kTab + v) = none;
                if ((v + 8) % kStep == 0) a.tabS[(size_t)g * split_count(kTab) + v / kStep] = (uint16_t)0xFFFFu;
            }
        }
    }
    // segment 0, the next decode step, what a pair needs of the instance
    const auto own_figures = [&](double& Gq0, double& H0, double& d, float4& K) {
        Gq0 = q; H0 = fma(cc.gamma, Ctot, fma(cc.beta, (double)(N + 1), cc.alpha));
        if (blended) { Gq0 = keep * Gq0 + a.lam * bq; H0 = keep * H0 + a.lam * bd; }
        d = fma(cc.gamma, Ctot, fma(cc.beta, (double)N, cc.alpha));
        if (blended) d = keep * d + a.lam * bd;
        K = inst_coef(a, cc, bp, N);
    };
    double Gq0, H0, d;
    float4 K;
    if constexpr (kOffer) own_figures(Gq0, H0, d, K);
    if (lane == 0 && part == 0) {
        if constexpr (kSums) {
            offer->sums_yx[(size_t)g * (kTab + 1)] = make_double2(0.0, 0.0);
            offer->sums_c[(size_t)g * (kTab + 1)] = 0.0;
            offer->base[g] = FeedBase{Ctot, qtot, N, in.pend + (int)__popcll(in.joins), min(kTab, a.max_entries - A - Q), 0};
        }
        if constexpr (!kOffer) own_figures(Gq0, H0, d, K);
        a.tabGH[gh_at(g, 0, kTab)] = make_float2((float)Gq0, (float)H0);
        a.instK[g] = K;
        a.pend_touched[g] = 0;
        if (!a.use_pending) a.pend_cnt[g] = 0;
        else if (in.joins) a.pend_cnt[g] = in.pend + __popcll(in.joins);     // (every wave has read it: the sort's barriers)
        a.hD[g] = d;
        a.slot_key[kQuiet ? slot : a.slot_of[g]] = falling_bits(d);
        if (a.out_d) a.out_d[g] = d;
    }
    if constexpr (kOffer) {
        // the new table in LDS, where the contexts and the sort's exchange were (the last reads of both
        // are before the barrier of the totals)
        static_assert(kSplit > 1 && kQuiet && 2 * (kCap + 1) <= kInstWords);
        float2* const gh = reinterpret_cast<float2*>(smem);
        uint16_t* const R = reinterpret_cast<uint16_t*>(xch);
#pragma unroll
        for (int r = 0; r < kEPL; ++r) {
            gh[1 + first + lane * kEPL + r] = tGH[r];
            R[first + lane * kEPL + r] = tR[r];
        }
        if (lane == 0 && part == 0) gh[0] = make_float2((float)Gq0, (float)H0);
        __syncthreads();
        if (part == 0) {
            int k = 0;      // entries that are no longer than the request
#pragma unroll
            for (int step = kCap / 2; step > 0; step /= 2) k += (int)R[k + step - 1] <= offer->L ? step : 0;
            k += (int)R[k] <= offer->L;
            offer->T = latency_at(offer->c0, offer->L, K, gh[k], k);
            offer->key = falling_bits(d);
        }
    }
}

// The instance's slices and the lengths of its lists, from the caller's offsets.  kListed: its list may have grown beyond the
// table without anybody having said so (requests that were added to sums).
template <int kTab, bool kListed = false>
__device__ __forceinline__ void clamp_instance(const BuildArgs& a, InstanceIn& in, int a_begin, int a_end, int q_begin, int q_end, int pend)
{
    // offsets are clamped into the arrays, so broken CSR data cannot index outside them
    in.a0 = (int)min((int64_t)max(a_begin, 0), a.n_active);
    in.q0 = (int)min((int64_t)max(q_begin, 0), a.n_queued);
    in.A = (int)max(min((int64_t)a_end, a.n_active) - in.a0, (int64_t)0);
    in.Q = (int)max(min((int64_t)q_end, a.n_queued) - in.q0, (int64_t)0);
    in.status = 0;
    if (in.A > a.max_entries) { in.A = a.max_entries; in.status |= GR_DEV_ENTRIES_DROPPED; }
    if (in.Q > a.max_entries - in.A) { in.Q = a.max_entries - in.A; in.status |= GR_DEV_ENTRIES_DROPPED; }
    in.pend = pend;
    in.P = in.pend + __popcll(in.joins);
    if (in.P > kTab) { in.P = kTab; if (kListed || in.joins) in.status |= GR_DEV_ENTRIES_DROPPED; }
    if (in.P > a.max_entries - in.A - in.Q) { in.P = a.max_entries - in.A - in.Q; in.status |= GR_DEV_ENTRIES_DROPPED; }
}

// A handle's tables have room for the most an instance may hold, which can be several times what
// it does hold: with kFit an instance that a half or a quarter of the sort words would do for takes
// those (see fit_words).  kQuiet: a rebuild of feedback routing, whose finish times nobody asks for and of
// which most instances take no part: 32 rounds of 64 requests on 256 instances 451 us with the plain
// build and reads in the order of their use, 400 this way.
template <int kEPL, int kSplit, bool kFit, bool kQuiet>
__global__ __launch_bounds__(kSplit == 1 ? kBlock : kWave * kSplit, (kEPL <= 8 ? 4 : 1)) void k_build_lean(BuildArgs a)
{
    if constexpr (kSplit > 1) fetch_args<BuildArgs>();
    extern __shared__ uint32_t smem[];
    constexpr int kTab = kWave * kEPL * kSplit;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    InstanceIn in;
    in.g = kSplit == 1 ? blockIdx.x * kBuildWaves + wave : blockIdx.x;   // wave-uniform: what follows is scalar
    const int g = in.g;
    if (g >= a.n_inst) return;
    const int a_begin = a.act_off[g], a_end = a.act_off[g + 1], q_begin = a.q_off[g], q_end = a.q_off[g + 1];
    const int pend = a.use_pending ? a.pend_cnt[g] : 0;
    if constexpr (kQuiet) asm volatile("" :: "s"(a_begin), "s"(a_end), "s"(q_begin), "s"(q_end), "s"(pend));   // (not after the branch below)
    // feedback routing: an instance that has been given nothing since its table was built keeps it
    // (the mark is cleared at the very end, when every wave of the instance has read it)
    in.joins = 0;
    if (a.chunk_n) {
        const int lane = lane_id();
        in.joins = __ballot(lane < a.chunk_n && a.chunk_inst[min(lane, a.chunk_n - 1)] == g);
        if (a.only_touched && !in.joins) return;
    } else if (a.only_touched && a.pend_touched[g] == 0) {
        return;
    }
    clamp_instance<kTab>(a, in, a_begin, a_end, q_begin, q_end, pend);
    const int N = in.A + in.Q + in.P;
    if constexpr (kFit) {
        if constexpr (kEPL >= 4)
            if (N <= kTab / 4) return build_instance<kEPL / 4, kSplit, kTab, kQuiet>(a, in, wave, smem);
        if constexpr (kEPL >= 2)
            if (N <= kTab / 2) return build_instance<kEPL / 2, kSplit, kTab, kQuiet>(a, in, wave, smem);
    }
    build_instance<kEPL, kSplit, kTab, kQuiet>(a, in, wave, smem);
}

// Feedback routing, a launch per decision round (chunks of up to kWave requests; a workgroup per instance, all
// of whose waves share it).  Launch k decides the chunk before it from what every instance has offered (every
// workgroup for itself: a lane per request, the waves share the instances), takes in what was sent to the instance, and
// offers for the next chunk: each request's latency here, whether its deadline is met, and d_g.
// The launches themselves are the wait of one round for the other.  What was sent to an instance is taken in by building its
// table anew.  (For few rounds, and for many requests to an instance and round: see in_one_launch.  Else the tables are all built once at
// the start, with the sums behind them, kSums, and those that have been given any at the end.)
//
// What bounds it is the chain of a round: the offers (64 requests x 256 instances are 64 KB for every workgroup, from
// L2), the choice, then the rebuild, whose table is still in LDS when the next requests are looked up in it.  A round was
// two launches, a scoring and a rebuild, each with its own start and its own reads of what the other had just written:
// 256 instances x 512, 32 rounds of 64, with the status build 400 us, this way 329.  An instance only finds out
// whether it is chosen itself: looking for everybody's choice took 17 us a round instead of 10.5 (8 bytes of every instance
// as scalars, one after the other), and 12.3 with those read a lane each.
struct FeedArgs {
    BuildArgs b;                        // with the chunk that is decided here
    const int *next_ctx0, *next_len, *next_exclude;     // the chunk to offer for
    const float* next_budget;
    int next_n;
    const uint32_t* T_in;               // [M][kWave], [M], [M], see gr_fleet
    const unsigned long long *met_in, *key_in;
    uint32_t* T_out;
    unsigned long long *met_out, *key_out;
    const float* budget;
    int* out_inst;
    float* out_slack;
    uint8_t* out_fallback;
};

// The launches before and behind k_feedback_rounds, which adds what comes to the tables' sums (see gr_fleet).
struct FeedSumsArgs {
    FeedArgs f;
    int move;
    double2* sums_yx;
    double* sums_c;
    FeedBase* base;
    FeedWords words;      // n = 0: nobody exchanges any
};

// What such a launch does to the tables: nothing; all of them are built; all that have been given requests since are.
enum FeedMove { kFeedNone = 0, kFeedAll, kFeedTouched };

// Segment and latency of a request in the instance's table as it stands, in two steps as k_direct.
template <int kTab>
__device__ __forceinline__ int segment_in_table(const BuildArgs& a, int g, int L)
{
    constexpr int kS = split_count(kTab), kStride = kTab / kS;
    const uint4* __restrict__ S = reinterpret_cast<const uint4*>(a.tabS + (size_t)g * kS);
    int b = 0;
#pragma unroll
    for (int i = 0; i < kS / 8; ++i) b += count_upto(S[i], (uint32_t)L);
    int k = min(b, kS - 1) * kStride;
    const uint4* __restrict__ R = reinterpret_cast<const uint4*>(a.tabR + (size_t)g * kTab + k);
    uint4 w[kStride / 8];
#pragma unroll
    for (int i = 0; i < kStride / 8; ++i) w[i] = R[i];
#pragma unroll
    for (int i = 0; i < kStride / 8; ++i) k += count_upto(w[i], (uint32_t)L);
    return k;
}

template <int kTab>
__device__ __forceinline__ float latency_in_table(const BuildArgs& a, int g, float c0, int L)
{
    const int k = segment_in_table<kTab>(a, g, L);
    return latency_at(c0, L, a.instK[g], a.tabGH[gh_at(g, k, kTab)], k);
}

// The bits of a wave's lanes together (the steps of wave_incl_scan_i32).
__device__ __forceinline__ uint32_t wave_or_u32(uint32_t v)
{
    const auto step = [&](auto ctrl, auto rows) {
        v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, decltype(rows)::value, 0xf, false);
    };
    using std::integral_constant;
    step(integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});
    step(integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});
    step(integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});
    step(integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});
    step(integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});
    step(integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});
    return (uint32_t)__builtin_amdgcn_readlane((int)v, kWave - 1);
}

__device__ __forceinline__ unsigned long long wave_or_u64(unsigned long long v)
{
    return ((unsigned long long)wave_or_u32((uint32_t)(v >> 32)) << 32) | wave_or_u32((uint32_t)v);
}

template <int kEPL, int kSplit, bool kSums>
__global__ __launch_bounds__(kWave * kSplit, (kEPL <= 8 ? 4 : 1)) void k_feedback(std::conditional_t<kSums, FeedSumsArgs, FeedArgs> args)
{
    extern __shared__ uint32_t smem[];
    __shared__ uint32_t share[kSplit][kWave];
    __shared__ unsigned long long met_by[kSplit][2];
    constexpr int kTab = kWave * kEPL * kSplit;
    fetch_args<decltype(args)>();
    const auto of = [&]() -> const FeedArgs& {
        if constexpr (kSums) return args.f;
        else return args;
    };
    const FeedArgs& f = of();
    const BuildArgs& a = f.b;
    int move = kFeedNone;
    if constexpr (kSums) move = args.move;
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    InstanceIn in;
    in.g = blockIdx.x;
    in.joins = 0;
    const int g = in.g, M = a.n_inst;
    const int a_begin = a.act_off[g], a_end = a.act_off[g + 1], q_begin = a.q_off[g], q_end = a.q_off[g + 1];
    const int pend = a.pend_cnt[g];
    const int touched = move == kFeedTouched ? a.pend_touched[g] : 0;
    Offer offer{};
    if constexpr (kSums) {
        offer.sums_yx = args.sums_yx; offer.sums_c = args.sums_c; offer.base = args.base;
        if (move == kFeedAll)
            for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < args.words.n; i += gridDim.x * blockDim.x) args.words.least[i] = 0;
    }
    float D = 0.f;
    int ex = -1;
    if (f.next_n && wave == 0) {
        const int j = min(lane, f.next_n - 1);
        offer.L = min(max(f.next_len[j], 0), a.max_len);
        offer.c0 = (float)f.next_ctx0[j];
        D = f.next_budget[j];
        if (f.next_exclude) ex = f.next_exclude[j];
    }

    if (a.chunk_n) {
        // Alg. 1 for the instance itself, lane = request: where a deadline can be met, it is met here and by nobody
        // more capable; else nobody's latency is less, or as little at a lower index
        const uint32_t own = f.T_in[(size_t)g * kWave + lane];
        const unsigned long long own_key = f.key_in[g], own_met = f.met_in[g];
        unsigned long long any = 0, above = 0;         // requests whose deadline is met by somebody, by somebody more capable
        for (int h = threadIdx.x; h < M; h += kSplit * kWave) {
            const unsigned long long met = f.met_in[h], key = f.key_in[h];
            any |= met;
            above |= key < own_key || (key == own_key && h < g) ? met : 0ull;
        }
        // the waves share the latencies; those at lower indices count as one less, so that `own` has to be below them
        const int per = (M + kSplit - 1) / kSplit, h0 = wave * per, n_here = min(per, M - h0);
        uint32_t least = ~0u;
        if (n_here > 0) {
            constexpr int kAhead = 16;
            const uint32_t* __restrict__ row = f.T_in + (size_t)h0 * kWave + lane;
            const int end = n_here * kWave, below = (g - h0) * kWave;
            uint32_t T[kAhead], T_next[kAhead];
#pragma unroll
            for (int i = 0; i < kAhead; ++i) T[i] = row[min(i * kWave, end - kWave)];       // (a repeat of the last one changes nothing)
            for (int at = 0; at < end; at += kAhead * kWave) {
                if (at + kAhead * kWave < end) {
#pragma unroll
                    for (int i = 0; i < kAhead; ++i) T_next[i] = row[min(at + (kAhead + i) * kWave, end - kWave)];
                }
#pragma unroll
                for (int i = 0; i < kAhead; ++i) least = min(least, T[i] - (min(at + i * kWave, end - kWave) < below ? 1u : 0u));
#pragma unroll
                for (int i = 0; i < kAhead; ++i) T[i] = T_next[i];
            }
        }
        any = wave_or_u64(any);
        above = wave_or_u64(above);
        share[wave][lane] = least;
        if (lane == 0) { met_by[wave][0] = any; met_by[wave][1] = above; }
        __syncthreads();
        any = above = 0;
#pragma unroll
        for (int w = 0; w < kSplit; ++w) {
            least = min(least, share[w][lane]);
            any |= met_by[w][0];
            above |= met_by[w][1];
        }
        const bool live = lane < a.chunk_n, served = (any >> lane) & 1ull;
        const bool mine = live && (served ? ((own_met & ~above) >> lane) & 1ull : own != ~0u && own <= least);
        if (wave == 0 && mine) {
            f.out_inst[lane] = g;
            f.out_slack[lane] = f.budget[lane] - from_ordered_bits(own);
            if (f.out_fallback) f.out_fallback[lane] = !served;
        }
        if (g == 0 && wave == 0 && live && !served && least == ~0u) {      // nobody is allowed
            f.out_inst[lane] = -1;
            f.out_slack[lane] = 0.f;
            if (f.out_fallback) f.out_fallback[lane] = 1;
        }
        in.joins = __ballot(mine);
    }

    const bool rebuild = !kSums ? a.chunk_n && (in.joins || !a.only_touched)
                         : move == kFeedTouched ? in.joins || touched : move == kFeedAll;
    if (rebuild) {
        clamp_instance<kTab, kSums>(a, in, a_begin, a_end, q_begin, q_end, pend);
        const int N = in.A + in.Q + in.P;
        bool built = false;
        if constexpr (kEPL >= 4)
            if (N <= kTab / 4) { build_instance<kEPL / 4, kSplit, kTab, true, true, kSums>(a, in, wave, smem, &offer); built = true; }
        if constexpr (kEPL >= 2)
            if (!built && N <= kTab / 2) { build_instance<kEPL / 2, kSplit, kTab, true, true, kSums>(a, in, wave, smem, &offer); built = true; }
        if (!built) build_instance<kEPL, kSplit, kTab, true, true, kSums>(a, in, wave, smem, &offer);
    } else if (f.next_n && wave == 0) {
        offer.T = latency_in_table<kTab>(a, g, offer.c0, offer.L);
        offer.key = falling_bits(a.hD[g]);
    }
    if (!f.next_n || wave != 0) return;
    const float Dc = D > FLT_MAX ? FLT_MAX : D;
    const bool ok = g != ex;      // (batches of this size take infinite latencies for latencies, see pairs_finite)
    const unsigned long long met = __ballot(ok && offer.T <= Dc);
    // (the least and the largest integer are NaNs with every bit set; here nothing is below the one, and the other is not allowed)
    f.T_out[(size_t)g * kWave + lane] = ok ? min(max(ordered_bits(offer.T), 1u), ~0u - 1u) : ~0u;
    if (lane == 0) { f.met_out[g] = met; f.key_out[g] = offer.key; }
}

// Feedback routing, all rounds in one launch.  A launch for every round costs its start, its arguments and cold reads, 9 us of which
// the round itself is a third; here the workgroups go from round to round by words that they leave for each other in memory: each
// carries its round in its lower half, is written and read past the caches that are not common (relaxed, agent scope), and is valid by itself,
// so nothing is fenced or flushed.  32 to 64 workgroups see each other's words 1.55 us after they are written, 128 2.2 us, 256 3.6 us
// (512 bytes each; on one XCD or on all of them alike): hence four instances to a workgroup, a wave each.
//
// A round.  Each wave has left d_g and the met deadlines of its instance, the workgroup the least latency over its four, per
// request (with the instance, so that the least word is the answer).  While those are on their way the wave gathers what its next
// offers are added up from.  Then every workgroup takes the least words of all for itself, each wave finds the
// requests that its own instance is chosen for, puts them on its list, adds them to the sums and offers for the next chunk.  Nothing is built
// anew meanwhile: what has come is held in LDS, as terms of the sums, and kFeedBlock of them are put away sorted, with their prefix sums,
// as a block that is searched like the table itself.
//
// A lone wave's instructions are eight cycles each, so their number is what counts next to the exchange: other waves wait for the words,
// so that the look at them is not behind the gathering (5.4 us a round instead of 6.5), and new requests are terms in LDS, written by
// their lanes (as lanes read off one by one 5.4, now 4.1).  A form that built long lists' tables anew on the way spilled 150 registers: 13.
//
// Every wait ends.  A workgroup is counted as it starts (FeedWords::gate), and looks until all have been, which takes no longer than its first
// offers.  Where one has looked in vain (compute units full of others' work, several such
// launches of which each has a part of the chip) it closes the gate.  Who comes later returns at once, and those counted until then
// share the instances, several to a wave in turn; nothing has been changed up to there, and they use words of their own.  So all that
// anybody waits for is running.  Four streams of 512 instances each, 2 048 requests, 64 a round, which do not fit side by side: 141 to 174 us a
// call (a launch per round 182; where a lone workgroup did what the others had given up 95 to 485).  By how many workgroups: 256/64, 2 048
// requests 160 us by all 64, 326 by 32, 512 by 16, 6 400 by one; 512/64, 2 000 186 by all 128, 354 by 64, 575 by 32.
// Two sets of words in turn are enough: a workgroup writes a round's when it has seen all of the round before, whose writers had read
// all of the one before that.
//
// 256 instances x 512, 32 rounds of 64, with the status build: 309 us with a launch for each, this way 160: a round is 4.1 us, of which the words
// take 0.9, gathering with two blocks 1.3, the choice 0.5 to 0.9, adding and offering 0.6.
constexpr uint32_t kFeedCount = 0xFFFFu, kFeedClosed = 1u << 31;      // of the gate: workgroups that have started; closed, and in between how many had then
constexpr int kFeedShareAt = 16;
constexpr int kFeedTagBits = 22, kFeedInstAt = kFeedTagBits;      // of a least word, below the latency: the round, the instance
static_assert(kFeedInst <= 1 << (32 - kFeedInstAt));
constexpr int kFeedMostRounds = 1 << (kFeedTagBits - 1);      // of one launch
constexpr int kFeedPollsMore = 1 << 21;   // looks at the words of later rounds, which are there in microseconds
constexpr int kFeedWaves = 4;             // instances of a workgroup
constexpr int kFeedBlock = 32;            // requests that are put away together
constexpr int kFeedHeld = kFeedBlock + kWave;      // requests of an instance that are held: less than a block, and a chunk

struct FeedRoundsArgs {
    BuildArgs b;
    const int *ctx0, *pred_len, *exclude;
    const float* budget;
    int* out_inst;
    float* out_slack;
    uint8_t* out_fallback;
    int64_t n;
    int chunk, first, rounds;      // requests of a round, the first round here, rounds in all
    int polls;                     // looks at the gate, about a microsecond each, before a workgroup closes it, if all but itself were here
    int team;                      // workgroups that may share the work (see gr_set_feedback_team)
    const double2* sums_yx;
    const double* sums_c;
    const FeedBase* base;
    FeedBlocks blocks;
    FeedWords words;
    uint32_t* T;                   // [M][kWave] latencies offered, where a wave has several instances
};

__device__ __forceinline__ unsigned long long peek(const unsigned long long* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void leave(unsigned long long* p, unsigned long long v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// An instance's sorted lengths in LDS, with the last of every eight and of every 64: #{R_i <= L} is three short steps.  And those
// of its blocks.
template <int kTab>
struct FeedLengths {
    uint4 all[kTab / 8], eighths[kTab / 64], splits[(kTab / 64 + 7) / 8], blocks[kTab / 8];

    __device__ __forceinline__ void load(const uint16_t* __restrict__ R)
    {
        uint16_t* const e = reinterpret_cast<uint16_t*>(eighths);
        uint16_t* const s = reinterpret_cast<uint16_t*>(splits);
        const int lane = lane_id();
        if (kTab / 64 < 8 && lane < 8) s[lane] = 0xFFFF;
#pragma unroll
        for (int i = lane; i < kTab / 8; i += kWave) {
            const uint4 w = reinterpret_cast<const uint4*>(R)[i];
            all[i] = w;
            e[i] = (uint16_t)(w.w >> 16);
            if (i % 8 == 7) s[i / 8] = (uint16_t)(w.w >> 16);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }

    __device__ __forceinline__ int upto(uint32_t L) const
    {
        uint32_t c = 0;
#pragma unroll
        for (int i = 0; i < (kTab / 64 + 7) / 8; ++i) c += count_upto2(splits[i], L);
        const int b = min(both_counts(c), kTab / 64 - 1);
        const int e = 8 * b + min(count_upto(eighths[b], L), 7);
        return 8 * e + count_upto(all[e], L);
    }
};

// What the waves of a workgroup share, in LDS: arrays of their own (as members of one object, each write was in the way of the reads of
// the others, 0.13 us a round).
struct FeedState {
    int over, ticket, team;           // a wait was in vain; see pass_gate
};
template <int kTab>
struct FeedShared {
    FeedLengths<kTab>* lengths;                                // [kFeedWaves]
    unsigned long long (*least)[kWave], (*offer)[kWave], *met; // [kFeedWaves]
    double4 (*held)[kFeedHeld];       // [kFeedWaves] R, c*R + tri(R), the context
    ulonglong2* infos;                // [kFeedInst] met deadlines and d_g (as an integer that falls with it) of every instance
    FeedState& state;
};

__device__ __forceinline__ uint32_t gate_of(const FeedWords& words)
{
    return __hip_atomic_load(words.gate, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Counts this workgroup, one of W, and waits for the others: how many share the work, and the how manieth of them this is (-1: come too late).
__device__ inline int2 pass_gate(const FeedWords& words, int W, int polls)
{
    uint32_t v = __hip_atomic_fetch_add(words.gate, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int ticket = v & kFeedClosed ? -1 : (int)(v & kFeedCount);
    v += v & kFeedClosed ? 0u : 1u;
    for (int64_t looks = 0; !(v & kFeedClosed); ++looks) {
        const int here = (int)(v & kFeedCount);
        if (here == W) return make_int2(W, ticket);
        if (looks * here < (int64_t)polls * W) { v = gate_of(words); continue; }      // (the fewer are here, the more is to be gained by those to come)
        const uint32_t closed = kFeedClosed | (uint32_t)here << kFeedShareAt | (uint32_t)here;
        if (__hip_atomic_compare_exchange_strong(words.gate, &v, closed, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) v = closed;
    }
    return make_int2((int)(v >> kFeedShareAt & (kFeedClosed - 1u) >> kFeedShareAt), ticket);
}

// The rounds by W workgroups, of which this is the w-th.  kPart: by fewer than have an instance for every wave.  Otherwise nothing is done where not
// all have come in time.
template <int kTab, bool kPart>
__device__ __forceinline__ void feedback_rounds(const FeedRoundsArgs& f, const FeedShared<kTab>& sh, const int W, const int w)
{
    constexpr int kAhead = 16;
    static_assert(kFeedWaves * kFeedWaves == 16 && kAhead * 16 == kFeedWaves * kWave, "a wave's share of the workgroups and of their instances is read together");
    const BuildArgs& a = f.b;
    const int lane = lane_id(), both = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), wave = both % kFeedWaves;
    const bool reader = both >= kFeedWaves;      // these wait for the words of all, the others have the instances
    const int M = a.n_inst;
    const FeedWords words = f.words.of(kPart, M);
    const auto inst_of = [&](int u) { return (u * W + w) * kFeedWaves + wave; };
    const auto each_inst = [&](auto turn) {
        if constexpr (kPart) { for (int u = 0; !reader && inst_of(u) < M; ++u) turn(u); }
        else if (!reader && inst_of(0) < M) turn(0);
    };
    FeedLengths<kTab>& lengths = sh.lengths[wave];
    const bool blended = a.lam != 0.0;
    const double keep = 1.0 - a.lam;

    // the requests of a round, a lane each
    struct Requests { int n, ctx0, length, ex; float D; };
    const auto requests = [&](int round) {
        Requests q;
        const int64_t at = (int64_t)round * f.chunk;
        q.n = (int)min(f.n - at, (int64_t)f.chunk);
        const int64_t i = at + min(lane, q.n - 1);
        q.ctx0 = f.ctx0[i]; q.length = f.pred_len[i]; q.D = f.budget[i];
        q.ex = f.exclude ? f.exclude[i] : -1;
        return q;
    };
    const auto clamped = [&](int length) { return min(max(length, 0), a.max_len); };

    // The instance at hand: its table's sums, and what has come since that was built: whole blocks in memory, the
    // others held in LDS.
    int g = 0, pend = 0, room = 0, since = 0, away = 0;      // requests on its list, those that count (up to its room), those put away
    FeedBase base{};
    ClassCoef cc{};
    double bq = 0.0, bp = 0.0, bd = 0.0;
    double since_ctx = 0.0;
    double4* const held = sh.held[wave];
    const auto block_at = [&](int b) { return (size_t)g * kTab + b * kFeedBlock; };
    const auto settled = [&]() {      // (the wave's own words in LDS)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    const auto terms = [&](int ctx, int length) {
        const int R = clamped(length);
        const double Rd = (double)R, cd = (double)ctx;
        return make_double4(Rd, fma(cd, Rd, (double)(R * (R - 1) / 2)), cd, 0.0);
    };
    const auto enter = [&](int inst) {
        g = inst;
        base = f.base[g];
        cc = a.cls[a.inst_class[g]];
        if (blended) { bq = a.emaQ[g]; bp = a.emaP[g]; bd = a.emaD[g]; }
        pend = a.pend_cnt[g];
        room = max(base.room - base.listed, 0);
        since = min(max(pend - base.listed, 0), room);
        away = since / kFeedBlock * kFeedBlock;
        lengths.load(a.tabR + (size_t)g * kTab);
        const size_t at = (size_t)g * kTab + min(base.listed + away + lane, kTab - 1);
        const double4 e = terms(a.pend_prompt[at], a.pend_len[at]);
        if (lane < since - away) held[lane] = e;
        since_ctx = readlane_f64(wave_incl_scan_f64(lane < since - away ? e.z : 0.0), kWave - 1);
        for (int b = 0; b < away / kFeedBlock; ++b) since_ctx += f.blocks.c[block_at(b) + kFeedBlock - 1];
        for (int i = lane; i < away / 8; i += kWave) lengths.blocks[i] = reinterpret_cast<const uint4*>(f.blocks.R + block_at(0))[i];
        settled();
    };
    // The first kFeedBlock of those held put away: their lengths sorted, and the sums up to each.
    const auto put_away = [&]() {
        uint32_t key[1] = {((uint32_t)(int)held[lane].x << 6) | (uint32_t)lane};
        bitonic_levels<true, 1, 2, kFeedBlock>(key, lane, lane << 2);
        const double4 e = held[key[0] & 63u];
        const double y = wave_incl_scan_f64(e.x), x = wave_incl_scan_f64(e.y), c = wave_incl_scan_f64(e.z);
        if (lane < kFeedBlock) {
            const size_t at = block_at(away / kFeedBlock) + lane;
            reinterpret_cast<uint16_t*>(lengths.blocks)[away + lane] = (uint16_t)(key[0] >> 6);
            if (kPart) f.blocks.R[at] = (uint16_t)(key[0] >> 6);
            f.blocks.yx[at] = make_double2(y, x);
            f.blocks.c[at] = c;
        }
        const double4 left = held[kFeedBlock + lane];      // (what is left moves down)
        settled();
        held[lane] = left;
        away += kFeedBlock;
        settled();
    };
    // What the offers for `q` are added up from, with all that has come so far.  Every sum is one of integers below 2^53, so the order
    // does not matter.
    struct Gathered { double y, x, pc; int k; };
    const auto add_held = [&](Gathered& G, int from, int to, double L) {
        for (int i = from; i < to; i += 4) {      // (those behind the last one: not read for what they are)
            double4 e[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) e[t] = held[min(i + t, kFeedHeld - 1)];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const bool left = i + t < to && e[t].x <= L;
                G.y += left ? e[t].x : 0.0; G.x += left ? e[t].y : 0.0; G.pc += left ? e[t].z : 0.0;
                G.k += left;
            }
        }
    };
    const auto gather = [&](const Requests& q) {
        Gathered G;
        const uint32_t L = (uint32_t)clamped(q.length);
        constexpr int kTogether = 4, kWords = kFeedBlock / 8;      // blocks side by side, on their way with the table's own segment
        const int blocks = away / kFeedBlock;
        double2 yx[kTogether];
        double c[kTogether];
        int n[kTogether];
        const auto read = [&](int b0) {
            uint4 R[kTogether][kWords];
#pragma unroll
            for (int t = 0; t < kTogether; ++t)
#pragma unroll
                for (int i = 0; i < kWords; ++i) R[t][i] = lengths.blocks[min(b0 + t, blocks - 1) * kWords + i];
#pragma unroll
            for (int t = 0; t < kTogether; ++t) {
                uint32_t c2 = 0;
#pragma unroll
                for (int i = 0; i < kWords; ++i) c2 += count_upto2(R[t][i], L);
                n[t] = b0 + t < blocks ? both_counts(c2) : 0;
                const size_t last = block_at(min(b0 + t, blocks - 1)) + max(n[t] - 1, 0);
                yx[t] = f.blocks.yx[last];
                c[t] = f.blocks.c[last];
            }
        };
        const auto sum = [&]() {
#pragma unroll
            for (int t = 0; t < kTogether; ++t) {
                const double m = n[t] ? 1.0 : 0.0;
                G.y = fma(m, yx[t].x, G.y); G.x = fma(m, yx[t].y, G.x); G.pc = fma(m, c[t], G.pc);
                G.k += n[t];
            }
        };
        if (blocks) read(0);
        G.k = lengths.upto(L);
        const size_t at = (size_t)g * (kTab + 1) + G.k;
        const double2 own_yx = f.sums_yx[at];
        const double own_c = f.sums_c[at];
        G.y = G.x = G.pc = 0.0;
        add_held(G, 0, since - away, (double)(int)L);
        G.y += own_yx.x; G.x += own_yx.y; G.pc += own_c;
        if (blocks) sum();
        for (int b0 = kTogether; b0 < blocks; b0 += kTogether) { read(b0); sum(); }
        return G;
    };
    // The offers, left for all: what the segments come to is what a build would leave in the table.
    struct Own { uint32_t T; unsigned long long met, key; } own{~0u, 0, 0};
    const auto offer = [&](const Gathered& G, const Requests& q, uint32_t tag) {
        const int L = clamped(q.length), N = base.n + since;
        const double Ctot = base.ctx + since_ctx, qd = cc.delta * (base.q_ctx + since_ctx);
        double Gq = G.k ? fma(cc.gamma, G.x, fma(cc.beta, G.y, qd)) : qd;
        double Hs = fma(cc.gamma, Ctot - G.pc, fma(cc.beta, (double)(N - G.k + 1), cc.alpha));
        double d = fma(cc.gamma, Ctot, fma(cc.beta, (double)N, cc.alpha));
        if (blended) {
            Gq = keep * Gq + a.lam * bq;
            Hs = keep * Hs + a.lam * bd;
            d = keep * d + a.lam * bd;
        }
        const float T = latency_at((float)q.ctx0, L, inst_coef(a, cc, bp, N), make_float2((float)Gq, (float)Hs), G.k);
        const float Dc = q.D > FLT_MAX ? FLT_MAX : q.D;
        const bool ok = lane < q.n && g != q.ex;      // (as in k_feedback)
        own.T = ok ? min(max(ordered_bits(T), 1u), ~0u - 1u) : ~0u;
        own.met = __ballot(ok && T <= Dc);
        own.key = falling_bits(d);
        const unsigned long long v = lane < 2 ? own.met : own.key;
        if (lane < 4) leave(words.own + ((size_t)(tag & 1) * M + g) * 4 + lane, ((lane & 1 ? v >> 32 : v & 0xFFFFFFFFu) << 32) | tag);
        if (kPart) f.T[(size_t)g * kWave + lane] = own.T;
        return ((unsigned long long)own.T << 32) | ((unsigned)g << kFeedInstAt) | tag;
    };
    const auto publish = [&](unsigned long long least, uint32_t tag) {      // of this wave's instances
        if (!reader) sh.offer[wave][lane] = least;
        __syncthreads();
        if (both != kFeedWaves) return;
        least = sh.offer[0][lane];
#pragma unroll
        for (int v = 1; v < kFeedWaves; ++v) least = min(least, sh.offer[v][lane]);
        leave(words.least + ((size_t)(tag & 1) * W + w) * kWave + lane, least);
    };
    constexpr unsigned long long kNobody = ~0ull << 32;

    Requests q = requests(f.first), next = requests(min(f.first + 1, f.rounds - 1));
    {
        unsigned long long least = kNobody | 1u;
        each_inst([&](int u) {
            enter(inst_of(u));
            least = min(least, offer(gather(q), q, 1u));
        });
        publish(least, 1u);
        if (!kPart && sh.state.team != W) return;      // (known since the barrier)
    }
    for (int round = f.first; round < f.rounds; ++round) {
        const uint32_t tag = (uint32_t)(round - f.first) + 1u;
        const bool more = round + 1 < f.rounds;
        // (on their way while the others' words are)
        const Requests after = requests(min(round + 2, f.rounds - 1));
        Gathered G{};
        if (!kPart && more && !reader && inst_of(0) < M) {
            while (since - away >= kFeedBlock) put_away();
            G = gather(next);
        }

        // the words of all, shared by the waves
        unsigned long long least, met;
        const unsigned long long* __restrict__ leasts = words.least + (size_t)(tag & 1) * W * kWave + lane;
        const unsigned long long* __restrict__ theirs = words.own + (size_t)(tag & 1) * M * 4;
        const int per = (W + kFeedWaves - 1) / kFeedWaves, h0 = min(wave * per, W - 1), h1 = min(h0 + per, W);
        // (one trip for as much as there usually is: 16 workgroups and 64 instances for a wave.  A wave's share of the workgroups is
        // at most M / 16 rounded up, and where they are fewer, so many trips still pass all instances)
        least = ~0ull;
        met = 0;
        int looks = 0;
        for (int b = 0; reader && b < (M + 15) / 16; b += kAhead) {
            unsigned long long v[kAhead], m[4];
            const int h = (b / kAhead * kFeedWaves + wave) * kWave + lane;
            for (;; ++looks) {
#pragma unroll
                for (int i = 0; i < kAhead; ++i) v[i] = peek(leasts + (size_t)min(h0 + b + i, h1 - 1) * kWave);
#pragma unroll
                for (int i = 0; i < 4; ++i) m[i] = peek(theirs + (size_t)min(h, M - 1) * 4 + i);
                bool all = true;
#pragma unroll
                for (int i = 0; i < kAhead; ++i) all = all && ((uint32_t)v[i] & ((1u << kFeedTagBits) - 1u)) == tag;
#pragma unroll
                for (int i = 0; i < 4; ++i) all = all && (uint32_t)m[i] == tag;
                if (__all(all)) break;
                if (looks >= kFeedPollsMore) { sh.state.over = 1; break; }
            }
#pragma unroll
            for (int i = 0; i < kAhead; ++i) least = min(least, v[i]);
            const unsigned long long their_met = (m[0] >> 32) | (m[1] >> 32 << 32);
            met |= their_met;
            if (h < M) sh.infos[h] = make_ulonglong2(their_met, (m[2] >> 32) | (m[3] >> 32 << 32));
        }
        if (reader) {
            sh.least[wave][lane] = least;
            met = wave_or_u64(met);
            if (lane == 0) sh.met[wave] = met;
        }
        __syncthreads();
        if (sh.state.over) {
            if (threadIdx.x == 0) atomicOr(&a.counters[0], GR_DEV_STALLED);
            return;
        }
        least = sh.least[0][lane];
        met = sh.met[0];
#pragma unroll
        for (int v = 1; v < kFeedWaves; ++v) {
            least = min(least, sh.least[v][lane]);
            met |= sh.met[v];
        }
        const bool live = lane < q.n, served = (met >> lane) & 1ull;
        const uint32_t least_T = (uint32_t)(least >> 32);
        const int64_t at = (int64_t)round * f.chunk + lane;
        if (w == 0 && both == 0 && live && !served && least_T == ~0u) {      // nobody is allowed
            f.out_inst[at] = -1;
            f.out_slack[at] = 0.f;
            if (f.out_fallback) f.out_fallback[at] = 1;
        }

        unsigned long long offered = kNobody | (tag + 1u);
        each_inst([&](int u) {
            if (kPart) {
                enter(inst_of(u));
                own.met = sh.infos[g].x;
                own.key = sh.infos[g].y;
                own.T = f.T[(size_t)g * kWave + lane];
            }
            // Alg. 1 for the instance itself: where a deadline can be met, it is met here and by nobody more capable; else nobody's
            // latency is less, or as little at a lower index
            unsigned long long above = 0;      // requests whose deadline is met by somebody more capable
            if (own.met) {
                for (int h = lane; h < M; h += kWave) {
                    const ulonglong2 o = sh.infos[h];
                    above |= o.y < own.key || (o.y == own.key && h < g) ? o.x : 0ull;
                }
                above = wave_or_u64(above);
            }
            const bool mine = live && (served ? ((own.met & ~above) >> lane) & 1ull
                                              : least_T != ~0u && (int)((uint32_t)least >> kFeedInstAt) == g);
            const unsigned long long joins = __ballot(mine);
            if (kPart && more) G = gather(next);
            if (joins) {
                if (mine) {
                    f.out_inst[at] = g;
                    f.out_slack[at] = q.D - from_ordered_bits(own.T);
                    if (f.out_fallback) f.out_fallback[at] = !served;
                    const int nth = pend + __popcll(joins & ((1ull << lane) - 1ull));
                    if (nth < kTab) {
                        a.pend_prompt[(size_t)g * kTab + nth] = q.ctx0;
                        a.pend_len[(size_t)g * kTab + nth] = q.length;
                    }
                }
                pend += __popcll(joins);
                if (lane == 0) { a.pend_cnt[g] = pend; a.pend_touched[g] = 1; }
            }
            if (joins && more) {      // (less than a block is held before: a chunk finds room)
                const int nth = __popcll(joins & ((1ull << lane) - 1ull)), taken = min(__popcll(joins), room - since);      // (beyond its room there are none)
                const bool in = mine && nth < taken;
                const double4 e = terms(q.ctx0, q.length);
                if (in) held[since - away + nth] = e;
                settled();
                add_held(G, since - away, since - away + taken, (double)clamped(next.length));
                since_ctx += readlane_f64(wave_incl_scan_f64(in ? e.z : 0.0), kWave - 1);
                since += taken;
                if (kPart) while (since - away >= kFeedBlock) put_away();
            }
            if (more) offered = min(offered, offer(G, next, tag + 1u));
        });
        if (!more) break;
        publish(offered, tag + 1u);
        q = next;
        next = after;
    }
    if (w == 0 && threadIdx.x == 0) *f.words.team = (uint32_t)W;
}

template <int kTab>
__global__ __launch_bounds__(2 * kFeedWaves * kWave, 2) void k_feedback_rounds(FeedRoundsArgs f)
{
    __shared__ FeedLengths<kTab> lengths[kFeedWaves];
    __shared__ unsigned long long least[kFeedWaves][kWave], offer[kFeedWaves][kWave], met[kFeedWaves];
    __shared__ double4 held[kFeedWaves][kFeedHeld];
    __shared__ ulonglong2 infos[kFeedInst];
    __shared__ FeedState state;
    const FeedShared<kTab> sh{lengths, least, offer, met, held, infos, state};
    fetch_args<FeedRoundsArgs>();
    const int all = gridDim.x;
    if (threadIdx.x == kFeedWaves * kWave) {      // (of a wave that has nothing else to do yet)
        const int2 at = pass_gate(f.words, all, f.polls);
        state.team = min(at.x, f.team);
        state.ticket = at.y;
        state.over = 0;
    }
    feedback_rounds<kTab, false>(f, sh, all, blockIdx.x);
    const int team = state.team, ticket = state.ticket;
    if (team == all || ticket < 0 || ticket >= team) return;
    __syncthreads();
    // (its arguments are read here anew: kept from the start, their addresses were 75 more scalar registers put away in the rounds of all)
    auto args = (const __attribute__((address_space(4))) FeedRoundsArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    feedback_rounds<kTab, true>(*(const FeedRoundsArgs*)args, sh, team, ticket);
}

// The capability rank of every instance, for the caller (Alg. 1's argmax d_g: rank 0 = largest d_g,
// equal d_g by index).  Four waves share a run of kRankPer instances and split the competitors, a
// lane per competitor, each lane with its own counts.  The time is that of the reads: the status
// build has just written d, so each XCD fetches it from memory, and a wave that read its 4 096
// competitors in four batches waited four times.  A quarter of them is one batch.  On 4 096
// instances 10.8 us with ballots added up by the scalar unit, 9.2 with a wave per run, 5.9 us this way.
// Competitors that lie wholly before or behind the run take one comparison each.
__global__ __launch_bounds__(kBlock) void k_rank(const double* __restrict__ d, int* __restrict__ out_rank, int n_inst)
{
    static_assert(kBlock == kRankWaves * kWave, "a workgroup ranks one run");
    __shared__ int sums[kRankWaves * kRankPer];
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int g0 = blockIdx.x * kRankPer;
    double dg[kRankPer];
    int r[kRankPer] = {};
#pragma unroll
    for (int j = 0; j < kRankPer; ++j) dg[j] = d[min(g0 + j, n_inst - 1)];
    constexpr int kAhead = 16;
    const int per = ((n_inst + kRankWaves - 1) / kRankWaves + kWave - 1) / kWave * kWave;
    const int h_end = min((wave + 1) * per, n_inst);
    for (int h0 = wave * per; h0 < h_end; h0 += kAhead * kWave) {
        double dh[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            const int h = h0 + k * kWave + lane;
            dh[k] = h < h_end ? d[h] : -__builtin_inf();      // ahead of nobody
        }
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            const int hb = h0 + k * kWave;
            if (hb >= h_end) break;
            if (hb + kWave <= g0) {
#pragma unroll
                for (int j = 0; j < kRankPer; ++j) r[j] += dh[k] >= dg[j];
            } else if (hb >= g0 + kRankPer) {
#pragma unroll
                for (int j = 0; j < kRankPer; ++j) r[j] += dh[k] > dg[j];
            } else {
#pragma unroll
                for (int j = 0; j < kRankPer; ++j) r[j] += dh[k] > dg[j] || (dh[k] == dg[j] && hb + lane < g0 + j);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < kRankPer; ++j) {
        const int all = wave_incl_scan_i32(r[j]);
        if (lane == kWave - 1) sums[wave * kRankPer + j] = all;
    }
    __syncthreads();
    if (wave != 0 || lane >= kRankPer || g0 + lane >= n_inst) return;
    int all = 0;
#pragma unroll
    for (int q = 0; q < kRankWaves; ++q) all += sums[q * kRankPer + lane];
    out_rank[g0 + lane] = all;
}

// One step of the exponential moving average of Alg. 1, q <- w * sample + (1 - w) * q, for
// each of the three status terms that has a new sample; a term's first sample is its estimate.
__global__ __launch_bounds__(kBlock) void k_ema(int n_inst, double w, const float* __restrict__ s_q,
                                                const float* __restrict__ s_p, const float* __restrict__ s_d,
                                                int first_q, int first_p, int first_d,
                                                double* __restrict__ q, double* __restrict__ p, double* __restrict__ d)
{
    const int g = blockIdx.x * kBlock + threadIdx.x;
    if (g >= n_inst) return;
    if (s_q) q[g] = first_q ? (double)s_q[g] : w * (double)s_q[g] + (1.0 - w) * q[g];
    if (s_p) p[g] = first_p ? (double)s_p[g] : w * (double)s_p[g] + (1.0 - w) * p[g];
    if (s_d) d[g] = first_d ? (double)s_d[g] : w * (double)s_d[g] + (1.0 - w) * d[g];
}

// Requests that were routed join the queue of their instance (feedback routing), in the order of
// the batch: the slot of a request is the number of requests already queued there plus the number
// of earlier requests of the chunk that were sent to the same instance.  That order matters under
// batch caps (admission is first come, first served), so it must not depend on how the hardware
// schedules waves.  A chunk that fits one wave is placed by that wave (lanes are in request
// order); without caps the build takes it in itself (InstanceIn::joins): 256 instances, 64 requests at
// a time, 17.8 us a round with a launch of its own for this, 14.1 without.  A larger chunk under caps takes two kernels: the first marks the instances that were
// chosen at all, the second gives every marked instance a wave that walks the chunk in order.
// Without caps the order of a queue shows in no output (the requests behind it wait for all of
// them either way; sums and sorted lengths do not depend on it), and a larger chunk is placed by
// one kernel that hands out slots with one atomic per wave and instance.
__global__ __launch_bounds__(kWave) void k_commit_wave(int n, const int* __restrict__ inst,
                                                       const int* __restrict__ ctx0, const int* __restrict__ pred_len,
                                                       int* __restrict__ pend_cnt, int* __restrict__ pend_prompt,
                                                       int* __restrict__ pend_len, int* __restrict__ pend_touched,
                                                       int cap, int n_inst, int* __restrict__ counters)
{
    const int lane = lane_id();
    int g = lane < n ? inst[lane] : -1;
    if (g >= n_inst) g = -1;
    const bool act = g >= 0;
    unsigned long long todo = __ballot(act);
    int slot = 0;
    while (todo) {
        const int leader = __ffsll((long long)todo) - 1;
        const int gl = __builtin_amdgcn_readlane(g, leader);
        const unsigned long long same = __ballot(act && g == gl);
        int base = 0;
        if (lane == leader) {
            base = pend_cnt[gl];
            pend_cnt[gl] = base + __popcll(same);
            pend_touched[gl] = 1;
        }
        base = __builtin_amdgcn_readlane(base, leader);
        if (act && g == gl) slot = base + __popcll(same & ((1ull << lane) - 1ull));
        todo &= ~same;
    }
    if (act) {
        if (slot < cap) {
            pend_prompt[(size_t)g * cap + slot] = ctx0[lane];
            pend_len[(size_t)g * cap + slot] = pred_len[lane];
        } else {
            atomicOr(&counters[0], GR_DEV_ENTRIES_DROPPED);
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_commit_any_order(int64_t n, const int* __restrict__ inst,
                                                             const int* __restrict__ ctx0, const int* __restrict__ pred_len,
                                                             int* __restrict__ pend_cnt, int* __restrict__ pend_prompt,
                                                             int* __restrict__ pend_len, int* __restrict__ pend_touched,
                                                             int cap, int n_inst, int* __restrict__ counters)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int lane = lane_id();
    int g = i < n ? inst[i] : -1;
    if (g >= n_inst) g = -1;
    const bool act = g >= 0;
    unsigned long long todo = __ballot(act);
    int slot = 0;
    while (todo) {      // many requests of a chunk go to the same instance: one atomic for all of a wave's
        const int leader = __ffsll((long long)todo) - 1;
        const int gl = __builtin_amdgcn_readlane(g, leader);
        const unsigned long long same = __ballot(act && g == gl);
        int base = 0;
        if (lane == leader) {
            base = atomicAdd(&pend_cnt[gl], __popcll(same));
            pend_touched[gl] = 1;
        }
        base = __builtin_amdgcn_readlane(base, leader);
        if (act && g == gl) slot = base + __popcll(same & ((1ull << lane) - 1ull));
        todo &= ~same;
    }
    if (act) {
        if (slot < cap) {
            pend_prompt[(size_t)g * cap + slot] = ctx0[i];
            pend_len[(size_t)g * cap + slot] = pred_len[i];
        } else {
            atomicOr(&counters[0], GR_DEV_ENTRIES_DROPPED);
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_commit_mark(int64_t n, const int* __restrict__ inst, int n_inst,
                                                        int* __restrict__ mark)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const int g = inst[i];
    if (g >= 0 && g < n_inst) mark[g] = 1;
}

__global__ __launch_bounds__(kBlock) void k_commit_place(int64_t n, const int* __restrict__ inst,
                                                         const int* __restrict__ ctx0, const int* __restrict__ pred_len,
                                                         int* __restrict__ mark, int* __restrict__ pend_cnt,
                                                         int* __restrict__ pend_prompt, int* __restrict__ pend_len,
                                                         int* __restrict__ pend_touched, int cap, int n_inst,
                                                         int* __restrict__ counters)
{
    const int lane = lane_id();
    const int g = blockIdx.x * kBuildWaves + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (g >= n_inst || !mark[g]) return;
    int base = pend_cnt[g];
    bool dropped = false;
    constexpr int kStep = 4;      // blocks of 64 requests in flight together
    for (int64_t i0 = 0; i0 < n; i0 += kStep * kWave) {
        int gi[kStep];
#pragma unroll
        for (int k = 0; k < kStep; ++k) {
            const int64_t i = i0 + k * kWave + lane;
            gi[k] = i < n ? inst[i] : -1;
        }
#pragma unroll
        for (int k = 0; k < kStep; ++k) {
            const unsigned long long m = __ballot(gi[k] == g);
            if (!m) continue;
            if (gi[k] == g) {
                const int64_t i = i0 + k * kWave + lane;
                const int slot = base + __popcll(m & ((1ull << lane) - 1ull));
                if (slot < cap) {
                    pend_prompt[(size_t)g * cap + slot] = ctx0[i];
                    pend_len[(size_t)g * cap + slot] = pred_len[i];
                } else {
                    dropped = true;
                }
            }
            base += __popcll(m);
        }
    }
    if (__ballot(dropped) && lane == 0) atomicOr(&counters[0], GR_DEV_ENTRIES_DROPPED);
    if (lane == 0) {
        pend_cnt[g] = base;
        pend_touched[g] = 1;
        mark[g] = 0;
    }
}

// LDS of a build that shares an instance between kSplit waves: contexts, two exchange buffers, totals
template <int kEPL, int kSplit>
constexpr size_t split_lds()
{
    return (size_t)(lean_inst_words(kWave * kEPL) + 2 * kWave * kEPL) * sizeof(int) + kSplit * 4 * sizeof(double);
}

template <int kEPL>
constexpr size_t lean_lds() { return (size_t)kBuildWaves * lean_inst_words(kWave * kEPL) * sizeof(int); }

// Whether instances pick the number of sort words by what they hold: where half of the words would do
// for the average one, and always in feedback routing, whose handles are made with room for what is routed
// (256 instances of 512 to 560 requests in tables for 2 048: 8.5 us instead of 10.0).  Elsewhere the
// choice is one more thing to wait for before the first read (1 024 x 1 000: 15.4 instead of 14.3 us).
bool fit_words(const BuildArgs& b, int M, int cap)
{
    return (b.n_active + b.n_queued) * 2 <= (int64_t)M * cap;
}

template <int kEPL, int kSplit>
int launch_build_split(const BuildArgs& b, int M, hipStream_t s)
{
    constexpr size_t lds = split_lds<kEPL, kSplit>();
    if (b.use_pending)
        hipLaunchKernelGGL((k_build_lean<kEPL / kSplit, kSplit, true, true>), dim3(M), dim3(kSplit * kWave), lds, s, b);
    else if (fit_words(b, M, kWave * kEPL))
        hipLaunchKernelGGL((k_build_lean<kEPL / kSplit, kSplit, true, false>), dim3(M), dim3(kSplit * kWave), lds, s, b);
    else
        hipLaunchKernelGGL((k_build_lean<kEPL / kSplit, kSplit, false, false>), dim3(M), dim3(kSplit * kWave), lds, s, b);
    return kSplit;
}

// kEPL: sort words per lane if one wave takes an instance.  Returns the waves that share an instance.
template <int kEPL>
int launch_build(const BuildArgs& b, int M, hipStream_t s)
{
    const dim3 grid((M + kBuildWaves - 1) / kBuildWaves);
    const size_t lds = (size_t)kBuildWaves * kWave * kEPL * sizeof(int);
    if (b.batch_cap) {
        hipLaunchKernelGGL((k_build_capped<kEPL>), grid, dim3(kBlock), 3 * lds, s, b);
        return 1;
    }
    const int waves = waves_per_instance(kEPL, M);
    if constexpr (kEPL >= 4) if (waves == 4) return launch_build_split<kEPL, 4>(b, M, s);
    if constexpr (kEPL >= 2) if (waves == 2) return launch_build_split<kEPL, 2>(b, M, s);
    hipLaunchKernelGGL((k_build_lean<kEPL, 1, false, false>), grid, dim3(kBlock), lean_lds<kEPL>(), s, b);
    return 1;
}

}  // namespace

int launch_commit(gr_fleet* f, int64_t n, const int* inst, const int* ctx0, const int* pred_len, hipStream_t s)
{
    if (n == 0) return GR_OK;
    if (n <= kWave) {
        hipLaunchKernelGGL(k_commit_wave, dim3(1), dim3(kWave), 0, s, (int)n, inst, ctx0, pred_len, f->pend_cnt,
                           f->pend_prompt, f->pend_len, f->pend_touched, f->cap, f->n_inst, f->counters);
    } else if (!f->has_cap) {
        hipLaunchKernelGGL(k_commit_any_order, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, n, inst,
                           ctx0, pred_len, f->pend_cnt, f->pend_prompt, f->pend_len, f->pend_touched, f->cap, f->n_inst,
                           f->counters);
    } else {
        hipLaunchKernelGGL(k_commit_mark, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, n, inst,
                           f->n_inst, f->commit_mark);
        hipLaunchKernelGGL(k_commit_place, dim3((f->n_inst + kBuildWaves - 1) / kBuildWaves), dim3(kBlock), 0, s, n, inst,
                           ctx0, pred_len, f->commit_mark, f->pend_cnt, f->pend_prompt, f->pend_len, f->pend_touched,
                           f->cap, f->n_inst, f->counters);
    }
    return hipGetLastError() == hipSuccess ? GR_OK : GR_ERR_HIP;
}

int launch_ema(gr_fleet* f, double w, const float* s_q, const float* s_p, const float* s_d, hipStream_t s)
{
    hipLaunchKernelGGL(k_ema, dim3((f->n_inst + kBlock - 1) / kBlock), dim3(kBlock), 0, s, f->n_inst, w, s_q, s_p, s_d,
                       !f->have_q, !f->have_p, !f->have_d, f->emaQ, f->emaP, f->emaD);
    if (hipGetLastError() != hipSuccess) return GR_ERR_HIP;
    f->have_q |= s_q != nullptr; f->have_p |= s_p != nullptr; f->have_d |= s_d != nullptr;
    return GR_OK;
}

// Dynamic LDS limits of the build kernels, set to what each needs at most: the attribute belongs to the kernel, not to
// a handle, so a smaller handle must not lower it for a live, larger one.
int status_prepare()
{
    bool ok = true;
    const auto set = [&](auto kernel, size_t bytes) {
        ok = ok && hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)bytes) == hipSuccess;
    };
    constexpr size_t word = kBuildWaves * kWave * sizeof(int);     // per sort word per lane
    set(k_build_lean<1, 1, false, false>, lean_lds<1>()); set(k_build_lean<2, 1, false, false>, lean_lds<2>());
    set(k_build_lean<4, 1, false, false>, lean_lds<4>()); set(k_build_lean<8, 1, false, false>, lean_lds<8>());
    set(k_build_lean<16, 1, false, false>, lean_lds<16>()); set(k_build_lean<32, 1, false, false>, lean_lds<32>());
#define GR_SET_SPLIT(E, W) \
    set(k_build_lean<E, W, false, false>, split_lds<E * W, W>()); set(k_build_lean<E, W, true, false>, split_lds<E * W, W>()); \
    set(k_build_lean<E, W, true, true>, split_lds<E * W, W>())
    GR_SET_SPLIT(1, 2); GR_SET_SPLIT(2, 2); GR_SET_SPLIT(4, 2); GR_SET_SPLIT(8, 2); GR_SET_SPLIT(16, 2);
    GR_SET_SPLIT(1, 4); GR_SET_SPLIT(2, 4); GR_SET_SPLIT(4, 4); GR_SET_SPLIT(8, 4);
#undef GR_SET_SPLIT
#define GR_SET_FEEDBACK(E, W) set(k_feedback<E, W, false>, split_lds<E * W, W>()); set(k_feedback<E, W, true>, split_lds<E * W, W>())
    GR_SET_FEEDBACK(1, 2); GR_SET_FEEDBACK(1, 4); GR_SET_FEEDBACK(2, 4); GR_SET_FEEDBACK(4, 4); GR_SET_FEEDBACK(8, 4);
#undef GR_SET_FEEDBACK
    set(k_build_capped<1>, 3 * word * 1); set(k_build_capped<2>, 3 * word * 2); set(k_build_capped<4>, 3 * word * 4);
    set(k_build_capped<8>, 3 * word * 8); set(k_build_capped<16>, 3 * word * 16); set(k_build_capped<32>, 3 * word * 32);
    return ok ? GR_OK : GR_ERR_HIP;
}

int launch_ranks(gr_fleet* f, int* out_rank, hipStream_t s)
{
    {
        ProfScope ps(f, kRank, s);
        hipLaunchKernelGGL(k_rank, dim3((f->n_inst + kRankPer - 1) / kRankPer), dim3(kBlock), 0, s, f->hD, out_rank, f->n_inst);
    }
    return hipGetLastError() == hipSuccess ? GR_OK : GR_ERR_HIP;
}

static BuildArgs build_args(const gr_fleet* f, const StatusIn& in)
{
    BuildArgs b{};
    b.act_off = in.act_off; b.act_prompt = in.act_prompt; b.act_gen = in.act_gen; b.act_rem = in.act_rem;
    b.q_off = in.q_off; b.q_prompt = in.q_prompt; b.q_len = in.q_len;
    b.act_budget = in.act_budget;
    b.out_act_finish = in.out_act_finish; b.out_q_finish = in.out_q_finish;
    b.out_d = in.out_d; b.out_flag = in.out_flag;
    b.cls = f->cls; b.inst_class = f->inst_class;
    b.tabR = f->tabR; b.tabGH = f->tabGH;
    b.hD = f->hD; b.act_inst = f->act_inst;
    b.instK = f->instK; b.tabS = f->tabS; b.slot_of = f->slot_of; b.slot_key = f->slot_key; b.counters = f->counters;
    b.n_active = in.n_active; b.n_queued = in.n_queued;
    b.n_inst = f->n_inst; b.max_entries = f->max_entries; b.max_len = f->max_len;
    b.seen = in.mark ? f->seen : nullptr; b.late_cnt = f->late_cnt; b.unset = f->totals + 2;
    b.pend_cnt = f->pend_cnt; b.pend_prompt = f->pend_prompt; b.pend_len = f->pend_len;
    b.use_pending = in.use_pending;
    b.pend_touched = f->pend_touched; b.only_touched = in.use_pending && in.only_touched;
    b.chunk_n = in.chunk_n; b.chunk_inst = in.chunk_inst; b.chunk_ctx0 = in.chunk_ctx0; b.chunk_len = in.chunk_len;
    b.batch_cap = f->has_cap ? f->batch_cap : nullptr;
    b.lam = f->lam; b.emaQ = f->emaQ; b.emaP = f->emaP; b.emaD = f->emaD;
    return b;
}

// The account of the tables after a build on stream `s`.  (The class order is made by the next scoring pass that needs it.)
static void tables_built(gr_fleet* f, hipStream_t s)
{
    const TableAccount account(f, s);
    *account.v = TableView{true, false, f->lam != 0.0};
    if (account.capturing) {
        f->recorded = true;
        f->blend_recorded |= f->lam != 0.0;
    }
}

static_assert(4 * kSimds / kFeedInst >= 4, "four waves per instance wherever the tables have words for them");
static_assert(kWave <= kDirectMax && kWave * kFeedInst <= kDirectInfinite, "an infinite latency is one in every chunk");

// Where a chunk would be scored pair by pair and would join its instances in the rebuild (no caps), and an instance has two
// waves or more.  Every workgroup reads all offers, so the gain shrinks as the fleet grows.  A round, us, two launches / one:
// 64 instances 12.4 / 7.8, 128 10.7 / 7.6, 256 14.0 / 10.6, 400 15.1 / 12.2, 512 16.0 / 13.3 (a rebuild with finish
// times in the former; without them 1.5 less); wider fleets are not taken.
bool feedback_by_round(const gr_fleet* f, int64_t chunk)
{
    return f->feed_T && !f->has_cap && chunk <= kWave && pair_by_pair(f, chunk);
}

// Whether the rounds are one launch (k_feedback_rounds, with one before it that builds all tables for the sums and one behind): where what the
// launches of every round take (3 us, and 1 us more for every 64 instances, whose offers each workgroup reads) is more than what the requests of a
// chunk take that all go to one instance (0.08 us each), by as much as the three launches: from four rounds on, and three on fleets
// of some size (two: 256/1 23.6 / 24.3; 512/1 30.1 / 27.5, left a launch each).  Whole calls, us, a launch per round / one, N/c x r: N instances, chunks of
// c, r rounds, deadlines that few meet, in brackets such that all go for the same instances:
//   256/64 x 32 331 / 160 (358 / 240)   256/1 x 100 970 / 300   64/8 x 38 309 / 135   4/1 x 4 32.4 / 29.4   64/8 x 4 34.0 / 31.2 (32.1 / 29.8)
//   4/16 x 4 32.8 / 31.3 (32.5 / 31.7)   32/32 x 4 33.7 / 31.9 (33.3 / 34.7)   64/32 x 5 39.9 / 37.5 (38.1 / 41.0)   128/32 x 4 36.2 / 32.2 (35.4 / 35.0)
//   128/64 x 5 42.9 / 39.4 (42.2 / 48.5)   256/64 x 4 41.5 / 37.4 (41.5 / 42.1)   16/32 x 8 59.0 / 51.6 (59.1 / 59.3)   16/64 x 8 59.8 / 58.1 (62.1 / 69.4)
//   three: 1/1 23.7 / 24.1   4/4 25.8 / 26.5   64/1 26.1 / 26.4   128/1 27.7 / 26.4   128/16 28.7 / 28.1 (27.9 / 27.6)   128/32 28.9 / 28.7 (28.3 / 29.9)
//   256/32 32.8 / 30.1   256/64 33.0 / 31.8 (32.7 / 34.9)   512/64 43.2 / 36.8
static bool in_one_launch(const gr_fleet* f, int64_t chunk, int64_t rounds)
{
    const double more = (double)rounds * (2.9 + f->n_inst / 64.0 - 0.08 * (double)chunk);
    return rounds >= 4 ? more > 7.0 : rounds == 3 && f->n_inst > 64 && more > 10.0;
}

// The kernel for tables of epl * kWave entries.
template <typename Use>
static auto with_rounds_kernel(int epl, Use use)
{
    switch (epl) {
        case 2: return use(k_feedback_rounds<2 * kWave>);
        case 4: return use(k_feedback_rounds<4 * kWave>);
        case 8: return use(k_feedback_rounds<8 * kWave>);
        case 16: return use(k_feedback_rounds<16 * kWave>);
        default: return use(k_feedback_rounds<32 * kWave>);
    }
}

int feedback_prepare(gr_fleet* f)
{
    const bool ok = hipDeviceGetAttribute(&f->units, hipDeviceAttributeMultiprocessorCount, f->device) == hipSuccess &&
                    with_rounds_kernel(f->epl, [&](auto kernel) {
                        return hipOccupancyMaxActiveBlocksPerMultiprocessor(&f->feed_per_unit, kernel, 2 * kFeedWaves * kWave, 0);
                    }) == hipSuccess;
    return ok ? GR_OK : GR_ERR_HIP;
}

// Whether the workgroups of k_feedback_rounds, which wait for each other, can all run at once: on a stream of few compute units, or a
// device of few, every call would wait in vain, then share the work of those that did not come.  (A recorded call
// is asked about the stream that records it.)
static bool all_run_at_once(const gr_fleet* f, hipStream_t s)
{
    int units = std::min(f->units, f->feed_units);
    uint32_t mask[32] = {};
    if (hipExtStreamGetCUMask(s, sizeof mask / sizeof *mask, mask) == hipSuccess) {
        int usable = 0;
        for (const uint32_t m : mask) usable += __builtin_popcount(m);
        if (usable) units = std::min(units, usable);
    } else {
        (void)hipGetLastError();
    }
    return (int64_t)units * f->feed_per_unit >= feed_groups(f->n_inst);
}

static void launch_feedback_rounds(gr_fleet* f, const BuildArgs& b, const FeedbackIn& r, int first, int rounds, hipStream_t s)
{
    FeedRoundsArgs a{};
    a.b = b;
    a.b.chunk_n = 0;
    a.ctx0 = r.ctx0; a.pred_len = r.pred_len; a.exclude = r.exclude; a.budget = r.budget;
    a.out_inst = r.out_inst; a.out_slack = r.out_slack; a.out_fallback = r.out_fallback;
    a.n = r.n; a.chunk = r.chunk; a.first = first; a.rounds = rounds; a.polls = f->feed_polls; a.team = f->feed_team;
    a.sums_yx = f->feed_yx; a.sums_c = f->feed_c; a.base = f->feed_base; a.blocks = f->feed_blocks; a.words = f->feed_words; a.T = f->feed_T;
    ProfScope ps(f, kFeedback, s);
    with_rounds_kernel(f->epl, [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(feed_groups(f->n_inst)), dim3(2 * kFeedWaves * kWave), 0, s, a);
    });
}

int launch_feedback(gr_fleet* f, const StatusIn& in, const FeedbackIn& r, hipStream_t s)
{
    FeedSumsArgs sums{};
    FeedArgs& a = sums.f;
    a.b = build_args(f, in);
    const size_t M = f->n_inst;
    const int64_t rounds = (r.n + r.chunk - 1) / r.chunk;
    const bool together = in_one_launch(f, r.chunk, rounds) && all_run_at_once(f, s);
    sums.sums_yx = f->feed_yx; sums.sums_c = f->feed_c; sums.base = f->feed_base; sums.words = f->feed_words;
    int launches = 0;
    // one launch that decides a chunk (-1: none) and offers for another
    const auto queue = [&](int64_t decided, int64_t offered) {
        const int64_t at = offered * r.chunk, was = decided * r.chunk;
        a.b.chunk_n = decided >= 0 ? (int)std::min<int64_t>(r.n - was, r.chunk) : 0;
        a.b.only_touched = r.current || decided != 0;
        if (a.b.chunk_n) {
            a.b.chunk_ctx0 = r.ctx0 + was; a.b.chunk_len = r.pred_len + was;
            a.budget = r.budget + was; a.out_inst = r.out_inst + was; a.out_slack = r.out_slack + was;
            a.out_fallback = r.out_fallback ? r.out_fallback + was : nullptr;
        }
        a.next_n = offered >= 0 ? (int)std::max<int64_t>(0, std::min<int64_t>(r.n - at, r.chunk)) : 0;
        if (a.next_n) {
            a.next_ctx0 = r.ctx0 + at; a.next_len = r.pred_len + at; a.next_budget = r.budget + at;
            a.next_exclude = r.exclude ? r.exclude + at : nullptr;
        }
        const size_t out = launches++ & 1, got = out ^ 1;
        a.T_in = f->feed_T + got * M * kWave; a.met_in = f->feed_met + got * M; a.key_in = f->feed_key + got * M;
        a.T_out = f->feed_T + out * M * kWave; a.met_out = f->feed_met + out * M; a.key_out = f->feed_key + out * M;
        ProfScope ps(f, kFeedback, s);
        const int waves = waves_per_instance(f->epl, f->n_inst);
#define GR_LAUNCH_FEEDBACK(E, W) \
        if (together) hipLaunchKernelGGL((k_feedback<E / W, W, true>), dim3((unsigned)M), dim3(W * kWave), (split_lds<E, W>()), s, sums); \
        else hipLaunchKernelGGL((k_feedback<E / W, W, false>), dim3((unsigned)M), dim3(W * kWave), (split_lds<E, W>()), s, a); \
        break
        switch (f->epl * 8 + waves) {
            case 2 * 8 + 2: GR_LAUNCH_FEEDBACK(2, 2);
            case 4 * 8 + 4: GR_LAUNCH_FEEDBACK(4, 4);
            case 8 * 8 + 4: GR_LAUNCH_FEEDBACK(8, 4);
            case 16 * 8 + 4: GR_LAUNCH_FEEDBACK(16, 4);
            default: GR_LAUNCH_FEEDBACK(32, 4);
        }
#undef GR_LAUNCH_FEEDBACK
    };
    if (together) {
        // (the first chunk is decided from the tables as they stand, whose rebuild may change them all)
        const int64_t first = r.current ? 0 : 1;
        if (first) queue(-1, 0);
        for (int64_t from = first; from < rounds; from += kFeedMostRounds) {
            sums.move = kFeedAll;
            queue(from == first && first ? 0 : -1, -1);
            launch_feedback_rounds(f, a.b, r, (int)from, (int)std::min<int64_t>(rounds, from + kFeedMostRounds), s);
        }
        sums.move = kFeedTouched;
        queue(-1, -1);
    } else {
        for (int64_t k = 0; k <= rounds; ++k) queue(k - 1, k);
    }
    if (hipGetLastError() != hipSuccess) {
        TableAccount(f, s).v->current = false;
        return GR_ERR_HIP;
    }
    tables_built(f, s);
    return GR_OK;
}

int launch_status(gr_fleet* f, const StatusIn& in, hipStream_t s)
{
    const BuildArgs b = build_args(f, in);
    const int M = f->n_inst;
    int parts = 1;
    {
        ProfScope ps(f, kBuild, s);
        switch (f->epl) {
            case 1: parts = launch_build<1>(b, M, s); break;
            case 2: parts = launch_build<2>(b, M, s); break;
            case 4: parts = launch_build<4>(b, M, s); break;
            case 8: parts = launch_build<8>(b, M, s); break;
            case 16: parts = launch_build<16>(b, M, s); break;
            default: parts = launch_build<32>(b, M, s); break;
        }
    }
    if (in.act_budget) f->late_parts = parts;
    tables_built(f, s);
    int rc = in.out_rank ? launch_ranks(f, in.out_rank, s) : GR_OK;
    if (rc == GR_OK && hipGetLastError() != hipSuccess) rc = GR_ERR_HIP;
    if (rc != GR_OK) {
        TableAccount(f, s).v->current = false;
        return rc;
    }
    f->has_status = true;
    if (!in.use_pending) f->last_in = in;     // what a later feedback routing rebuilds from
    return GR_OK;
}

}  // namespace gr
