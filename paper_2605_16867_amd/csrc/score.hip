// Pair scoring (steps 2 and 3 of the path): Alg. 1 for a batch of requests
// against one snapshot of the instance tables.
//
// T(r,g) = E_g(L_r) + c0_r * kappa_g(L_r) (see common.h), and E, kappa depend on
// the request only through its length.  So E is tabulated once per (distinct
// length, instance) from the instance's sorted lengths, by counting, with its
// least value over every run of 16 positions of the class order (instances
// class by class, inside a class in capability order).  A run's least E with
// its least kappa bounds every latency of the run from below, formed with the
// same two fused multiply-adds, which are monotone in each operand, so the bound
// also holds after rounding; without a blend it is the least latency itself.
// A request then looks at the runs first and at the positions of a run only
// where the bound leaves the run in question (k_select), and large batches look
// at the classes before the runs, or at the few instances that can have the least
// latency at a length (k_lines).  The choice is Alg. 1's over all pairs, bit for bit.
//
// A batch of a few requests skips the table: a thread per pair with its own
// two-step search (k_direct).
#include <algorithm>
#include <cfloat>
#include <type_traits>

#include "common.h"

namespace gr {
namespace {

// ------------------------------------------------------------------ distinct lengths
// Which lengths a routing batch has: a byte per length (for the flagged requests of a risk scan
// the status build leaves them).  Every writer stores the same byte and a wave's stores to one
// line are one access, so no atomics and no LDS: 262 144 requests take 2.7 us where a histogram
// with LDS counters took 8.3.
constexpr int kMarkItems = 4;

__global__ __launch_bounds__(kBlock) void k_mark(const int* __restrict__ pred_len, int64_t n, uint8_t* __restrict__ seen,
                                                 int max_len)
{
    const int64_t base = (int64_t)blockIdx.x * (kBlock * kMarkItems) + threadIdx.x;
    int L[kMarkItems];
#pragma unroll
    for (int k = 0; k < kMarkItems; ++k) L[k] = pred_len[min(base + k * kBlock, n - 1)];
#pragma unroll
    for (int k = 0; k < kMarkItems; ++k) seen[min(max(L[k], 0), max_len)] = 1;
}

constexpr int kScanBlock = 1024;
constexpr int kScanWaves = kScanBlock / kWave;
constexpr int kScanGroups = 16;     // workgroups
constexpr int kScanChunks = 2;      // blocks of 64 lengths per wave
static_assert(kMaxLen + 1 <= kWave * kScanChunks * kScanWaves * kScanGroups, "every length has a lane of some wave");

struct ScanArgs {
    uint8_t* seen;
    int* row_len;
    uint16_t* len_row;
    int* totals;
    const int* late_cnt;    // flagged requests, n_late counts
    int* out_n;             // may be null
    // a risk scan's running requests (null: a routing batch)
    const uint8_t* flag;
    const int *act_rem, *act_off;
    int64_t n;
    int bins, n_late, n_inst;
};

// The list of lengths present ("rows", ascending) and, per length, the number of rows that are
// shorter.  A wave owns one or two blocks of 64 consecutive lengths (lane = length within the
// block); instead of passing sums from workgroup to workgroup each workgroup counts everything
// before its own lengths itself (the bytes sit in L2); the last one also has the total.
//
// The migration pass goes by the flags as they are, and a flag that no instance sets is the caller's own:
// of running entries in nobody's slice, and of those the build passes over (totals[2]).  With such entries the
// lengths and the count are taken from the flags, by each workgroup for itself.
//
// Workgroups past the first kScanGroups place the instances in class order, which the next kernel
// needs as well and which would cost a launch of its own otherwise.
__global__ __launch_bounds__(kScanBlock) void k_scan(ScanArgs a, OrderArgs order)
{
    __shared__ int w_rows[2][kScanWaves];
    __shared__ int sums[kScanWaves * kRankPer];
    if ((int)blockIdx.x >= kScanGroups) {
        order_block<kScanBlock>(order, blockIdx.x - kScanGroups, sums);
        return;
    }
    const int lane = lane_id(), wave = threadIdx.x / kWave;
    const int chunks = (a.bins + kWave - 1) / kWave;
    const int per = (chunks + kScanWaves * kScanGroups - 1) / (kScanWaves * kScanGroups);    // 1 or 2
    const int first = min((int)blockIdx.x * kScanWaves * per * kWave, a.bins);    // first length of this workgroup
    const auto wave_total = [](int v) { return __builtin_amdgcn_readlane(wave_incl_scan_i32(v), kWave - 1); };

    bool unset = false;
    if (a.flag) unset = a.totals[2] != 0 || a.act_off[0] > 0 || a.act_off[a.n_inst] < a.n;

    bool here[kScanChunks];
    int n_flags = 0;
    for (int pass = 0;; ++pass) {
        // everything before this workgroup's lengths, 16 at a time (`first` is a
        // multiple of 64 or the end, and behind the end are zeros)
        int before = 0;
        for (int i = threadIdx.x; i < (first + 15) / 16; i += kScanBlock) {
            const uint4 v = reinterpret_cast<const uint4*>(a.seen)[i];
            before += __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
        }
        // this wave's own lengths
        int own = 0;
#pragma unroll
        for (int k = 0; k < kScanChunks; ++k) {
            const int i = first + (wave * per + k) * kWave + lane;
            here[k] = k < per && i < a.bins && a.seen[i] != 0;
            own += __popcll(__ballot(here[k]));
        }
        before = wave_total(before);
        if (lane == 0) { w_rows[0][wave] = before; w_rows[1][wave] = own; }
        __syncthreads();
        if (!unset || pass) break;
        for (int64_t i = threadIdx.x; i < a.n; i += kScanBlock) {
            if (!a.flag[i]) continue;
            a.seen[min(max(a.act_rem[i], 0), a.bins - 1)] = 1;
            ++n_flags;
        }
        __syncthreads();
    }
    int u = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kScanWaves; ++w) {
        u += w_rows[0][w] + (w < wave ? w_rows[1][w] : 0);
        all += w_rows[0][w] + w_rows[1][w];
    }
    const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
    for (int k = 0; k < kScanChunks; ++k) {
        const int i = first + (wave * per + k) * kWave + lane;
        const unsigned long long present = __ballot(here[k]);
        const int row = u + __popcll(present & below);
        if (k < per && i < a.bins) {
            a.len_row[i] = (uint16_t)row;
            if (here[k]) a.row_len[row] = i;
        }
        u += __popcll(present);
    }
    if (blockIdx.x != kScanGroups - 1) return;
    if (threadIdx.x == 0) a.totals[1] = all;        // the last workgroup has seen every length
    if (a.out_n) {
        int n = n_flags;
        for (int i = threadIdx.x; !unset && i < a.n_late; i += kScanBlock) n += a.late_cnt[i];
        n = wave_total(n);
        if (lane == 0) sums[wave] = n;
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int w = 1; w < kScanWaves; ++w) n += sums[w];
            *a.out_n = n;
        }
    }
}

// The flagged requests of a risk scan, counted by one workgroup where k_scan does not: by the build's counts, or by the
// flags where the build has not set every one (see ScanArgs).
struct CountArgs {
    int *totals, *out_n;      // totals null: no risk scan
    const int *late_cnt, *act_off;
    const uint8_t* flag;
    int64_t n;
    int n_late, n_inst;
};

__device__ __forceinline__ void count_flagged(const CountArgs& a, int threads, int* sums)
{
    const int tid = threadIdx.x;
    const bool unset = a.totals[2] != 0 || a.act_off[0] > 0 || a.act_off[a.n_inst] < a.n;
    int n = 0;
    if (a.out_n) {
        if (unset) for (int64_t i = tid; i < a.n; i += threads) n += a.flag[i] != 0;
        else for (int i = tid; i < a.n_late; i += threads) n += a.late_cnt[i];
    }
    n = wave_sum(n);
    if (lane_id() == 0) sums[tid / kWave] = n;
    __syncthreads();
    if (tid != 0) return;
    for (int w = 1; w < threads / kWave; ++w) n += sums[w];
    if (a.out_n) *a.out_n = n;
    a.totals[2] = 0;
}

// The row of a length: its place in the list, or the length itself where every length has a row.
__device__ inline int row_at(const uint16_t* len_row, int L) { return len_row ? (int)len_row[L] : L; }

// ------------------------------------------------------------------ E per length and position
struct MemoArgs {
    int* totals;
    const int *row_len, *order;
    const uint16_t* len_row;
    const float4* instK;
    const uint16_t* tabR;
    const float2* tabGH;
    float* memo;           // see memo_at
    float* grp_min;        // see runs_at
    float4* run_k;         // [n_run]
    uint32_t *run_rank, *pos_thr;   // [n_run], [m_pos], see gr_fleet
    int* run_at;                    // [n_run]
    const float2* posK;
    const unsigned long long* posKey;
    const uint4* run_head;
    uint4* seen;           // cleared here for the next batch (its reader is done), as is totals[2]
    int seen_words;        // of 16 bytes
    int n_run, run_pad, cap, bins;
    const int2* run_cls;
    CountArgs count;       // of a risk scan, where every length has a row
    OrderArgs own;         // the class order, made here (small classes)
};

// The table is cut into blocks of kMemoU rows; a run's part of a block is consecutive, row by row, so that the
// kMemoP values of a row and run are one piece of 64 bytes: what a request looks at, and what a lane per row
// reads.  (With a position's values of 256 rows together instead every one of them was a cache line of its own.)
constexpr int kTile = kMemoU * kMemoP;

__device__ inline size_t memo_at(int64_t row, int run, int n_run)
{
    return ((size_t)(row / kMemoU) * n_run + run) * kTile + (size_t)(row % kMemoU) * kMemoP;
}

// The runs' least values: row by row where a request's lanes take 16 runs of its row at a time, in
// blocks like the table where the classes' least values are formed first, a lane per row.
template <bool kBlocks>
__device__ inline size_t runs_at(int64_t row, int run_pad)
{
    return kBlocks ? (size_t)(row / kMemoU) * run_pad * kMemoU + (size_t)(row % kMemoU) : (size_t)row * run_pad;
}
template <bool kBlocks>
constexpr int kRunStride = kBlocks ? kMemoU : 1;

// minimum of two values of which none is a NaN that must not come out quiet (the compiler guards
// against that with an instruction per operand)
__device__ inline float min_plain(float a, float b)
{
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

template <int kCtrl>
__device__ inline float quad_move(float x)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kCtrl, 0xf, 0xf, true));
}

// E of every (distinct length, instance).  A workgroup takes a run of kMemoP positions of the class
// order and a block of kMemoU consecutive distinct lengths ("rows", ascending), a wave four of the
// positions, a lane four rows.  The segment of a row is k = #{R_i <= L}.  The instance's lengths R
// and the rows are both sorted: the last of every eight lengths (a lane each; tables of up to 512 are read whole, eight
// lengths a lane, and kept in LDS) says where the entries of the block begin to within eight, and the entries from there on
// (a lane each, almost always one read) add one to the counter of the first row that is at least as long; a prefix sum
// over the counters gives k for every row.  The four instances of a wave are in flight together.
//
// What bounds it is the chain of reads a workgroup begins with (instance; its lengths; the entries' rows; the
// segments), then the vector ALU and the store.  A lane has four rows of four positions: the values are
// turned in LDS, so that the store is consecutive, and the least of a run is taken on the way out.  A run's blocks are
// all on one XCD (every eighth workgroup), whose L2 then has its instances' tables.  Kernel time, us, on 4 096 instances of 512
// requests 2 726 rows 25, 7 061 rows 33 (its 117 MB at the rate of a copy 23); 1 024 x 1 000, 3 900 rows 15.5; 256 x 512 8.2.
// With two searches per instance (splitters, then a stride), 64 entries at a time, 30 / 46 / 18.6 / 11.2, without the XCDs 31 / 43 / 17.5 / 8.5.
// A workgroup for several blocks, the next one's entries on their way: 104 registers, 27 / 43 / 21.5 / 9.0.  Workgroups for blocks
// that are not there cost nothing (four rounds of workgroups and blocks in a loop: 42.5 instead of 41).
constexpr int kMemoPerSimd = 7;     // waves per SIMD
constexpr int kMemoWaves = kBlock / kWave;
constexpr unsigned kMemoRound = kSimds * kMemoPerSimd / kMemoWaves;      // workgroups on the chip at once
constexpr int kMemoInst = kMemoP / kMemoWaves;      // instances of a wave
static_assert(kMemoU == 4 * kWave, "a lane owns four consecutive rows");

// The class order by each workgroup itself, on fleets small enough for that (dense_rows; a launch of its own takes 5 us,
// this 2): everything a workgroup needs comes with one read, a thread then counts for one of the class's
// instances over a share of the others.
constexpr int kOwnClass = 128;       // most instances of a class
constexpr int kOwnSlots = 2 * kBlock;    // most positions of the fleet

struct OwnLds {
    uint32_t rough[kOwnSlots];           // the keys as single precision: in the same order or equal; all ones where there is no instance
    __align__(16) unsigned long long key[kOwnSlots];
    int inst[kOwnSlots];
    int rank[kOwnClass];
    int slot[kMemoP];      // the slot of each of the run's positions, -1: none
    uint4 head[kOwnSlots / kMemoP];      // as gr_fleet::run_head
};

// a key (falling_bits) to single precision
__device__ inline uint32_t rough_key(unsigned long long key)
{
    const unsigned long long b = (key >> 63) ? key : ~key ^ 0x8000000000000000ull;
    const uint32_t f = __float_as_uint((float)__longlong_as_double((long long)b));
    return ~(f ^ ((f >> 31) ? 0xFFFFFFFFu : 0x80000000u));
}

// What the keys in full say where the rough ones are equal: of the slots h0 .. h1 of this lane's class (from slot `first` on), how
// many have its rough key and come before its own, `me`.  `tied`: the lane has an equal there.  All lanes of a wave
// together, a rough key at a time: a lane looks at a slot, and equal keys (idle instances) are in the order of their slots.
// (A lane that goes through its class by itself, with two instructions of 64 bits a slot, made one equal pair among
// 256 instances cost 7 us, the table 18 us instead of 11.)
__device__ __forceinline__ int tied_before(const OwnLds& l, bool tied, int first, int me, int h0, int h1)
{
    unsigned long long open = __ballot(tied);
    if (!open) return 0;
    const auto lane_of = [](unsigned long long v, int lane) {
        return ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), lane) << 32) |
               (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
    };
    const int lane = lane_id();
    const uint32_t rough = l.rough[first + me];
    const unsigned long long key = l.key[first + me];
    int less = 0;
    while (open) {
        const int t = __ffsll((long long)open) - 1;
        const int f = __builtin_amdgcn_readlane(first, t), b = __builtin_amdgcn_readlane(h0, t), e = __builtin_amdgcn_readlane(h1, t);
        const uint32_t r = (uint32_t)__builtin_amdgcn_readlane((int)rough, t);
        const unsigned long long kt = lane_of(key, t);
        const bool with = tied && first == f && rough == r;
        for (int h = b; h < e; h += kWave) {
            const int at = f + min(h + lane, e - 1);
            const unsigned long long k = l.key[at];
            unsigned long long equal = __ballot(h + lane < e && l.rough[at] == r);
            if (!__any(with && key != kt) && !(equal & ~__ballot(k == kt))) {
                const int n = min(max(me - h, 0), kWave);
                less += with ? __popcll(n < kWave ? equal & ((1ull << n) - 1ull) : equal) : 0;
                continue;
            }
            for (; equal; equal &= equal - 1) {
                const int m = __ffsll((long long)equal) - 1;
                const unsigned long long km = lane_of(k, m);
                less += with && (km < key || (km == key && h + m < me));
            }
        }
        open &= ~__ballot(with);
    }
    return less;
}

__device__ __forceinline__ void own_order(const OrderArgs& a, int run, OwnLds& l)
{
    const int tid = threadIdx.x;
    const int2 rc = a.run_cls[run];      // first position, instances of the class
#pragma unroll
    for (int s = tid; s < kOwnSlots; s += kBlock) {
        const unsigned long long k = a.key[min(s, a.m_pos - 1)];
        const int g = a.slot_inst[min(s, a.m_pos - 1)];
        l.key[s] = k;
        l.inst[s] = g;
        l.rough[s] = g >= 0 ? rough_key(k) : ~0u;
    }
    if (tid < kOwnClass) l.rank[tid] = 0;
    if (tid < kMemoP) l.slot[tid] = -1;
    __syncthreads();
    // by the keys in single precision; hardly any two are equal, or all of them are (idle instances)
    const int n = rc.y, per = n <= kWave ? kWave : kOwnClass, parts = kBlock / per;
    const int me = min(tid % per, n - 1), step = ((n + parts - 1) / parts + 3) & ~3, h0 = tid / per * step, h1 = min(h0 + step, n);
    const uint32_t own = l.rough[rc.x + me];
    int less = 0, same = 0;
#pragma unroll 4
    for (int h = h0; h < h1; h += 4) {      // (a class is padded to 16 slots)
        const uint4 k = *reinterpret_cast<const uint4*>(l.rough + rc.x + h);
        less += (k.x < own) + (k.y < own) + (k.z < own) + (k.w < own);
        same += (k.x == own) + (k.y == own) + (k.z == own) + (k.w == own);
    }
    less += tied_before(l, same > (me >= h0 && me < h1), rc.x, me, h0, h1);
    if (tid % per < n && less) atomicAdd(&l.rank[me], less);
    __syncthreads();
    if (tid < n) {
        const int p = l.rank[tid] + rc.x - run * kMemoP;
        if (p >= 0 && p < kMemoP) l.slot[p] = rc.x + tid;
    }
    __syncthreads();
}

// The first instance of every run, from the ranks of all instances in their classes (of the workgroups that write
// the order down; own_order has read the keys).
__device__ __forceinline__ void own_heads(const OrderArgs& a, OwnLds& l)
{
    for (int s0 = 0; s0 < a.m_pos; s0 += kBlock) {
        const int s = min(s0 + (int)threadIdx.x, a.m_pos - 1);
        const int2 rc = a.run_cls[s / kMemoP];
        const uint32_t own = l.rough[s];
        int less = 0, same = 0;
#pragma unroll 4
        for (int h = 0; h < rc.y; h += 4) {
            const uint4 k = *reinterpret_cast<const uint4*>(l.rough + rc.x + h);
            less += (k.x < own) + (k.y < own) + (k.z < own) + (k.w < own);
            same += (k.x == own) + (k.y == own) + (k.z == own) + (k.w == own);
        }
        const bool there = l.inst[s] >= 0;
        less += tied_before(l, there && same > 1, rc.x, s - rc.x, 0, rc.y);
        if (there && less % kMemoP == 0)
            l.head[(rc.x + less) / kMemoP] = make_uint4((uint32_t)l.key[s], (uint32_t)(l.key[s] >> 32), (uint32_t)l.inst[s], 0u);
    }
    __syncthreads();
}

// For each position of a run, how many runs begin with a more capable instance: 16 lanes each.  And what the
// selection needs of the run: its least and largest delta (gamma is the same for all of a class) and its lowest instance.
//
// Where the workgroups make the class order themselves (kOwn), this one writes it down for the selection.
template <bool kOwn>
__device__ __forceinline__ void rank_run(const MemoArgs& a, int run, int* lds)
{
    for (int i = run * kBlock + threadIdx.x; i < a.seen_words; i += a.n_run * kBlock) a.seen[i] = make_uint4(0u, 0u, 0u, 0u);
    // (a pass that counts the flagged requests here clears totals[2] when all of the workgroup have read it)
    if (run == 0 && threadIdx.x == 0 && !a.count.totals) a.totals[2] = 0;
    static_assert(kBlock == kMemoP * kMemoP, "16 lanes per position of the run");
    if (run == 0 && a.count.totals) count_flagged(a.count, kBlock, lds);
    const int p = run * kMemoP + threadIdx.x / kMemoP, sub = threadIdx.x % kMemoP;
    unsigned long long key;
    int g, gi;
    float2 kk;
    uint32_t n = 0;
    if constexpr (kOwn) {
        __syncthreads();
        OwnLds& l = *reinterpret_cast<OwnLds*>(lds);
        own_order(a.own, run, l);
        const int s = l.slot[threadIdx.x / kMemoP], si = l.slot[sub];
        g = s >= 0 ? l.inst[s] : -1;
        gi = si >= 0 ? l.inst[si] : -1;
        key = s >= 0 ? l.key[s] : ~0ull;
        kk = make_float2(__builtin_inff(), 0.f);
        if (gi >= 0) { const float4 k = a.instK[gi]; kk = make_float2(k.x, k.y); }
        own_heads(a.own, l);
#pragma unroll
        for (int r = sub; r < kOwnSlots / kMemoP; r += kMemoP) {
            const uint4 h = l.head[r];
            const unsigned long long hk = ((unsigned long long)h.y << 32) | h.x;
            n += r < a.n_run && (hk < key || (hk == key && (int)h.z < g));
        }
        if (sub == 0) {
            a.own.order[p] = g;
            a.own.posKey[p] = key;
            if (g >= 0) a.own.pos_of[g] = p;
            if (p % kMemoP == 0) a.own.run_head[run] = make_uint4((uint32_t)key, (uint32_t)(key >> 32), (uint32_t)g, 0u);
        }
        if (threadIdx.x < kMemoP) a.own.posK[run * kMemoP + sub] = kk;
    } else {
        key = a.posKey[p];
        g = a.order[p];
        kk = a.posK[run * kMemoP + sub];
        gi = a.order[run * kMemoP + sub];
        constexpr int kAhead = 8;
        for (int r0 = sub; r0 < a.n_run; r0 += kAhead * kMemoP) {
            uint4 h[kAhead];
#pragma unroll
            for (int i = 0; i < kAhead; ++i) h[i] = a.run_head[min(r0 + i * kMemoP, a.n_run - 1)];
#pragma unroll
            for (int i = 0; i < kAhead; ++i) {
                const unsigned long long hk = ((unsigned long long)h[i].y << 32) | h[i].x;
                n += r0 + i * kMemoP < a.n_run && (hk < key || (hk == key && (int)h[i].z < g));
            }
        }
    }
    float lo = kk.x, hi = gi >= 0 ? kk.x : -__builtin_inff();
    float gm = gi >= 0 ? kk.y : 0.f;
    int low = gi >= 0 ? gi : 0x7fffffff;
#pragma unroll
    for (int d = 1; d < kMemoP; d <<= 1) {
        n += __shfl_xor(n, d, kMemoP);
        lo = fminf(lo, __shfl_xor(lo, d, kMemoP));
        hi = fmaxf(hi, __shfl_xor(hi, d, kMemoP));
        gm = fmaxf(gm, __shfl_xor(gm, d, kMemoP));
        low = min(low, __shfl_xor(low, d, kMemoP));
    }
    if (sub == 0) {
        a.pos_thr[p] = n;
        if (threadIdx.x == 0) {
            a.run_rank[run] = n;
            a.run_at[n] = run;
            a.run_k[run] = make_float4(lo, gm, hi, __int_as_float(low));
        }
    }
}

// Rows of the tile in LDS are kTileRow words apart, and a row's four pieces change places every 16 rows: the lanes'
// writes (four rows of 16 bytes each, 80 words from lane to lane) and the consecutive reads both spread over the banks.
constexpr int kTileRow = kMemoP + 4;
__device__ inline int tile_at(int row, int piece) { return row * kTileRow + 4 * (piece ^ ((row >> 4) & 3)); }

// kDense: every length up to the largest has a row (see dense_rows): no list, no row numbers to look up.
//
// kSparse: an instance has few entries in a block of rows (see sparse_rows); where a wave's four have up to kFewEntries, none of
// which is the last of its 64, the rows go through those one after the other, and the segments come with the entries: no rows
// of the entries to look up, no counters, no gather.  Scan of 4 096 instances x 512 with long tails, 7 061 rows, in turn on one card:
// 106.3 us without, 100.3 this way with six waves per SIMD (seven spill 16 bytes a lane, 18 MB written: 3.7 us more).  Up to 24 or 32 entries
// 99.8 and 99.3, but spread evenly, four an instance, 153 and 154 instead of 146.5; 48 and more lose there and at eight.
constexpr int kFewEntries = 16;
constexpr int kSparsePerSimd = 6;

template <int kEighths, bool kBlocks, bool kDense, bool kOwn, bool kSparse>     // kEighths x 64 eighths of an instance's lengths at most
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kSparse ? kSparsePerSimd : kMemoPerSimd, kSparse ? kSparsePerSimd : kMemoPerSimd))) void k_memo(MemoArgs a)
{
    if constexpr (kDense) fetch_args<MemoArgs>();
    __shared__ __align__(16) int lds[kMemoU * kTileRow];       // the counters, then the tile
    static_assert(kMemoU * kTileRow >= kMemoWaves * kMemoInst * kMemoU, "room for the counters");
    // (the first workgroups rank the runs for the selection: next to the others, not behind them)
    const int pass = (int)blockIdx.y - 1, run = blockIdx.x;
    if (run >= a.n_run) return;
    if (pass < 0) return rank_run<kOwn>(a, run, lds);
    const int tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int ub = pass * kMemoU, p0 = run * kMemoP + wave * kMemoInst;
    // Past the first round of workgroups the number of rows is in the scalar cache: those without rows end at once, not behind
    // the reads below (a list of rows that nobody has written comes from memory).  Heavy fleet, scan with its build
    // 120.0 -> 114.6 us, refresh and route 78.8 -> 74.6; in the first round the check would be one more thing to wait for.
    if (!kDense && blockIdx.y * gridDim.x >= kMemoRound && ub >= a.totals[1]) return;

    int g[kMemoInst], gs[kMemoInst];
    if constexpr (kOwn) {
        static_assert(sizeof(OwnLds) <= sizeof lds, "the order is made where the counters will be");
        OwnLds& l = *reinterpret_cast<OwnLds*>(lds);
        own_order(a.own, run, l);
#pragma unroll
        for (int j = 0; j < kMemoInst; ++j) {
            const int s = __builtin_amdgcn_readfirstlane(l.slot[wave * kMemoInst + j]);
            g[j] = s >= 0 ? __builtin_amdgcn_readfirstlane(l.inst[s]) : -1;
        }
        __syncthreads();
    } else {
#pragma unroll
        for (int j = 0; j < kMemoInst; ++j) g[j] = a.order[p0 + j];
    }
    // this lane's rows, the length before the block, the wave's instances: one trip, and the number of rows with it
    int4 r;
    int L_before = ub - 1, L_last = 0, U = a.bins;      // the lengths before the block's first row and of its last
    if constexpr (kDense) {
        r = make_int4(ub + 4 * lane, ub + 4 * lane + 1, ub + 4 * lane + 2, ub + 4 * lane + 3);
    } else {
        r = *reinterpret_cast<const int4*>(a.row_len + ub + 4 * lane);
        if (ub > 0) L_before = a.row_len[ub - 1];
        if constexpr (kSparse) L_last = a.row_len[ub + kMemoU - 1];
        U = a.totals[1];
        asm volatile("" : "+v"(r.x), "+v"(r.y), "+v"(r.z), "+v"(r.w));
        if (ub >= U) return;
        if (kSparse && U - ub < kMemoU) L_last = kMaxLen;
    }
    const int2 rc = a.run_cls[run];
    const int here = rc.x + rc.y - run * kMemoP;      // positions of the run that have an instance (or more)
    const int ue = ub + kMemoU;

    float4 K[kMemoInst];
    const uint16_t* R[kMemoInst];
    // Of each instance the 64 entries from kb on, this lane's.  kb: entries before the block, less up to seven.  (0xFFFF:
    // behind the instance's table.)
    int* const cnt = lds + wave * kMemoInst * kMemoU;
    int kb[kMemoInst], er[kMemoInst];
    float2 seg[kMemoInst];
#pragma unroll
    for (int j = 0; j < kMemoInst; ++j) {
        gs[j] = max(g[j], 0);
        K[j] = a.instK[gs[j]];
        R[j] = a.tabR + (size_t)gs[j] * a.cap;
    }
    if constexpr (kEighths == 1) {
        // all of the lengths, eight a lane, and through LDS (where the counters will be) those from kb on
        static_assert(kWave * sizeof(uint4) == kMemoU * sizeof(int), "an instance's lengths fit where its counters will be");
        uint4 w[kMemoInst];
#pragma unroll
        for (int j = 0; j < kMemoInst; ++j) w[j] = reinterpret_cast<const uint4*>(R[j])[min(lane, a.cap / 8 - 1)];
#pragma unroll
        for (int j = 0; j < kMemoInst; ++j) {
            kb[j] = min(8 * __popcll(__ballot((int)(w[j].w >> 16) <= L_before)), a.cap);      // (past the table: the last ones again)
            if constexpr (kSparse) seg[j] = a.tabGH[gh_at(gs[j], kb[j], a.cap) + lane];      // (segment kb + lane: what is before that entry has left)
            reinterpret_cast<uint4*>(cnt + j * kMemoU)[lane] = w[j];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int j = 0; j < kMemoInst; ++j) er[j] = reinterpret_cast<const uint16_t*>(cnt + j * kMemoU)[min(kb[j] + lane, 8 * kWave - 1)];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        static_assert(!kSparse, "the segments come with the entries only where the lengths are read whole");
        int eighth[kMemoInst][kEighths];
#pragma unroll
        for (int j = 0; j < kMemoInst; ++j) {
#pragma unroll
            for (int c = 0; c < kEighths; ++c) eighth[j][c] = R[j][(unsigned)min(8 * (lane + c * kWave) + 7, a.cap - 1)];      // (past the table: the last one again)
        }
#pragma unroll
        for (int j = 0; j < kMemoInst; ++j) {
            int n = 0;
#pragma unroll
            for (int c = 0; c < kEighths; ++c) n += __popcll(__ballot(eighth[j][c] <= L_before));
            kb[j] = min(8 * n, a.cap);
            er[j] = R[j][(unsigned)(kb[j] + lane)];      // (what lies behind the instance's table is read as well)
        }
    }
#pragma unroll
    for (int j = 0; j < kMemoInst; ++j)
        if (lane >= a.cap - kb[j]) er[j] = 0xFFFF;
    float Lf[4], tri[4];
    {
        const int L[4] = {r.x, r.y, r.z, r.w};        // (past the last row: whatever is there, never read)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            Lf[i] = (float)L[i];
            tri[i] = Lf[i] * (Lf[i] - 1.0f) * 0.5f;
        }
    }
    float E[4][kMemoInst];
    bool few = false;
    if constexpr (kSparse) {
        unsigned long long in[kMemoInst];
        int begin[kMemoInst], n_in = 0;
        bool more = false;
#pragma unroll
        for (int j = 0; j < kMemoInst; ++j) {
            const unsigned long long up_to = __ballot(er[j] <= L_last), before = __ballot(er[j] <= L_before);
            in[j] = up_to & ~before;
            begin[j] = __popcll(before);
            n_in += __popcll(in[j]);
            more = more || (in[j] >> (kWave - 1));
        }
        few = n_in <= kFewEntries && !more;
        if (few) {
            const auto lane_of = [](float x, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l)); };
#pragma unroll
            for (int j = 0; j < kMemoInst; ++j) {
                const int N1 = entries_of(K[j]) + 1 - kb[j];
                float Gq[4], H[4], curve[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    Gq[i] = lane_of(seg[j].x, begin[j]); H[i] = lane_of(seg[j].y, begin[j]); curve[i] = K[j].z * (float)(N1 - begin[j]);
                }
                for (; in[j]; in[j] &= in[j] - 1) {
                    const int l = __ffsll((long long)in[j]);      // (its segment is that of the next lane)
                    const float R_l = (float)__builtin_amdgcn_readlane(er[j], l - 1);
                    const float g_l = lane_of(seg[j].x, l), h_l = lane_of(seg[j].y, l), c_l = K[j].z * (float)(N1 - l);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const bool left = R_l <= Lf[i];
                        Gq[i] = left ? g_l : Gq[i]; H[i] = left ? h_l : H[i]; curve[i] = left ? c_l : curve[i];
                    }
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) E[i][j] = fmaf(tri[i], curve[i], fmaf(Lf[i], H[i], Gq[i]));
            }
        }
    }
    if (!few) {
#pragma unroll
        for (int j = 0; j < kMemoInst; ++j) reinterpret_cast<int4*>(cnt + j * kMemoU)[lane] = make_int4(0, 0, 0, 0);
#pragma unroll
        for (int j = 0; j < kMemoInst; ++j)
            if (!kDense) er[j] = a.len_row[(unsigned)min(er[j], a.bins)];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int j = 0; j < kMemoInst; ++j) {
            const bool in = (unsigned)(er[j] - ub) < (unsigned)kMemoU;
            if (in) atomicAdd(&cnt[j * kMemoU + er[j] - ub], 1);
            const int from = kb[j] + kWave;
            kb[j] += __popcll(__ballot(er[j] < ub));
            // more than 64 are in the block (the shortest lengths): 512 at a time
            if (!(__ballot(in) >> (kWave - 1))) continue;
            for (int e0 = from; e0 < a.cap; e0 += 8 * kWave) {
                const int e = e0 + 8 * lane;
                uint4 w = make_uint4(~0u, ~0u, ~0u, ~0u);
                if (e < a.cap) w = *reinterpret_cast<const uint4*>(R[j] + (unsigned)e);
                const uint32_t words[4] = {w.x, w.y, w.z, w.w};
                int row[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    row[i] = (int)(i % 2 ? words[i / 2] >> 16 : words[i / 2] & 0xFFFFu);
                    if (!kDense) row[i] = a.len_row[(unsigned)min(row[i], a.bins)];
                }
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (row[i] < ue) atomicAdd(&cnt[j * kMemoU + row[i] - ub], 1);       // (in order: none is before the block)
                if (__builtin_amdgcn_readlane(row[7], kWave - 1) >= ue) break;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        int k[kMemoInst][4];
        float2 gh[kMemoInst][4];
#pragma unroll
        for (int j = 0; j < kMemoInst; ++j) {
            int4 c = reinterpret_cast<const int4*>(cnt + j * kMemoU)[lane];
            c.y += c.x; c.z += c.y; c.w += c.z;
            const int before = kb[j] + wave_incl_scan_i32(c.w) - c.w;
            k[j][0] = before + c.x; k[j][1] = before + c.y; k[j][2] = before + c.z; k[j][3] = before + c.w;
            const char* __restrict__ GH = reinterpret_cast<const char*>(a.tabGH + gh_at(gs[j], 0, a.cap));
#pragma unroll
            for (int i = 0; i < 4; ++i) gh[j][i] = *reinterpret_cast<const float2*>(GH + (unsigned)k[j][i] * (unsigned)sizeof(float2));
        }
#pragma unroll
        for (int j = 0; j < kMemoInst; ++j) {
            const int N1 = entries_of(K[j]) + 1;
#pragma unroll
            for (int i = 0; i < 4; ++i) E[i][j] = fmaf(tri[i], K[j].z * (float)(N1 - k[j][i]), fmaf(Lf[i], gh[j][i].y, gh[j][i].x));
        }
    }
    __syncthreads();        // (every wave has its counters)
#pragma unroll
    for (int i = 0; i < 4; ++i)
        *reinterpret_cast<float4*>(lds + tile_at(4 * lane + i, wave)) = make_float4(E[i][0], E[i][1], E[i][2], E[i][3]);
    __syncthreads();
    float* __restrict__ out = a.memo + memo_at(ub, run, a.n_run);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int c = tid + i * kBlock, row = c / 4;
        float4 e = *reinterpret_cast<const float4*>(lds + tile_at(row, c % 4));
        if (here < kMemoP) {      // (the end of a class)
            const float inf = __builtin_inff();
            const int q = 4 * (c % 4);
            e = make_float4(q < here ? e.x : inf, q + 1 < here ? e.y : inf, q + 2 < here ? e.z : inf, q + 3 < here ? e.w : inf);
        }
        reinterpret_cast<float4*>(out)[c] = e;
        float m = min_plain(min_plain(e.x, e.y), min_plain(e.z, e.w));
        m = min_plain(m, quad_move<0xB1>(m));      // quad_perm [1,0,3,2], [2,3,0,1]
        m = min_plain(m, quad_move<0x4E>(m));
        if (c % 4 == 0 && ub + row < U) a.grp_min[runs_at<kBlocks>(ub + row, a.run_pad) + (size_t)run * kRunStride<kBlocks>] = m;
    }
}

// ------------------------------------------------------------------ Alg. 1, runs first
constexpr int kGroup = 16;       // lanes that take a request together: a run's positions, or 16 runs
static_assert(kGroup == kMemoP, "a lane per position of a run");

// Bit i: lane i of this lane's group of kGroup.
__device__ inline uint32_t group_ballot(bool v)
{
    return (uint32_t)(__ballot(v) >> (lane_id() & (kWave - kGroup))) & 0xFFFFu;
}

// Value of lane `l` of this lane's group.
template <typename T>
__device__ inline T group_lane(T v, int l) { return __shfl(v, l, kGroup); }

struct ClassArgs {
    const int* totals;
    const int2* cls_run;
    const int* order;
    const float *memo, *grp_min;
    const float4* run_k;
    float* row_min;       // see k_class
    const int* row_len;
    uint2* class_least;   // see class_at
    const uint32_t* run_rank;
    uint32_t* cls_rank;   // of each class's first run
    int n_class, class_shift, n_run, run_pad;
};

// What decides most requests of a large batch is kept by length, not by row: the least E of every class, and in one word the lowest
// instance that has it and the exponent of the distance to the next larger E (which says whether rounding may have made the two
// latencies equal).  A length's classes are 16, 32, 64 or 128 bytes together, and the lanes of a request read them side by side.
__device__ inline size_t class_at(int L, int shift) { return (size_t)L << shift; }
constexpr int kLowBits = 20, kCountAt = 28;      // bits of the instance (gr_create takes no more); see ClassesOf::least
__device__ inline uint32_t low_and_gap(int low, float least, float next)
{
    return ((__float_as_uint(next - least) >> 23 & 0xFFu) << kLowBits) | ((uint32_t)low & ((1u << kLowBits) - 1u));
}

// Per row and class: the least E, the lowest instance that has it, and the least E above it among
// what could still change the answer.  Without a blend the prefill part is the same for all of a
// class, so these decide a request's least latency (k_select).  A workgroup takes 64 rows and one
// class, a lane per row (the reads are whole cache lines) and a quarter of the class's runs per wave: the
// runs first, then four positions per wave of the run that holds the least E.
//
// kRows: the runs' minima are left row by row as well, for a selection many of whose requests get as far as the runs (a
// request's 16 lanes read 16 runs from one cache line).  They pass here anyway and are turned in LDS; written row by row
// by the table's workgroups, four bytes to a line, they cost the table 3 us of 26 and this kernel's reads 2 of 7.5 (refresh and 262 144
// requests, 4 096 instances: 70.4 us before, 68.4 with both; in blocks alone 66.6, but 101.5 instead of 94.2 with deadlines that many meet).
template <bool kRows>
__global__ __launch_bounds__(kBlock) void k_class(ClassArgs a)
{
    constexpr int kW = kBlock / kWave, kAhead = 8, kCols = kAhead * kW;
    __shared__ float turned[kRows ? kWave * (kCols + 1) : 1];
    static_assert(kMemoU % kWave == 0, "the rows of a workgroup are in one block");
    __shared__ float m1_lds[kW][kWave], m2_lds[kW][kWave];
    __shared__ int r1_lds[kW][kWave], low_lds[kW][kWave];
    const int lane = lane_id(), w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int c = blockIdx.x % a.n_class;
    const int64_t u0 = (int64_t)(blockIdx.x / a.n_class) * kWave, u = u0 + lane;
    const int U = a.totals[1];
    if (u0 >= U) return;
    const int2 cr = a.cls_run[c];
    const int L = a.row_len[min(u, (int64_t)U - 1)];
    const float inf = __builtin_inff();
    if (u0 == 0 && threadIdx.x == 0) a.cls_rank[c] = cr.y ? a.run_rank[cr.x] : ~0u;
    const float* __restrict__ runs = a.grp_min + runs_at<true>(min(u, (int64_t)U - 1), a.run_pad) + (size_t)cr.x * kRunStride<true>;
    const float* __restrict__ E = a.memo + memo_at(u, cr.x, a.n_run);
    const int* __restrict__ order = a.order + cr.x * kMemoP;

    float m1 = inf, m2 = inf;       // of this wave's runs: the least, the least of the others
    int r1 = 0;
    for (int b = 0; b < cr.y; b += kCols) {
        const int r0 = b + w;
        float e[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) e[k] = runs[(size_t)min(r0 + k * kW, cr.y - 1) * kRunStride<true>];
        if constexpr (kRows) {
            if (b) __syncthreads();
#pragma unroll
            for (int k = 0; k < kAhead; ++k) turned[lane * (kCols + 1) + k * kW + w] = e[k];
        }
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            const int r = r0 + k * kW;
            if (r >= cr.y) break;
            if (e[k] < m1) { m2 = m1; m1 = e[k]; r1 = r; }
            else m2 = fminf(m2, e[k]);
        }
        if constexpr (kRows) {
            __syncthreads();
            const int col = threadIdx.x % kCols;
            float* __restrict__ out = a.row_min + (size_t)u0 * a.run_pad + cr.x + b + col;
#pragma unroll
            for (int i = 0; i < kWave * kCols / kBlock; ++i) {
                const int row = threadIdx.x / kCols + i * (kBlock / kCols);
                if (b + col < cr.y && u0 + row < U) out[(size_t)row * a.run_pad] = turned[row * (kCols + 1) + col];
            }
        }
    }
    m1_lds[w][lane] = m1; m2_lds[w][lane] = m2; r1_lds[w][lane] = r1;
    __syncthreads();
    float E1 = inf, above = inf;
    int tied = 0;                   // runs that hold the least E
    r1 = 0;
#pragma unroll
    for (int q = 0; q < kW; ++q)
        if (m1_lds[q][lane] < E1) { E1 = m1_lds[q][lane]; r1 = r1_lds[q][lane]; }
#pragma unroll
    for (int q = 0; q < kW; ++q) {
        const float x = m1_lds[q][lane], y = m2_lds[q][lane];
        tied += (x == E1) + (y == E1);
        if (x > E1) above = fminf(above, x);
        if (y > E1) above = fminf(above, y);
    }
    const bool any = u < U && E1 < inf;
    int low = 0x7fffffff;
    const auto take = [&](int r, int piece) {      // four positions of a run
        const float4 v = *reinterpret_cast<const float4*>(E + (size_t)r * kTile + 4 * piece);
        const int4 g = *reinterpret_cast<const int4*>(order + r * kMemoP + 4 * piece);
        const auto one = [&](float v, int g) {
            if (g < 0) return;
            if (v > E1) above = fminf(above, v);
            else if (v == E1) low = min(low, g);
        };
        one(v.x, g.x); one(v.y, g.y); one(v.z, g.z); one(v.w, g.w);
    };
    static_assert(kMemoP == 4 * kW, "four positions per wave");
    if (any) take(r1, w);
    low_lds[w][lane] = low;
    if (__syncthreads_or(any && tied > 1)) {
        // Several runs hold the least E: those are looked at as well, unless all of a run's instances
        // come behind the one at hand (where another latency of such a run ties with the least one, the
        // instance at hand wins as well).
        if (any && tied > 1) {
            int low1 = low_lds[0][lane];
#pragma unroll
            for (int q = 1; q < kW; ++q) low1 = min(low1, low_lds[q][lane]);
            for (int r = w; r < cr.y; r += kW) {
                const float e = runs[(size_t)r * kRunStride<true>];
                if (e > E1) above = fminf(above, e);
                else if (r != r1 && __float_as_int(a.run_k[cr.x + r].w) < low1)
                    for (int q = 0; q < kW; ++q) take(r, q);
            }
        }
        __syncthreads();
        low_lds[w][lane] = low;
    }
    m2_lds[w][lane] = above;
    __syncthreads();
    if (w != 0 || u >= U) return;
#pragma unroll
    for (int q = 1; q < kW; ++q) {
        low = min(low, low_lds[q][lane]);
        above = fminf(above, m2_lds[q][lane]);
    }
    a.class_least[class_at(L, a.class_shift) + c] = make_uint2(__float_as_uint(E1), low_and_gap(low, E1, above));
}

struct SelectArgs {
    ReqSrc s;
    const uint16_t* len_row;
    const int* order;
    const float *memo, *grp_min;
    const float4* run_k;
    const float2* posK;
    const unsigned long long* posKey;
    const uint32_t *run_rank, *pos_thr;
    const int* run_at;
    const int2* cls_run;
    const uint2* class_least;
    const float2* clsK;
    const uint32_t* cls_rank;
    float4* lines;           // see k_lines
    int *rest, *rest_cnt;    // see k_select_lines
    const int *totals, *row_len, *pos_of;
    int* out_inst;
    float* out_slack;
    uint8_t* out_fallback;
    int run_pad, n_run, n_class, class_shift, max_len, n_inst;
    int segments;      // by classes or lines first: workgroups of the launch
    int64_t first;     // a group of lanes per request: the launch's first request
};

struct Request {
    int L, c0, ex;
    float D;
    bool scored;       // a migration pass scores the flagged requests only
};

template <bool kMigrate>
__device__ __forceinline__ Request fetch(const ReqSrc& s, int64_t i, int max_len)
{
    Request q;
    if (kMigrate) {
        q.L = s.act_rem[i]; q.c0 = s.act_prompt[i] + s.act_gen[i]; q.D = s.act_budget[i]; q.ex = s.act_inst[i];
        q.scored = s.flag[i] != 0;
    } else {
        q.L = s.pred_len[i]; q.c0 = s.ctx0[i]; q.D = s.budget[i]; q.ex = s.exclude ? s.exclude[i] : -1;
        q.scored = true;
    }
    q.L = min(max(q.L, 0), max_len);
    return q;
}

template <bool kMigrate>
__device__ __forceinline__ void answer(const SelectArgs& a, int64_t i, int g, float slack, bool found)
{
    a.out_inst[i] = g;
    a.out_slack[i] = slack;
    if (!kMigrate && a.out_fallback) a.out_fallback[i] = !found;
}

// Alg. 1 for one request by the kGroup lanes of a group, in two moves that take a range of runs.
//
// Feasible choice (scan<true, ., .>): of every run whose bound meets the deadline and whose most capable
// instance would be an improvement, the first feasible position (a run's positions are in
// capability order, and classes of slow steps come first).  The improvement is one comparison: the runs are
// ranked by their first instances, and every position knows how many runs begin with a better one (with
// the d_g themselves, 64 bits and the index on ties, the search took half of the selection's instructions).  Least latency (scan<., true, .>, then
// settle): the run with the least bound is looked at, then every other run whose bound does not
// exceed the least latency at hand (equal ones only if they hold a lower instance).  kChunks x
// kGroup runs are read together: the reads of the runs' values are what a request waits for.
template <int kChunks>
struct Selection {
    const SelectArgs& a;
    const int sub, ex;
    const float* __restrict__ runs;
    const float* __restrict__ E;      // (this lane's position)
    const int* run_at;          // (of a, or a copy in LDS)
    const float4* run_k;
    const float Lf, c0, Dc;
    // the feasible choice so far
    unsigned long long feasKey = ~0ull;
    int feasG = -1;
    float feasT = 0.f;
    uint32_t feasThr = ~0u;      // runs of a smaller rank may hold a better one
    // the least latency so far
    float bestT = __builtin_inff();
    int bestG = -1;
    // of the range scanned last, this lane's least bound, its run, and the least of its other bounds
    float m1, m2;
    int r1;

    __device__ __forceinline__ Selection(const SelectArgs& args, const Request& q, int row, int sub_)
        : a(args), sub(sub_), ex(q.ex), runs(args.grp_min + runs_at<false>(row, args.run_pad)),
          E(args.memo + memo_at(row, 0, args.n_run) + sub_), run_at(args.run_at), run_k(args.run_k), Lf((float)q.L), c0((float)q.c0),
          Dc(q.D > FLT_MAX ? FLT_MAX : q.D) {}

    __device__ __forceinline__ float bound(float e, const float4& k) const
    {
        return fmaf(c0, kappa_of(make_float2(c0 >= 0.f ? k.x : k.z, k.y), Lf), e);
    }

    // kRanked (all runs): by rank, not in class order, so that the search ends where no run can improve the choice;
    // for requests that can be served in time (the runs of a rank lie anywhere in a row: a search that goes
    // through all of them takes 29 us by rank and 23 in class order, 65 536 requests x 4 096 instances).
    template <bool kFeasible, bool kLeast, bool kRanked>
    __device__ __forceinline__ void scan(int first, int n)
    {
        const float inf = __builtin_inff();
        m1 = inf; m2 = inf; r1 = -1;
        for (int r0 = 0; r0 < n; r0 += kChunks * kGroup) {
            if (kRanked && (uint32_t)r0 >= feasThr) break;
            float b[kChunks];
            float4 k[kChunks];
            int run[kChunks];
            uint32_t rank[kChunks];      // (in class order read where there is a run in question)
#pragma unroll
            for (int j = 0; j < kChunks; ++j) {
                const int i = min(r0 + j * kGroup + sub, n - 1);
                run[j] = kRanked ? run_at[i] : first + i;
                if (kRanked) rank[j] = (uint32_t)i;
            }
#pragma unroll
            for (int j = 0; j < kChunks; ++j) {
                b[j] = runs[run[j]];
                k[j] = run_k[run[j]];
            }
            bool any = false;
#pragma unroll
            for (int j = 0; j < kChunks; ++j) {
                b[j] = r0 + j * kGroup + sub < n ? bound(b[j], k[j]) : inf;
                if (kLeast) {
                    if (b[j] < m1) { m2 = m1; m1 = b[j]; r1 = run[j]; }
                    else m2 = fminf(m2, b[j]);
                }
                if (kFeasible) any = any || b[j] <= Dc;
            }
            if (!kFeasible || !__any(any)) continue;
#pragma unroll
            for (int j = 0; j < kChunks; ++j) {
                if (!kRanked) rank[j] = a.run_rank[run[j]];
                if (!(b[j] <= Dc)) rank[j] = ~0u;      // (not, or no longer, in question)
            }
            for (;;) {
                uint32_t at = ~0u;       // the first run in question
#pragma unroll
                for (int j = kChunks - 1; j >= 0; --j) at = rank[j] < feasThr ? j * kGroup + sub : at;
                at = min_over<true>(at);
                if (at == ~0u) break;
                int r = run[0];
#pragma unroll
                for (int j = 0; j < kChunks; ++j) {
                    if (kRanked) r = at / kGroup == (uint32_t)j ? run[j] : r;
                    rank[j] = at == (uint32_t)(j * kGroup + sub) ? ~0u : rank[j];
                }
                r = kRanked ? group_lane(r, at % kGroup) : first + r0 + (int)at;
                const int p = r * kMemoP + sub, g = a.order[p];
                const unsigned long long pk = a.posKey[p];
                const uint32_t thr = a.pos_thr[p];
                const float T = fmaf(c0, kappa_of(a.posK[p], Lf), E[(size_t)r * kTile]);
                const uint32_t hit = group_ballot(T <= Dc && g >= 0 && g != ex);
                if (!hit) continue;
                const int h = __ffs(hit) - 1;
                const unsigned long long hk = group_lane(pk, h);
                const int hg = group_lane(g, h);
                const float hT = group_lane(T, h);
                const uint32_t ht = group_lane(thr, h);
                if (feasG < 0 || hk < feasKey || (hk == feasKey && hg < feasG)) {
                    feasKey = hk; feasG = hg; feasT = hT; feasThr = ht;
                }
            }
        }
    }

    __device__ __forceinline__ void look(int run)
    {
        const int p = run * kMemoP + sub, g = a.order[p];
        const float T = fmaf(c0, kappa_of(a.posK[p], Lf), E[(size_t)run * kTile]);
        const bool in = g >= 0 && g != ex && T < __builtin_inff();
        const float least = from_ordered_bits(min_over<true>(in ? ordered_bits(T) : ~0u));
        if (!group_ballot(in) || least > bestT) return;
        const int low = (int)min_over<true>(in && T == least ? (uint32_t)g : 0x7fffffffu);
        if (least < bestT || low < bestG) { bestT = least; bestG = low; }
    }

    // may a run with this bound still hold the answer?
    __device__ __forceinline__ bool open(int run, float b) const
    {
        return b < bestT || (b == bestT && b < __builtin_inff() && __float_as_int(a.run_k[run].w) < bestG);
    }

    // the least latency of the range scanned last, into the least latency so far
    __device__ __forceinline__ void settle(int first, int n)
    {
        const float inf = __builtin_inff();
        const float least = from_ordered_bits(min_over<true>(ordered_bits(m1)));
        if (least > bestT) return;
        uint32_t mask = group_ballot(m1 == least && m1 < inf);
        if (!mask) return;
        const int l = __ffs(mask) - 1;
        look(group_lane(r1, l));
        mask = group_ballot(m1 <= bestT && m1 < inf) & ~(1u << l);
        while (mask) {
            const int lo = __ffs(mask) - 1;
            mask &= mask - 1;
            const int run = group_lane(r1, lo);
            if (open(run, group_lane(m1, lo))) look(run);
        }
        if (!group_ballot(m2 <= bestT && m2 < inf)) return;
        for (int rb = 0; rb < n; rb += kGroup) {       // some lane has a second run to look at: all runs again
            const int r = first + min(rb + sub, n - 1);
            const float b = rb + sub < n ? bound(runs[r], a.run_k[r]) : inf;
            uint32_t again = group_ballot(b <= bestT && b < inf && r != r1);
            while (again) {
                const int lo = __ffs(again) - 1;
                again &= again - 1;
                if (open(first + rb + lo, group_lane(b, lo))) look(first + rb + lo);
            }
        }
    }

    template <bool kMigrate>
    __device__ __forceinline__ void report(int64_t i, float D) const
    {
        if (sub != 0) return;
        if (feasG >= 0) answer<kMigrate>(a, i, feasG, D - feasT, true);
        else answer<kMigrate>(a, i, bestG, bestG >= 0 ? D - bestT : 0.f, false);
    }
};

// A group of lanes per request.
template <bool kMigrate, int kChunks>
__global__ __launch_bounds__(kBlock) void k_select(SelectArgs a)
{
    fetch_args<SelectArgs>();
    const int sub = threadIdx.x % kGroup;
    const int64_t i = a.first + (int64_t)blockIdx.x * (kBlock / kGroup) + threadIdx.x / kGroup;
    if (i >= a.s.n) return;
    const Request q = fetch<kMigrate>(a.s, i, a.max_len);
    if (!q.scored) {
        if (sub == 0) answer<kMigrate>(a, i, -1, 0.f, false);      // not flagged: no migration target
        return;
    }
    Selection<kChunks> sel(a, q, row_at(a.len_row, q.L), sub);
    sel.template scan<true, true, false>(0, a.n_run);
    if (sel.feasG < 0) sel.settle(0, a.n_run);
    sel.template report<kMigrate>(i, q.D);
}

// Four lanes per request on fleets of up to kLaneRuns runs.  The bounds of the runs of a request's row stay in
// registers, and a run is looked at by the same lanes, its 16 values being one piece of 64 bytes: about a quarter of the vector
// instructions that 16 lanes per request take, which is what batches of many requests wait for.  Whole calls, us, 16 lanes /
// four / one (fewer instructions still, but a wave for every SIMD at 65 536 requests, and nothing to hide its reads behind):
//   route 256 instances: 32 768 requests 14.9 / 14.3 / 17.4, 65 536 16.9 / 13.6 / 16.2, 262 144 31.8 / 18.3 / 20.6
//   (16 384 13.7 / 14.1 / 17.3); 480: 262 144 45.0 / 28.7 / 31.3, blended 48.3 / 30.3 / 33.5
//   scan 256 x 512 30.4 / 24.8 / 30.8, blended 33.8 / 25.0 / 28.1, 400 x 1 000 70.4 / 47.9 / 53.7
// The answers are Selection's.
constexpr int kLaneRuns = 32;
constexpr int kLanes = 4;

// over the lanes of a request
__device__ __forceinline__ uint32_t lanes_min(uint32_t v)
{
    return min_dpp<0x4E, 0xf>(min_dpp<0xB1, 0xf>(v));      // quad_perm [1,0,3,2], [2,3,0,1]
}

__device__ __forceinline__ uint32_t lanes_or(uint32_t v)
{
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, false);
    return v | (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, false);
}

template <bool kMigrate, int kRuns, bool kBlend>
__global__ __launch_bounds__(kBlock) void k_select_lanes(SelectArgs a)
{
    // of each run: its least delta, gamma, largest delta, its rank as a bit; the run of each rank; delta and gamma by position
    __shared__ float4 of_run[kRuns];
    __shared__ int at_rank[kRuns];
    __shared__ float2 of_pos[kBlend ? kRuns * kMemoP : 1];
    const int tid = threadIdx.x, sub = tid % kLanes;
    if (tid < a.n_run) {
        float4 k = a.run_k[tid];
        k.w = __uint_as_float(1u << a.run_rank[tid]);
        of_run[tid] = k;
        at_rank[tid] = a.run_at[tid];
    }
    if (kBlend)
        for (int p = tid; p < a.n_run * kMemoP; p += kBlock) of_pos[p] = a.posK[p];
    const int64_t i = a.first + ((int64_t)blockIdx.x * kBlock + tid) / kLanes;
    const Request q = fetch<kMigrate>(a.s, min(i, a.s.n - 1), a.max_len);
    const int row = row_at(a.len_row, q.L);
    const int ex_at = q.ex >= 0 && q.ex < a.n_inst ? a.pos_of[q.ex] : -1;
    __syncthreads();
    if (i >= a.s.n) return;
    const auto reply = [&](int g, float slack, bool found) { if (sub == 0) answer<kMigrate>(a, i, g, slack, found); };
    if (!q.scored) return reply(-1, 0.f, false);      // not flagged: no migration target

    // a lane's runs of a row, and its positions of a run: four together, then the other lanes' four
    const auto nth = [&](int x) { return x / 4 * (4 * kLanes) + 4 * sub + x % 4; };
    constexpr int kMine = kRuns / kLanes, kAt = kMemoP / kLanes;
    const float inf = __builtin_inff();
    const float c0 = (float)q.c0, Lf = (float)q.L, Dc = q.D > FLT_MAX ? FLT_MAX : q.D;
    const float* __restrict__ E = a.memo + memo_at(row, 0, a.n_run);
    float b[kMine];
    {
        const float* __restrict__ runs = a.grp_min + (size_t)row * a.run_pad;      // (a row's length is a multiple of 16)
#pragma unroll
        for (int x = 0; x < kMine; x += 4) {
            float4 e = make_float4(0.f, 0.f, 0.f, 0.f);
            if (x / 4 * (4 * kLanes) < a.n_run) e = *reinterpret_cast<const float4*>(runs + nth(x));
            b[x] = e.x; b[x + 1] = e.y; b[x + 2] = e.z; b[x + 3] = e.w;
        }
    }
    float least = inf;
    int least_run = -1;
    uint32_t open = 0;       // by rank: the runs that may hold a feasible instance
#pragma unroll
    for (int x = 0; x < kMine; ++x) {
        const int r = nth(x);
        if (r < a.n_run) {
            const float4 k = of_run[r];
            b[x] = fmaf(c0, kappa_of(make_float2(!kBlend || c0 >= 0.f ? k.x : k.z, k.y), Lf), b[x]);
            if (b[x] < least) { least = b[x]; least_run = r; }
            open |= b[x] <= Dc ? __float_as_uint(k.w) : 0u;
        } else {
            b[x] = inf;
        }
    }
    open = lanes_or(open);
    // every latency of a run, that of the excluded instance infinite
    const auto latencies = [&](int run, float (&T)[kAt]) {
        const float* __restrict__ line = E + (size_t)run * kTile;
#pragma unroll
        for (int x = 0; x < kAt; x += 4) {
            const float4 e = *reinterpret_cast<const float4*>(line + nth(x));
            T[x] = e.x; T[x + 1] = e.y; T[x + 2] = e.z; T[x + 3] = e.w;
        }
        const float4 k = of_run[run];
        const float kappa = kappa_of(make_float2(k.x, k.y), Lf);
        const int ex = ex_at - run * kMemoP;
#pragma unroll
        for (int x = 0; x < kAt; ++x) {
            T[x] = fmaf(c0, kBlend ? kappa_of(of_pos[run * kMemoP + nth(x)], Lf) : kappa, T[x]);
            T[x] = nth(x) == ex ? inf : T[x];
        }
    };
    int feasG = -1;
    float feasT = 0.f;
    unsigned long long feasKey = ~0ull;
    while (open) {       // the most capable run first
        const int run = at_rank[__ffs(open) - 1];
        open &= open - 1;
        float T[kAt];
        latencies(run, T);
        uint32_t hit = kMemoP;
        float hitT = 0.f;
#pragma unroll
        for (int x = kAt - 1; x >= 0; --x)
            if (T[x] <= Dc) { hit = nth(x); hitT = T[x]; }
        const uint32_t first = lanes_min(hit);
        if (first == kMemoP) continue;
        const int p = run * kMemoP + (int)first, g = a.order[p];
        const unsigned long long key = a.posKey[p];
        const uint32_t thr = a.pos_thr[p];
        hitT = from_ordered_bits(lanes_min(hit == first ? ordered_bits(hitT) : ~0u));
        if (feasG < 0 || key < feasKey || (key == feasKey && g < feasG)) {
            feasKey = key; feasG = g; feasT = hitT;
            if (thr < 32) open &= (1u << thr) - 1u;      // (the others begin with nobody better)
        }
    }
    if (feasG >= 0) return reply(feasG, q.D - feasT, true);

    float bestT = inf;
    int bestG = -1;
    const auto look = [&](int run) {
        float T[kAt];
        latencies(run, T);
        float m = inf;
#pragma unroll
        for (int x = 0; x < kAt; ++x) m = min_plain(m, T[x]);
        m = from_ordered_bits(lanes_min(ordered_bits(m)));
        if (!(m < inf) || m > bestT) return;
        uint32_t equal = 0;
#pragma unroll
        for (int x = 0; x < kAt; ++x) equal |= T[x] == m ? 1u << nth(x) : 0u;
        int low = 0x7fffffff;
        for (equal = lanes_or(equal); equal; equal &= equal - 1) low = min(low, a.order[run * kMemoP + __ffs(equal) - 1]);
        if (m < bestT || low < bestG) { bestT = m; bestG = low; }
    };
    // The least bound first, of equal ones that of the first run, until there is somebody (a request whose own instance is all of
    // a run finds nobody there; the few waves of such requests looked at every run for it, a scan of 482 x 512 47 us,
    // this way 30), then the runs that may hold somebody as good.
    for (;;) {
        const uint32_t all_least = lanes_min(ordered_bits(least));
        least_run = (int)lanes_min(least_run >= 0 && ordered_bits(least) == all_least ? (uint32_t)least_run : 0x7fffffffu);
        if (least_run == 0x7fffffff) break;
        look(least_run);
#pragma unroll
        for (int x = 0; x < kMine; ++x) b[x] = nth(x) == least_run ? inf : b[x];
        if (bestG >= 0) break;
        least = inf;
        least_run = -1;
#pragma unroll
        for (int x = 0; x < kMine; ++x)
            if (b[x] < least) { least = b[x]; least_run = nth(x); }
    }
    uint32_t others = 0;
#pragma unroll
    for (int x = 0; x < kMine; ++x) others |= b[x] <= bestT && b[x] < inf ? 1u << nth(x) : 0u;
    for (others = lanes_or(others); others; others &= others - 1) look(__ffs(others) - 1);
    reply(bestG, bestG >= 0 ? q.D - bestT : 0.f, false);
}

// The same where the least E of every class is known, and all of a class have the same prefill part: only the classes, and of
// those the runs, that can hold the answer.  A class's runs are in capability order, so the first run whose least latency meets a
// deadline has the class's choice (unless that is the excluded instance).
//
// Of the requests that large batches leave to this there are one or two to a workgroup, at its end: what it takes is the chain of
// one of them, reads and instructions (a lone wave's take eight cycles each, one after the other).  Kernel time of a scan of 1 024 x 1 000, of
// which one in 600 gets here, 19.6 us with the bounds, ranks and reads of Selection, 15.0 this way; refresh and 262 144 requests on 4 096
// instances, one in 30, 12.5 and 9.4; with deadlines that many meet (x 16) whole calls of 85.3 and 85.7 us, now 69.3 and 70.3.
template <bool kMigrate, bool kBlocks>
__device__ __forceinline__ void select_by_class(const SelectArgs& a, int64_t i, const Request& q, int sub)
{
    constexpr int kChunks = 4;      // times kGroup runs that are read together
    const float inf = __builtin_inff(), c0 = (float)q.c0, Lf = (float)q.L, Dc = q.D > FLT_MAX ? FLT_MAX : q.D;
    const int c = min(sub, a.n_class - 1), row = a.len_row[q.L];
    const float e = __uint_as_float(a.class_least[class_at(q.L, a.class_shift) + c].x);
    const int2 range = a.cls_run[c];
    const float kappa = kappa_of(a.clsK[c], Lf);
    const uint32_t rank = a.cls_rank[c];      // of the class's most capable instance
    const float T_least = sub < a.n_class && e < inf ? fmaf(c0, kappa, e) : inf;
    const float* __restrict__ runs = a.grp_min + runs_at<kBlocks>(row, a.run_pad);
    const float* __restrict__ E = a.memo + memo_at(row, 0, a.n_run) + sub;

    int first, n;      // the runs of the class at hand; its kappa
    float kap;
    const auto enter = [&](int l) { first = group_lane(range.x, l); n = group_lane(range.y, l); kap = group_lane(kappa, l); };
    const auto bounds = [&](int r0, float (&b)[kChunks]) {
#pragma unroll
        for (int j = 0; j < kChunks; ++j) b[j] = runs[(size_t)(first + min(r0 + j * kGroup + sub, n - 1)) * kRunStride<kBlocks>];
#pragma unroll
        for (int j = 0; j < kChunks; ++j) b[j] = r0 + j * kGroup + sub < n ? fmaf(c0, kap, b[j]) : inf;
    };

    unsigned long long feasKey = ~0ull;
    int feasG = -1;
    float feasT = 0.f;
    uint32_t feasThr = ~0u;
    uint32_t left_rank = T_least <= Dc ? rank : ~0u;
    for (;;) {
        const uint32_t top = min_over<true>(left_rank < feasThr ? left_rank : ~0u);      // the most capable of them
        if (top == ~0u) break;
        const int l = __ffs(group_ballot(left_rank == top)) - 1;
        if (sub == l) left_rank = ~0u;
        enter(l);
        for (int r0 = 0; r0 < n; r0 += kChunks * kGroup) {
            float b[kChunks];
            bounds(r0, b);
            unsigned long long open = 0;
#pragma unroll
            for (int j = kChunks - 1; j >= 0; --j) open = (open << kGroup) | group_ballot(b[j] <= Dc);
            uint32_t hit = 0;
            for (; open && !hit; open &= open - 1) {
                const int run = first + r0 + __ffsll((long long)open) - 1, p = run * kMemoP + sub, g = a.order[p];
                const unsigned long long pk = a.posKey[p];
                const uint32_t thr = a.pos_thr[p];
                const float T = fmaf(c0, kap, E[(size_t)run * kTile]);
                hit = group_ballot(T <= Dc && g >= 0 && g != q.ex);
                if (!hit) continue;
                const int h = __ffs(hit) - 1;
                const unsigned long long hk = group_lane(pk, h);
                const int hg = group_lane(g, h);
                const float hT = group_lane(T, h);
                const uint32_t ht = group_lane(thr, h);
                if (feasG < 0 || hk < feasKey || (hk == feasKey && hg < feasG)) {
                    feasKey = hk; feasG = hg; feasT = hT; feasThr = ht;
                }
            }
            if (hit) break;
        }
    }
    if (feasG >= 0) {
        if (sub == 0) answer<kMigrate>(a, i, feasG, q.D - feasT, true);
        return;
    }
    // the least latency: class by class, run by run, as long as the least one left does not exceed what there is
    float bestT = inf, left = T_least;
    int bestG = -1;
    for (;;) {
        const float least = from_ordered_bits(min_over<true>(ordered_bits(left)));
        const uint32_t mask = group_ballot(left == least && left < inf);
        if (!mask || least > bestT) break;
        const int l = __ffs(mask) - 1;
        if (sub == l) left = inf;
        enter(l);
        for (int r0 = 0; r0 < n; r0 += kChunks * kGroup) {
            float b[kChunks];
            bounds(r0, b);
            for (;;) {
                float m = b[0];
#pragma unroll
                for (int j = 1; j < kChunks; ++j) m = fminf(m, b[j]);
                m = from_ordered_bits(min_over<true>(ordered_bits(m)));
                if (!(m <= bestT && m < inf)) break;
                int at = 0;
#pragma unroll
                for (int j = kChunks - 1; j >= 0; --j) {
                    const uint32_t here = group_ballot(b[j] == m);
                    if (here) at = j * kGroup + __ffs(here) - 1;
                }
#pragma unroll
                for (int j = 0; j < kChunks; ++j) b[j] = j * kGroup + sub == at ? inf : b[j];
                const int run = first + r0 + at, p = run * kMemoP + sub;
                if (m == bestT && __float_as_int(a.run_k[run].w) > bestG) continue;      // (nobody at a lower index)
                const int g = a.order[p];
                const float T = fmaf(c0, kap, E[(size_t)run * kTile]);
                const bool in = g >= 0 && g != q.ex && T < inf;
                const float t = from_ordered_bits(min_over<true>(in ? ordered_bits(T) : ~0u));
                if (!group_ballot(in) || t > bestT) continue;
                const int low = (int)min_over<true>(in && T == t ? (uint32_t)g : 0x7fffffffu);
                if (t < bestT || low < bestG) { bestT = t; bestG = low; }
            }
        }
    }
    if (sub == 0) answer<kMigrate>(a, i, bestG, bestG >= 0 ? q.D - bestT : 0.f, false);
}

// With a blend every instance has its own prefill rate, and no least E decides a request.  But for a length and a
// range of prompts hardly ever more than one instance can have the least latency: T is linear in c0, the
// least latency a lower envelope of lines, and the lines cross seldom.  So for every row and each of
// kRanges ranges of c0 the instances that could be least somewhere in it are looked up once, and a request compares those.
//
// With any lines a, b and any c in a range lo .. hi, an instance g whose line is above a's at lo and c and above b's at c
// and hi is above the lesser of the two in all of the range (everything is linear): only the others count.
// a and b are the least of the run with the least bound at lo and at hi, c is where they cross.  "Above" is by 2^-20 of the largest
// value: T as a request forms it is off by 2^-24, so none of those left out can come out less, or equal.
//
// A wave per row and range: on up to 320 runs the bounds are read once, and what is waited for is those, the two
// runs, and the runs in question four at a time (4 096 instances, 4 000 rows: 14 us between events; a group of
// lanes that goes through the runs 64 at a time, three times over, for five ranges: 30).
__device__ constexpr float kRangeEnd[kRanges + 1] = {0.f, 1024.f, 4096.f, 16384.f, 131072.f};

// [row][range][2]: E, kappa (at the row's length), instance; the first one's fourth word: how many there are, 3 for more
// than two and 0 where some value is not finite
__device__ inline size_t lines_at(int64_t row, int range) { return ((size_t)row * kRanges + range) * 2; }

template <int kChunks>
__global__ __launch_bounds__(kBlock) void k_lines(SelectArgs a)
{
    if (blockIdx.x == 0 && threadIdx.x < kRestParts) a.rest_cnt[threadIdx.x * kRestStride] = 0;      // (for the kernel behind)
    const int lane = lane_id();
    const int i = __builtin_amdgcn_readfirstlane(blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave);
    const int row = i / kRanges, range = i % kRanges;
    if (row >= a.totals[1]) return;
    const float inf = __builtin_inff(), lo = kRangeEnd[range], hi = kRangeEnd[range + 1];
    const float Lf = (float)a.row_len[row];
    const float* __restrict__ runs = a.grp_min + runs_at<false>(row, a.run_pad);
    const float* __restrict__ E = a.memo + memo_at(row, 0, a.n_run);

    float e[kChunks], kappa[kChunks];       // least E of a run, its least kappa (no run: infinite)
    const auto read = [&](int r0) {
        float4 k[kChunks];
#pragma unroll
        for (int j = 0; j < kChunks; ++j) {
            const int r = min(r0 + j * kWave + lane, a.n_run - 1);
            e[j] = runs[r];
            k[j] = a.run_k[r];
        }
#pragma unroll
        for (int j = 0; j < kChunks; ++j) {
            kappa[j] = kappa_of(make_float2(k[j].x, k[j].y), Lf);
            if (r0 + j * kWave + lane >= a.n_run) e[j] = inf;
        }
    };
    // the run with the least bound at either end
    uint32_t least_lo = ~0u, least_hi = ~0u;
    int run_lo = 0, run_hi = 0;
    for (int r0 = 0; r0 < a.n_run; r0 += kChunks * kWave) {
        read(r0);
#pragma unroll
        for (int j = 0; j < kChunks; ++j) {
            const uint32_t l = ordered_bits(fmaf(lo, kappa[j], e[j])), h = ordered_bits(fmaf(hi, kappa[j], e[j]));
            if (l < least_lo) { least_lo = l; run_lo = r0 + j * kWave + lane; }
            if (h < least_hi) { least_hi = h; run_hi = r0 + j * kWave + lane; }
        }
    }
    const auto run_of_least = [&](uint32_t v, int run) {
        const uint32_t least = min_over<false>(v);
        return __builtin_amdgcn_readlane(run, __ffsll((long long)__ballot(v == least)) - 1);
    };
    run_lo = min(run_of_least(least_lo, run_lo), a.n_run - 1);
    run_hi = min(run_of_least(least_hi, run_hi), a.n_run - 1);

    // a, b: lanes 0 .. 15 look at the one run, lanes 16 .. 31 at the other
    float Ea, Eb, ka, kb, Ta_lo, Tb_hi;
    {
        const int run = lane & kGroup ? run_hi : run_lo, p = run * kMemoP + lane % kGroup;
        const float Ep = E[(size_t)run * kTile + lane % kGroup], kp = kappa_of(a.posK[p], Lf);
        const float T = fmaf(lane & kGroup ? hi : lo, kp, Ep);
        const uint32_t v = a.order[p] >= 0 && T < inf ? ordered_bits(T) : ~0u;      // (also not a NaN)
        const unsigned long long best = __ballot(v == min_over<true>(v));
        const int la = __ffsll((long long)best) - 1, lb = __ffsll((long long)(best & 0xFFFF0000ull)) - 1;
        const auto at = [&](float x, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l)); };
        Ea = at(Ep, la); ka = at(kp, la); Ta_lo = at(T, la);
        Eb = at(Ep, lb); kb = at(kp, lb); Tb_hi = at(T, lb);
    }
    const float cross = (Eb - Ea) / (ka - kb), c = cross > lo && cross < hi ? cross : hi;
    const float Ta = fmaf(c, ka, Ea), Tb = fmaf(c, kb, Eb);
    const float margin = 0x1p-20f * fmaxf(fmaxf(fabsf(Ta_lo), fabsf(Tb_hi)), fmaxf(fabsf(Ta), fabsf(Tb)));
    const float at_lo = Ta_lo + margin, at_c = fmaxf(Ta, Tb) + margin, at_hi = Tb_hi + margin;
    const bool fine = fabsf(Ta_lo) < inf && fabsf(Tb_hi) < inf && fabsf(Ta) < inf && fabsf(Tb) < inf;
    const auto counts = [&](float Ev, float kv) {
        return fmaf(lo, kv, Ev) <= at_lo || fmaf(c, kv, Ev) <= at_c || fmaf(hi, kv, Ev) <= at_hi;
    };

    float4 found[2] = {make_float4(0.f, 0.f, 0.f, 0.f), make_float4(0.f, 0.f, 0.f, 0.f)};
    int n = 0;
    for (int r0 = 0; fine && n <= 2 && r0 < a.n_run; r0 += kChunks * kWave) {      // (more than two are not told apart)
        if (a.n_run > kChunks * kWave) read(r0);
#pragma unroll
        for (int j = 0; j < kChunks; ++j) {
            unsigned long long open = __ballot(counts(e[j], kappa[j]));
            while (open && n <= 2) {
                int run = -1;       // four at a time, 16 lanes each
#pragma unroll
                for (int t = 0; t < kWave / kGroup; ++t) {
                    if (lane / kGroup == t && open) run = r0 + j * kWave + __ffsll((long long)open) - 1;
                    open &= open - 1;
                }
                const int p = max(run, 0) * kMemoP + lane % kGroup, g = a.order[p];
                const float Ep = E[(size_t)max(run, 0) * kTile + lane % kGroup], kp = kappa_of(a.posK[p], Lf);
                for (unsigned long long take = __ballot(run >= 0 && g >= 0 && counts(Ep, kp)); take && n <= 2; take &= take - 1, ++n) {
                    const int l = __ffsll((long long)take) - 1;
                    const float4 line = make_float4(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(Ep), l)),
                                                    __int_as_float(__builtin_amdgcn_readlane(__float_as_int(kp), l)),
                                                    __int_as_float(__builtin_amdgcn_readlane(g, l)), 0.f);
                    if (n == 0) found[0] = line;
                    else if (n == 1) found[1] = line;
                }
            }
        }
    }
    if (lane != 0) return;
    found[0].w = __int_as_float(min(n, 3));
    a.lines[lines_at(row, range)] = found[0];
    a.lines[lines_at(row, range) + 1] = found[1];
}

// The least latency of a request over the classes (infinite or not a number: none), by four lanes, and what is known of it: in the
// upper bits how many classes have it, then as in low_and_gap.
//
// Each of the four lanes reads 16 bytes of what is known of a length.  A lane that reads all of its own request's takes a cache
// line for every 16 bytes, and the address units take one line at a time: with the row of a length, its classes and the next larger E, one
// after the other, 256 lines a wave, now 64 (scan of 4 096 x 512 with 6 classes 106.4 us, 104.7; its refresh and 262 144
// requests 71.1, 69.4).
template <int kLoads>
struct ClassesOf {
    const SelectArgs& a;
    const int sub, pieces;
    float2 dg[kLoads][2];      // of this lane's classes (no such class: not a number, and so is every latency)

    __device__ __forceinline__ explicit ClassesOf(const SelectArgs& args)
        : a(args), sub(threadIdx.x % kLanes), pieces(1 << (args.class_shift - 1))
    {
#pragma unroll
        for (int l = 0; l < kLoads; ++l)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int c = 2 * (sub + l * kLanes) + h;
                dg[l][h] = a.clsK[min(c, a.n_class - 1)];
                if (c >= a.n_class) dg[l][h].x = __builtin_nanf("");
            }
    }

    __device__ __forceinline__ void read(int L, uint4 (&e)[kLoads]) const
    {
        const uint4* __restrict__ table = reinterpret_cast<const uint4*>(a.class_least) + ((uint32_t)L << (a.class_shift - 1));
#pragma unroll
        for (int l = 0; l < kLoads; ++l) e[l] = table[(sub + l * kLanes) & (pieces - 1)];
    }

    __device__ __forceinline__ void least(float c0, float Lf, const uint4 (&e)[kLoads], float& best, uint32_t& what) const
    {
        const float inf = __builtin_inff();
        float T = inf;
        uint32_t w = 0;
        const auto take = [&](float2 k, uint32_t ev, uint32_t wv) {
            const float t = min_plain(fmaf(c0, kappa_of(k, Lf), __uint_as_float(ev)), inf);
            wv |= 1u << kCountAt;
            w = t < T ? wv : t == T ? w | 2u << kCountAt : w;
            T = min_plain(T, t);
        };
#pragma unroll
        for (int l = 0; l < kLoads; ++l) { take(dg[l][0], e[l].x, e[l].y); take(dg[l][1], e[l].z, e[l].w); }
        best = min_plain(T, quad_move<0xB1>(T));
        best = min_plain(best, quad_move<0x4E>(best));
        w = T == best ? w : 0u;
        w += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0xB1, 0xf, 0xf, true);
        what = w + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0x4E, 0xf, 0xf, true);
    }
};

// Four lanes per request over the classes first; what that does not decide (a deadline that somebody
// meets, the least latency on the excluded instance, a tie that rounding may have made) is
// collected in LDS and taken by groups of lanes as above.  A workgroup takes its requests from all
// over the batch, kGroup consecutive ones at a time: the requests of one instance are neighbours,
// and those of the instance that most requests would pick all need the second half.
//
// kRequests of a workgroup: one of every lane, whose four lanes take their requests one after the other, or of four lanes.
template <bool kMigrate, int kRequests, int kLoads>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_select_by_class(SelectArgs a)
{
    static_assert(kRequests == kBlock || kRequests * kLanes == kBlock);
    constexpr bool kEach = kRequests == kBlock;
    struct Left { Request q; int index; };      // (kept: reading a request again is two more trips to memory)
    __shared__ Left todo[kRequests];
    __shared__ int n_todo;
    const int tid = threadIdx.x;
    if (tid == 0) n_todo = 0;
    __syncthreads();
    const auto index = [&](int r) { return ((int64_t)(r / kGroup) * a.segments + blockIdx.x) * kGroup + r % kGroup; };
    {
        const ClassesOf<kLoads> classes(a);
        const int r = kEach ? tid : tid / kLanes;
        const int64_t i = index(r);
        const Request q = fetch<kMigrate>(a.s, min(i, a.s.n - 1), a.max_len);
        float best;
        uint32_t what;
        if constexpr (kEach) {
            const auto of = [&](auto k, uint32_t x) {      // (quad_perm [k,k,k,k])
                return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, decltype(k)::value * 0x55, 0xf, 0xf, true);
            };
            using std::integral_constant;
            const auto each = [&](auto f) {
                f(integral_constant<int, 0>{}); f(integral_constant<int, 1>{}); f(integral_constant<int, 2>{}); f(integral_constant<int, 3>{});
            };
            uint4 e[kLanes][kLoads];
            each([&](auto k) { classes.read((int)of(k, (uint32_t)q.L), e[k]); });
            const uint32_t c0 = __float_as_uint((float)q.c0), Lf = __float_as_uint((float)q.L);
            each([&](auto k) {
                float b;
                uint32_t w;
                classes.least(__uint_as_float(of(k, c0)), __uint_as_float(of(k, Lf)), e[k], b, w);
                best = k == 0 || classes.sub == k ? b : best;
                what = k == 0 || classes.sub == k ? w : what;
            });
        } else {
            uint4 e[kLoads];
            classes.read(q.L, e);
            classes.least((float)q.c0, (float)q.L, e, best, what);
        }
        const float D = q.D, Dc = D > FLT_MAX ? FLT_MAX : D;
        const int g = (int)(what & ((1u << kLowBits) - 1u));
        // the next larger E of the class gives a larger T: by four units in the last place of T at least
        const int gap = (int)(what >> kLowBits & 0xFFu), size = (int)(__float_as_uint(best) >> 23 & 0xFFu);
        const bool alone = what >> kCountAt == 1u && gap > 0 && gap >= size - 21;
        const bool decided = alone && fabsf(best) < __builtin_inff() && g != q.ex && !(best <= Dc);
        const bool in = i < a.s.n && (kEach || classes.sub == 0), later = in && q.scored && !decided;
        if (in && !later) {
            if (q.scored) answer<kMigrate>(a, i, g, D - best, false);
            else answer<kMigrate>(a, i, -1, 0.f, false);
        }
        const unsigned long long m = __ballot(later);
        if (m) {
            int at = 0;
            if (lane_id() == 0) at = atomicAdd(&n_todo, __popcll(m));
            at = __builtin_amdgcn_readfirstlane(at);
            if (later) todo[at + __popcll(m & ((1ull << lane_id()) - 1ull))] = Left{q, r};
        }
    }
    __syncthreads();
    const int n = n_todo;
    for (int k = tid / kGroup; k < n; k += kBlock / kGroup) {
        const Left& t = todo[k];
        select_by_class<kMigrate, kMigrate>(a, index(t.index), t.q, tid % kGroup);
    }
}

// Alg. 1 for a request from the lines that can be least at its length and prompt (k_lines).  Not decided: a deadline that
// somebody meets, the least latency on the excluded instance, more than two lines.
struct LineChoice {
    float T;
    int g;
    bool decided;
};

// Where the lines of a request are.
__device__ __forceinline__ const float4* lines_of(const SelectArgs& a, const Request& q, int row)
{
    int range = 0;
#pragma unroll
    for (int k = 1; k < kRanges; ++k) range += q.c0 >= (int)kRangeEnd[k];
    return a.lines + lines_at(row, range);
}

__device__ __forceinline__ LineChoice choose_line(const Request& q, const float4& one, const float4& two)
{
    const int n = __float_as_int(one.w), g2 = __float_as_int(two.z);
    const float c0 = (float)q.c0, D = q.D, T2 = fmaf(c0, two.y, two.x);
    LineChoice r;
    r.T = fmaf(c0, one.y, one.x);
    r.g = __float_as_int(one.z);
    if (n == 2 && (T2 < r.T || (T2 == r.T && g2 < r.g))) { r.T = T2; r.g = g2; }
    r.decided = (n == 1 || n == 2) && q.c0 >= 0 && q.c0 <= (int)kRangeEnd[kRanges] && r.T < __builtin_inff() && r.g != q.ex &&
                !(r.T <= (D > FLT_MAX ? FLT_MAX : D));
    return r;
}

// What the lines leave open, by a group of lanes: mostly requests that can be served in time, so the least
// latency is not looked for along the way.
template <bool kMigrate>
__device__ __forceinline__ void select_rest(const SelectArgs& a, int64_t i, const Request& q, Selection<4>& sel)
{
    sel.template scan<true, false, true>(0, a.n_run);
    if (sel.feasG < 0) {
        sel.template scan<false, true, false>(0, a.n_run);
        sel.settle(0, a.n_run);
    }
    sel.template report<kMigrate>(i, q.D);
}

// A group of lanes per request, its lines first.
template <bool kMigrate>
__global__ __launch_bounds__(kBlock) void k_select_lines(SelectArgs a)
{
    const int sub = threadIdx.x % kGroup;
    const int64_t i = a.first + (int64_t)blockIdx.x * (kBlock / kGroup) + threadIdx.x / kGroup;
    if (i >= a.s.n) return;
    const Request q = fetch<kMigrate>(a.s, i, a.max_len);
    if (!q.scored) {
        if (sub == 0) answer<kMigrate>(a, i, -1, 0.f, false);      // not flagged: no migration target
        return;
    }
    const int row = a.len_row[q.L];
    const float4* at = lines_of(a, q, row);
    const LineChoice c = choose_line(q, at[0], at[1]);
    if (c.decided) {
        if (sub == 0) answer<kMigrate>(a, i, c.g, q.D - c.T, false);
        return;
    }
    Selection<4> sel(a, q, row, sub);
    select_rest<kMigrate>(a, i, q, sel);
}

constexpr int kRestBlocks = 24;      // workgroups per list: six on every compute unit, so that all are there at once

// First entry of list `part` where workgroup b of `blocks` appends at most `per` requests to list b % kRestParts.
__device__ inline int64_t rest_begin(int part, int blocks, int per)
{
    return (int64_t)per * ((blocks / kRestParts) * part + min(part, blocks % kRestParts));
}

// A risk scan, of which any share of the requests may be late, first half: a lane per request and its lines.
// What those leave open goes on a list for the second half; kRestParts lists, so that the workgroups do not
// wait for each other at one counter.
template <int kItems>
__global__ __launch_bounds__(kBlock) void k_late_lines(SelectArgs a)
{
    __shared__ int todo[kBlock * kItems];
    __shared__ int n_todo, at_todo;
    const int tid = threadIdx.x, part = blockIdx.x % kRestParts;
    if (tid == 0) n_todo = 0;
    __syncthreads();
    Request q[kItems];
    int row[kItems];
    float4 one[kItems], two[kItems];
    const int64_t i0 = (int64_t)blockIdx.x * (kBlock * kItems) + tid;
#pragma unroll
    for (int it = 0; it < kItems; ++it) q[it] = fetch<true>(a.s, min(i0 + it * kBlock, a.s.n - 1), a.max_len);
#pragma unroll
    for (int it = 0; it < kItems; ++it) row[it] = a.len_row[q[it].L];
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
        const float4* __restrict__ at = lines_of(a, q[it], row[it]);
        one[it] = at[0];
        two[it] = at[1];
    }
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
        const int64_t i = i0 + it * kBlock;
        const LineChoice c = choose_line(q[it], one[it], two[it]);
        const bool in = i < a.s.n, later = in && q[it].scored && !c.decided;
        if (in && !later) answer<true>(a, i, q[it].scored ? c.g : -1, q[it].scored ? q[it].D - c.T : 0.f, false);
        const unsigned long long m = __ballot(later);
        if (!m) continue;
        int at = 0;
        if (lane_id() == 0) at = atomicAdd(&n_todo, __popcll(m));
        at = __builtin_amdgcn_readfirstlane(at);
        if (later) todo[at + __popcll(m & ((1ull << lane_id()) - 1ull))] = (int)i;
    }
    __syncthreads();
    if (tid == 0 && n_todo) at_todo = atomicAdd(&a.rest_cnt[part * kRestStride], n_todo);
    __syncthreads();
    int* __restrict__ list = a.rest + rest_begin(part, a.segments, kBlock * kItems);
    for (int k = tid; k < n_todo; k += kBlock) list[at_todo + k] = todo[k];
}

// Second half: a group of lanes per listed request.  What it takes is the chain of reads of a request, so
// what all requests need of the runs is in LDS, and the next requests are on their way: per request its runs
// are waited for, and the runs looked at (147 000 requests of 1.6 M on 4 096 instances 60 us between events; without either 71).
__global__ __launch_bounds__(kBlock, 6) void k_late_rest(SelectArgs a, int wg_requests)
{
    __shared__ float4 lds_k[kRestRuns];
    __shared__ int lds_at[kRestRuns];
    for (int r = threadIdx.x; r < a.n_run; r += kBlock) { lds_k[r] = a.run_k[r]; lds_at[r] = a.run_at[r]; }
    __syncthreads();
    const int sub = threadIdx.x % kGroup, part = blockIdx.x % kRestParts;
    const int n = a.rest_cnt[part * kRestStride];
    const int* __restrict__ list = a.rest + rest_begin(part, a.segments, wg_requests);
    constexpr int kStep = kRestBlocks * (kBlock / kGroup);
    int k = blockIdx.x / kRestParts * (kBlock / kGroup) + threadIdx.x / kGroup;
    if (k >= n) return;
    // the request at hand and its row; the next one; the one after that by its index
    const auto index = [&](int k) { return list[min(k, n - 1)]; };
    int i = index(k), i1 = index(k + kStep), i2 = index(k + 2 * kStep);
    Request q = fetch<true>(a.s, i, a.max_len), q1 = fetch<true>(a.s, i1, a.max_len);
    int row = a.len_row[q.L];
    for (; k < n; k += kStep) {
        const int i3 = index(k + 3 * kStep), row1 = a.len_row[q1.L];
        const Request q2 = fetch<true>(a.s, i2, a.max_len);
        Selection<4> sel(a, q, row, sub);
        sel.run_at = lds_at;
        sel.run_k = lds_k;
        select_rest<true>(a, i, q, sel);
        i = i1; i1 = i2; i2 = i3;
        q = q1; q1 = q2;
        row = row1;
    }
}

// ------------------------------------------------------------------ cached prefixes
struct HitArgs {
    const int *ctx0, *pred_len;
    const float* budget;
    const int* exclude;
    const int *hit_off, *hit_inst, *hit_len;
    const uint16_t* len_row;
    const int* pos_of;
    const float* memo;
    const float2* posK;
    const unsigned long long* posKey;
    int* out_inst;
    float* out_slack;
    uint8_t* out_fallback;
    float* out_T;
    int64_t n, n_hits;
    int n_inst, n_run, max_len;
};

// Eq. 2's hit prefix H_{r,g}, after the pass without it: a cached prefix of h
// tokens on instance g takes delta_g * h off T(r,g) and changes nothing else,
// so Alg. 1's answer can only move to an instance the request has a prefix on.
// kLanes threads per request that has any: the choice made without prefixes
// against the request's own short list.  Feasible set: the earlier position in
// capability order wins; otherwise the smallest T, ties to the lowest index
// (the minimum over all instances is either the old one or among the hits,
// because a hit only lowers its own pair).
//
// What bounds it is the chain of dependent reads: offsets, hit, position, value.  Every lane reads the
// choice as it stands along with its own hit, so the two chains run side by side, and the hits of a
// request run side by side too.  Status build and routing of 32 768 requests with two hits on average,
// 1 024 instances: 69.0 us with a thread per request that takes the choice and its hits one after the other, 64.4 this way.
// With out_T one thread takes a request: an instance named twice is written twice.
constexpr int kHitLanes = 4;

template <int kLanes>
__global__ __launch_bounds__(kBlock) void k_hits(HitArgs a)
{
    const int64_t r = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / kLanes;
    if (r >= a.n) return;
    const int64_t h0 = min(max((int64_t)a.hit_off[r], (int64_t)0), a.n_hits);
    const int64_t h1 = min(max((int64_t)a.hit_off[r + 1], h0), a.n_hits);
    const int g0 = a.out_inst[r];
    const int L = min(max(a.pred_len[r], 0), a.max_len);
    const int ci = a.ctx0[r];
    const float c0 = (float)ci, Lf = (float)L, D = a.budget[r];
    const float Dc = D > FLT_MAX ? FLT_MAX : D;
    const int ex = a.exclude ? a.exclude[r] : -1;
    if (h0 >= h1) return;
    int64_t k = h0 + threadIdx.x % kLanes;
    const auto hit = [&](int64_t at, int& g, int& h) {
        const int64_t i = min(at, h1 - 1);
        g = a.hit_inst[i];
        h = min(max(a.hit_len[i], 0), max(ci, 0));
    };
    const auto place = [&](int g) { return a.pos_of[min(max(g, 0), a.n_inst - 1)]; };
    const float* __restrict__ rowE = a.memo + memo_at(row_at(a.len_row, L), 0, a.n_run);
    struct Pair { float2 K; unsigned long long key; float E; };
    const auto pair_at = [&](int p) {
        return Pair{a.posK[p], a.posKey[p], rowE[(size_t)(p / kMemoP) * kTile + p % kMemoP]};
    };

    int g, h;
    hit(k, g, h);
    const int p0 = place(g0);
    int p = place(g);
    const Pair b = pair_at(p0);
    Pair v = pair_at(p);

    unsigned long long feasKey = ~0ull;
    int feasG = -1, anyG = -1;
    float feasT = 0.f, anyT = __builtin_inff();
    if (g0 >= 0) {
        const float T0 = fmaf(c0, kappa_of(b.K, Lf), b.E);
        if (T0 <= Dc) { feasKey = b.key; feasG = g0; feasT = T0; }
        anyG = g0; anyT = T0;
    }
    while (k < h1) {
        const float T = fmaf(-(float)h, v.K.x, fmaf(c0, kappa_of(v.K, Lf), v.E));
        const bool there = g >= 0 && g < a.n_inst;
        if constexpr (kLanes == 1) {
            if (a.out_T && there) {          // (an instance named twice: the longer prefix, i.e. the smaller T, stays)
                float* t = a.out_T + (size_t)r * a.n_inst + g;
                *t = fminf(*t, T);
            }
        }
        if (there && g != ex) {
            if (T <= Dc &&
                (feasG < 0 || v.key < feasKey || (v.key == feasKey && (g < feasG || (g == feasG && T < feasT))))) {
                feasKey = v.key; feasG = g; feasT = T;
            }
            if (T < anyT || (T == anyT && g < anyG)) { anyT = T; anyG = g; }
        }
        k += kLanes;
        if (k < h1) {
            hit(k, g, h);
            v = pair_at(place(g));
        }
    }
    // the lanes started from the same choice: the least of them in the same order
#pragma unroll
    for (int d = 1; d < kLanes; d *= 2) {
        const unsigned long long key = __shfl_xor(feasKey, d);
        const int fg = __shfl_xor(feasG, d), ag = __shfl_xor(anyG, d);
        const float fT = __shfl_xor(feasT, d), aT = __shfl_xor(anyT, d);
        if (fg >= 0 && (feasG < 0 || key < feasKey || (key == feasKey && (fg < feasG || (fg == feasG && fT < feasT))))) {
            feasKey = key; feasG = fg; feasT = fT;
        }
        if (aT < anyT || (aT == anyT && ag < anyG)) { anyT = aT; anyG = ag; }
    }
    if (threadIdx.x % kLanes) return;
    const bool found = feasG >= 0;
    const int best = found ? feasG : anyG;
    a.out_inst[r] = best;
    a.out_slack[r] = best >= 0 ? D - (found ? feasT : anyT) : 0.f;
    if (a.out_fallback) a.out_fallback[r] = !found;
}

// ------------------------------------------------------------------ small batches, pair by pair
struct DirectArgs {
    ReqSrc s;
    const float4* instK;
    const double* hD;
    const uint16_t *tabR, *tabS;
    const float2* tabGH;
    DirectPart* parts_out;   // [n][parts]
    int* out_inst;
    float* out_slack;
    uint8_t* out_fallback;
    float* out_T;
    int n, n_inst, max_len, parts;
    int finite;              // 1: an infinite latency (or a NaN) is none, as in the pass over the table
    CountArgs count;         // a risk scan: by an extra workgroup
};

// The best of the lanes' selections, word by word: a minimum and, among the lanes that hold it, the
// least of the next word (a minimum through DPP is one instruction per step; comparing whole
// selections pairwise takes twenty).
template <bool kRow>
__device__ inline DirectPart best_over(const DirectPart& b)
{
    DirectPart r = no_selection();
    r.any_T = min_over<kRow>(b.any_T);
    r.any_g = min_over<kRow>(b.any_T == r.any_T ? b.any_g : ~0u);
    if (__ballot(b.g != ~0u)) {
        r.d_hi = min_over<kRow>(b.d_hi);
        bool in = b.d_hi == r.d_hi;
        r.d_lo = min_over<kRow>(in ? b.d_lo : ~0u);
        in = in && b.d_lo == r.d_lo;
        r.g = min_over<kRow>(in ? b.g : ~0u);
        r.T = min_over<kRow>(in && b.g == r.g ? b.T : ~0u);
    }
    return r;
}

__device__ inline void direct_answer(const DirectArgs& a, int r, float D, const DirectPart& b)
{
    const bool found = b.g != ~0u;
    const uint32_t fg = b.g, ag = b.any_g, fT = b.T, aT = b.any_T;
    const int g = (int)(found ? fg : ag);          // (-1: nobody is allowed)
    const float T = from_ordered_bits(found ? fT : aT);
    a.out_inst[r] = g;
    a.out_slack[r] = g >= 0 ? D - T : 0.f;
    if (a.out_fallback) a.out_fallback[r] = !found;
}

// A batch of a few requests (one arriving request is the paper's own case): grouping by length and
// a table of per-length values would cost more than they save, so kLanes lanes take a request, each
// an instance (or a few), and form T = E + c0 * kappa with E from the instance's own tables (the
// same expression as in k_memo).
//
// What bounds it is the chain of dependent reads, so the segment #{R_i <= L} is found in two steps
// instead of a binary search's ten: the splitters (every stride-th sorted length, a table of their
// own, 16 or 32 bytes), then the one stride they leave, read whole.  Alg. 1's argmax d_g is taken
// from d_g itself (the selections carry it), so no capability order is needed; the selections of
// the lanes are combined in registers and, between the waves of a request, through LDS, so there is
// no second launch and no workspace.  Fleets of more than kDirectSpan instances take several
// workgroups per request, combined by k_direct_merge.
//
// The flagged requests of a small risk scan are taken the same way (kMigrate; a workgroup of its own
// finishes what the table pass would have).
//
// A lane that reads all of its instance's words itself touches a cache line of its own with every read, 64 a wave, and the
// few compute units that a small batch takes wait for their first-level caches.  So the words of an instance are read by as
// many lanes side by side (up to four; of eight words two each), which take each other's instances in turn and add up
// what they count: 16 lines a read.  Where a build has left every segment of an instance alike (blend weight 1) there is no
// search at all.  Whole calls, us, before / now: 48 requests on 1 024 instances x 1 000 8.9 / 6.4, weight 1 9.0 / 4.6; 500 20 / 14.5;
// 100 on 4 096 x 512 29 / 18.8; 4 096 on 64 x 1 000 7.3 / 5.5; scan of 32 x 512 with its build 14.6 / 13.2.

// The pieces of the lanes' own kW words at `at` (in words of 16 bytes): piece lane % kW of every lane of the group in turn.
template <int kW>
__device__ __forceinline__ void read_pieces(const uint4* __restrict__ tab, uint32_t at, uint4 (&w)[kW])
{
    const uint32_t piece = lane_id() % (kW < 4 ? kW : 4);
    const auto of = [&](auto ctrl) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)at, decltype(ctrl)::value, 0xf, 0xf, true); };
    using std::integral_constant;
    if constexpr (kW == 1) {
        w[0] = tab[at];
    } else if constexpr (kW == 2) {
        w[0] = tab[of(integral_constant<int, 0xA0>{}) + piece];      // quad_perm [0,0,2,2], [1,1,3,3]
        w[1] = tab[of(integral_constant<int, 0xF5>{}) + piece];
    } else {
        const uint32_t o[4] = {of(integral_constant<int, 0x00>{}), of(integral_constant<int, 0x55>{}),
                               of(integral_constant<int, 0xAA>{}), of(integral_constant<int, 0xFF>{})};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
#pragma unroll
            for (int i = 0; i < kW / 4; ++i) w[j * (kW / 4) + i] = tab[o[j] + 4 * i + piece];
        }
    }
}

// How many of a lane's own lengths are at most L (the same for all lanes of a group).
template <int kW>
__device__ __forceinline__ int count_pieces(const uint4 (&w)[kW], uint32_t L)
{
    constexpr int kG = kW < 4 ? kW : 4;
    const int piece = lane_id() % kG;
    uint32_t own = 0;
#pragma unroll
    for (int j = 0; j < kG; ++j) {
        uint32_t c = 0;
#pragma unroll
        for (int i = 0; i < kW / kG; ++i) c += count_upto2(w[j * (kW / kG) + i], L);
        if constexpr (kG >= 2) c += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c, 0xB1, 0xf, 0xf, true);
        if constexpr (kG >= 4) c += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c, 0x4E, 0xf, 0xf, true);
        own = kG == 1 || piece == j ? c : own;
    }
    return both_counts(own);
}

// kU: instances of a lane in flight together; kS, kB: words of 16 bytes of the splitters, of a stride
template <bool kMigrate, int kLanes, int kU, int kS, int kB>
__global__ __launch_bounds__(kLanes <= 64 ? kBlock : kLanes) void k_direct(DirectArgs a)
{
    fetch_args<DirectArgs>();
    constexpr int kThreads = kLanes <= 64 ? kBlock : kLanes;
    __shared__ int sums[kThreads / kWave];
    if (kMigrate && blockIdx.x == gridDim.x - 1) return count_flagged(a.count, kThreads, sums);
    constexpr int kPerGroup = kThreads / kLanes;              // requests per workgroup
    const int sub = threadIdx.x % kLanes;
    int r, part = 0;
    if (kPerGroup > 1) {
        r = blockIdx.x * kPerGroup + threadIdx.x / kLanes;
    } else {
        r = blockIdx.x / a.parts;
        part = blockIdx.x % a.parts;
    }
    const bool live = r < a.n;
    const int rc = min(r, a.n - 1);
    const Request q = fetch<kMigrate>(a.s, rc, a.max_len);
    const int L = q.L, ex = q.ex;
    const float c0 = (float)q.c0, Lf = (float)L, D = q.D;
    const float Dc = D > FLT_MAX ? FLT_MAX : D;
    if (kMigrate && !__ballot(q.scored)) {      // not flagged: no migration target (a request is a workgroup's, or all of a wave's are alike)
        if (sub == 0 && live) { a.out_inst[r] = -1; a.out_slack[r] = 0.f; }
        return;
    }
    const float tri = Lf * (Lf - 1.0f) * 0.5f;
    constexpr int kSplits = 8 * kS, kStride = 8 * kB, kCap = kSplits * kStride;
    const uint4* __restrict__ S = reinterpret_cast<const uint4*>(a.tabS);
    const uint4* __restrict__ R = reinterpret_cast<const uint4*>(a.tabR);
    const int g_begin = part * kDirectSpan, g_end = a.parts > 1 ? min(g_begin + kDirectSpan, a.n_inst) : a.n_inst;

    DirectPart best = no_selection();
    const int wave_sub = kLanes > kWave ? sub & ~(kWave - 1) : 0;      // (all lanes of a wave go through the loop together)
    for (int g0 = g_begin + wave_sub; g0 < g_end; g0 += kLanes * kU) {
        int g[kU], k[kU];
        uint4 w[kU][kB > kS ? kB : kS];
        float4 K[kU];
        float2 gh[kU];
        double d[kU];
        bool search = false;
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            g[u] = min(g0 + sub - wave_sub + u * kLanes, g_end - 1);           // (a repeat of the last one changes nothing)
            K[u] = a.instK[g[u]];
            read_pieces<kS>(S, (uint32_t)g[u] * kS, reinterpret_cast<uint4 (&)[kS]>(w[u]));
            d[u] = a.hD[g[u]];
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            search = search || !all_alike(K[u]);
            k[u] = 0;
        }
        if (__any(search)) {      // (otherwise every segment is the first one)
#pragma unroll
            for (int u = 0; u < kU; ++u)      // (all of a full table: counted below)
                k[u] = min(count_pieces<kS>(reinterpret_cast<uint4 (&)[kS]>(w[u]), (uint32_t)L), kSplits - 1) * kStride;
#pragma unroll
            for (int u = 0; u < kU; ++u)
                read_pieces<kB>(R, (uint32_t)g[u] * (kCap / 8) + (uint32_t)k[u] / 8, reinterpret_cast<uint4 (&)[kB]>(w[u]));
#pragma unroll
            for (int u = 0; u < kU; ++u) k[u] += count_pieces<kB>(reinterpret_cast<uint4 (&)[kB]>(w[u]), (uint32_t)L);
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            gh[u] = a.tabGH[gh_at(g[u], k[u], kCap)];
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const float E = fmaf(tri, K[u].z * (float)(entries_of(K[u]) - k[u] + 1), fmaf(Lf, gh[u].y, gh[u].x));
            const float T = fmaf(c0, kappa_of(make_float2(K[u].x, K[u].y), Lf), E);
            if (a.out_T && live) a.out_T[(size_t)r * a.n_inst + g[u]] = T;
            if (g[u] != ex && (!a.finite || T < __builtin_inff())) {
                const unsigned long long db = falling_bits(d[u]);
                const uint32_t tb = ordered_bits(T);
                DirectPart one{tb, (uint32_t)g[u], ~0u, ~0u, ~0u, ~0u};
                if (T <= Dc) { one.d_hi = (uint32_t)(db >> 32); one.d_lo = (uint32_t)db; one.g = (uint32_t)g[u]; one.T = tb; }
                take_better(best, one);
            }
        }
    }

    if constexpr (kLanes <= 64) {
        best = best_over<kLanes == 16>(best);
        if (sub == 0 && live) direct_answer(a, r, D, q.scored ? best : no_selection());
    } else {
        constexpr int kN = kLanes / kWave;
        static_assert(kN <= 16, "one row of lanes takes the waves' selections");
        __shared__ DirectPart waves[kN];
        best = best_over<false>(best);
        if (lane_id() == 0) waves[threadIdx.x / kWave] = best;
        __syncthreads();
        if (threadIdx.x < 16) {
            best = no_selection();
            if (threadIdx.x < kN) best = waves[threadIdx.x];
            best = best_over<true>(best);
            if (threadIdx.x == 0) {
                if (a.parts == 1) direct_answer(a, r, D, best);
                else a.parts_out[(size_t)r * a.parts + part] = best;
            }
        }
    }
}

// The parts of each request of a wide fleet, a wave per request.
__global__ __launch_bounds__(kBlock) void k_direct_merge(DirectArgs a)
{
    const int r = blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    if (r >= a.n) return;
    DirectPart best = no_selection();
    for (int i = lane_id(); i < a.parts; i += kWave) take_better(best, a.parts_out[(size_t)r * a.parts + i]);
    best = best_over<false>(best);
    if (lane_id() == 0) direct_answer(a, r, a.s.budget[r], best);
}

// ------------------------------------------------------------------ every pair's latency (out_T)
// The table keeps the values of a run together, in class order, a request wants every instance in index order.  So
// `rows` lengths at a time the table is first turned into rows over the instances (k_rows, as much as the
// lengths, not the requests), and the latencies are then a stream over those (k_pairs).
struct PairsArgs {
    const int *ctx0, *pred_len, *totals;
    const float* budget;
    const int* exclude;
    const double* hD;
    int* out_inst;
    float* out_slack;
    uint8_t* out_fallback;
    const uint16_t* len_row;
    const int *order, *pos_of;
    const float* memo;
    const float4* instK;
    float* turned;     // [rows][n_inst]
    float* out_T;
    int64_t n, first;  // requests; the launch's first one
    int row0, rows;    // the part of the table at hand
    int n_inst, m_pos, max_len;
};

// Requests that a group of lanes takes together (with the selections, which take six registers each: fewer).
constexpr int pairs_requests(bool select) { return select ? 4 : 8; }

__global__ __launch_bounds__(kBlock) void k_rows(PairsArgs a)
{
    const int blocks = (a.m_pos + kWave - 1) / kWave;
    const int p0 = (int)(blockIdx.x % blocks) * kWave, u0 = (int)(blockIdx.x / blocks) * kWave;   // row u0 of the part
    if (a.row0 + u0 >= a.totals[1]) return;
    const int lane = lane_id(), wave = threadIdx.x / kWave;
    constexpr int kPer = kWave / (kBlock / kWave);
    const int p = min(p0 + lane, a.m_pos - 1);
    float v[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) v[i] = a.memo[memo_at(a.row0 + u0 + wave * kPer + i, p / kMemoP, a.m_pos / kMemoP) + p % kMemoP];
    const int g = p0 + lane < a.m_pos ? a.order[p] : -1;
    if (g < 0) return;
#pragma unroll
    for (int i = 0; i < kPer; ++i) a.turned[(size_t)(u0 + wave * kPer + i) * a.n_inst + g] = v[i];
}

// The same arithmetic as the selection's, exclusions not applied.  kLanes lanes take kReq requests together (one
// request is a chain of three reads and, on a small fleet, one store), kVec instances each.
//
// kSelect: with every latency of a request in its lanes' registers, Alg. 1 is decided here as well and the
// selection over runs is not launched.  On a small fleet that took longer than the latencies
// themselves: whole call on 262 144 requests x 64 instances 59 us with it, 46 without; 100 000 x 128 without it 40 us, x 129
// with it 50 (a row of lanes per request is kept up to 128 instances: eight of them per lane).
template <int kLanes, int kVec, bool kSelect, bool kWrite>
__device__ __forceinline__ void pairs(const PairsArgs& a)
{
    constexpr int kReq = pairs_requests(kSelect);
    static_assert(!kSelect || kLanes == 16, "a request's lanes are a row of a wave");
    static_assert(kWrite || kVec == 1, "read where they are, an instance's values are on their own");
    const int sub = threadIdx.x % kLanes;
    const int64_t r0 = a.first + ((int64_t)blockIdx.x * (kBlock / kLanes) + threadIdx.x / kLanes) * kReq;
    if (r0 >= a.n) return;
    int L[kReq], row[kReq], ex[kReq];
    float c0[kReq], D[kReq];
    // the lane's selections (its instances come in ascending order, so of equal ones the first stays)
    float anyT[kReq], feasT[kReq];
    int anyG[kReq], feasG[kReq];
    unsigned long long feasKey[kReq];
#pragma unroll
    for (int j = 0; j < kReq; ++j) {
        const int64_t r = min(r0 + j, a.n - 1);
        L[j] = min(max(a.pred_len[r], 0), a.max_len);
        c0[j] = (float)a.ctx0[r];
        if (kSelect) { D[j] = a.budget[r]; ex[j] = a.exclude ? a.exclude[r] : -1; }
        anyT[j] = __builtin_inff(); feasT[j] = 0.f; anyG[j] = feasG[j] = -1; feasKey[j] = ~0ull;
    }
#pragma unroll
    for (int j = 0; j < kReq; ++j) {
        row[j] = row_at(a.len_row, L[j]) - (kWrite ? a.row0 : 0);
        if (r0 + j >= a.n || (kWrite && (unsigned)row[j] >= (unsigned)a.rows)) row[j] = -1;
    }
    struct alignas(4 * kVec) Values { float v[kVec]; };
    for (int g = sub * kVec; g < a.n_inst; g += kLanes * kVec) {
        float2 K[kVec];
        unsigned long long key[kVec];
#pragma unroll
        for (int i = 0; i < kVec; ++i) {
            const float4 k = a.instK[g + i];
            K[i] = make_float2(k.x, k.y);
            if (kSelect) key[i] = falling_bits(a.hD[g + i]);
        }
        Values E[kReq];
#pragma unroll
        for (int j = 0; j < kReq; ++j)
            E[j] = *reinterpret_cast<const Values*>(
                kWrite ? a.turned + (size_t)max(row[j], 0) * a.n_inst + g
                       : a.memo + memo_at(max(row[j], 0), a.pos_of[g] / kMemoP, a.m_pos / kMemoP) + a.pos_of[g] % kMemoP);
#pragma unroll
        for (int j = 0; j < kReq; ++j) {
            if (row[j] < 0) continue;
            const float Dc = D[j] > FLT_MAX ? FLT_MAX : D[j];
#pragma unroll
            for (int i = 0; i < kVec; ++i) {
                const float T = fmaf(c0[j], kappa_of(K[i], (float)L[j]), E[j].v[i]);
                E[j].v[i] = T;
                if (!kSelect) continue;
                const float mine = g + i == ex[j] ? __builtin_inff() : T;      // (an infinite latency is none, as in the selection over runs)
                const bool less = mine < anyT[j], better = mine <= Dc && key[i] < feasKey[j];
                anyT[j] = less ? mine : anyT[j]; anyG[j] = less ? g + i : anyG[j];
                feasKey[j] = better ? key[i] : feasKey[j]; feasG[j] = better ? g + i : feasG[j]; feasT[j] = better ? mine : feasT[j];
            }
            if (kWrite) *reinterpret_cast<Values*>(a.out_T + (size_t)(r0 + j) * a.n_inst + g) = E[j];
        }
    }
    if constexpr (kSelect) {
#pragma unroll
        for (int j = 0; j < kReq; ++j) {
            const DirectPart b = best_over<true>(DirectPart{anyG[j] >= 0 ? ordered_bits(anyT[j]) : ~0u, (uint32_t)anyG[j],
                                                            (uint32_t)(feasKey[j] >> 32), (uint32_t)feasKey[j], (uint32_t)feasG[j],
                                                            feasG[j] >= 0 ? ordered_bits(feasT[j]) : ~0u});
            if (sub != 0 || row[j] < 0) continue;
            const bool found = b.g != ~0u;
            const int g = (int)(found ? b.g : b.any_g);          // (-1: nobody is allowed)
            a.out_inst[r0 + j] = g;
            a.out_slack[r0 + j] = g >= 0 ? D[j] - from_ordered_bits(found ? b.T : b.any_T) : 0.f;
            if (a.out_fallback) a.out_fallback[r0 + j] = !found;
        }
    }
}

template <int kLanes, int kVec, bool kSelect>
__global__ __launch_bounds__(kBlock) void k_pairs(PairsArgs a)
{
    if (a.row0 >= a.totals[1]) return;
    pairs<kLanes, kVec, kSelect, true>(a);
}

// The same decision on a fleet of up to kFewInst instances, where a run holds hardly more than one or two of them and the
// selection over runs looks at one after the other: every latency of a request from the table as it is.
// 193 397 requests, selection over runs / this, us a call: 12 instances with a blend 53 / 35 (every pair scored
// without the table of runs: 47), 16 without 33 / 26, 24 33 / 32, 32 34 / 34, 48 33 / 41.
__global__ __launch_bounds__(kBlock) void k_select_few(PairsArgs a) { pairs<kGroup, 1, true, false>(a); }

__global__ void k_set_int(int* p, int v) { *p = v; }

}  // namespace

static CountArgs count_args(const gr_fleet* f, const ReqSrc& src, const ScoreOut& out)
{
    return CountArgs{f->totals, out.n_selected, f->late_cnt, src.act_off, src.flag, src.n, f->n_inst * f->late_parts, f->n_inst};
}

// Alg. 1 pair by pair.
template <bool kMigrate>
static int launch_pair_by_pair(gr_fleet* f, const ReqSrc& src, const ScoreOut& out, bool finite, hipStream_t s)
{
    const int n = (int)src.n, M = f->n_inst;
    if (n == 0) return GR_OK;
    if (src.n > std::max<int64_t>(kDirectMax, kDirectLanes / kGroup)) return GR_ERR_TOO_LARGE;
    DirectArgs d{};
    d.s = src;
    d.instK = f->instK; d.hD = f->hD; d.tabR = f->tabR; d.tabS = f->tabS; d.tabGH = f->tabGH;
    d.parts_out = f->direct_part;
    d.out_inst = out.inst; d.out_slack = out.slack; d.out_fallback = out.fallback; d.out_T = out.T;
    d.n = n; d.n_inst = M; d.max_len = f->max_len; d.finite = finite;
    d.parts = kMigrate ? 1 : (M + kDirectSpan - 1) / kDirectSpan;
    if ((int64_t)n * d.parts > kDirectParts) d.parts = 1;      // (many requests fill the chip as they are)
    if (kMigrate) d.count = count_args(f, src, out);
    // lanes per request: an instance each as far as a workgroup goes (few requests: the chain of reads
    // of one instance is the time of the call); 64 lanes leave the fewest idle on small fleets, and
    // where there are requests enough, 16 with two instances each up to 32 (16 384 requests x 32 instances
    // 6.7 us, 8.9 with 64 lanes; 110 x 17 a microsecond more); with two each they do for 128 instances (6 000 requests 9.0 us,
    // with 256 lanes 10.4; four each for 256: 100 requests 4.9 us instead of 3.6)
    {
        ProfScope ps(f, kDirect, s);
#define GR_LAUNCH_DIRECT(N, U) do { \
        constexpr int per = N <= 64 ? kBlock / (N <= 64 ? N : 1) : 1;      /* requests per workgroup */ \
        const dim3 grid((per > 1 ? (n + per - 1) / per : n * d.parts) + (kMigrate ? 1 : 0)), block(per > 1 ? kBlock : N); \
        switch (f->epl) {      /* (tables of 64 .. 2 048 lengths: 8, 16 or 32 splitters, see split_count) */ \
            case 1: hipLaunchKernelGGL((k_direct<kMigrate, N, U, 1, 1>), grid, block, 0, s, d); break; \
            case 2: hipLaunchKernelGGL((k_direct<kMigrate, N, U, 2, 1>), grid, block, 0, s, d); break; \
            case 4: hipLaunchKernelGGL((k_direct<kMigrate, N, U, 2, 2>), grid, block, 0, s, d); break; \
            case 8: hipLaunchKernelGGL((k_direct<kMigrate, N, U, 2, 4>), grid, block, 0, s, d); break; \
            case 16: hipLaunchKernelGGL((k_direct<kMigrate, N, (U > 2 ? 2 : U), 4, 4>), grid, block, 0, s, d); break; \
            default: hipLaunchKernelGGL((k_direct<kMigrate, N, (U > 2 ? 2 : U), 4, 8>), grid, block, 0, s, d); break; \
        } } while (0)
        if (M <= 16) GR_LAUNCH_DIRECT(16, 1);
        else if (M <= 32 && n > kDirectMax) GR_LAUNCH_DIRECT(16, 2);
        else if (M <= 64) GR_LAUNCH_DIRECT(64, 1);
        else if (M <= 128) GR_LAUNCH_DIRECT(64, 2);
        else if (M <= 512) GR_LAUNCH_DIRECT(256, 1);
        else if (M <= 1024) GR_LAUNCH_DIRECT(1024, 1);
        else GR_LAUNCH_DIRECT(1024, 4);
#undef GR_LAUNCH_DIRECT
    }
    if (d.parts > 1) {
        ProfScope ps(f, kDirectMerge, s);
        constexpr int per = kBlock / kWave;
        hipLaunchKernelGGL(k_direct_merge, dim3((n + per - 1) / per), dim3(kBlock), 0, s, d);
    }
    return hipGetLastError() == hipSuccess ? GR_OK : GR_ERR_HIP;
}

int launch_direct(gr_fleet* f, const ReqSrc& src, const ScoreOut& out, hipStream_t s)
{
    return launch_pair_by_pair<false>(f, src, out, false, s);
}

// Whether a batch is scored pair by pair: as the caller says (gr_set_small_batch_pairs), or by the number of pairs,
// and of those that its lanes go through (see launch_pair_by_pair).  A pass over the table is two to four launches whose time hardly depends on
// the batch; this is one that grows with the pairs.  Whole calls, us, table / pairs, with the status build where it says refresh or scan:
//   routing  16 instances x 40 000 requests 11.4 / 6.4, 49 152 11.3 / 7.05;  24 x 32 768 11.0 / 7.7;  32 x 24 576 11.05 / 6.7
//            64 x 12 000 9.9 / 8.2, 16 384 10.1 / 9.9, 32 768 10.4 / 17.5;  128 x 6 000 10.2 / 9.0, 8 192 10.2 / 11.4
//            256 x 3 000 11.4 / 10.4, 4 096 11.3 / 13.0;  with out_T 64 x 12 000 15.8 / 8.5, 256 x 3 000 24.8 / 10.4
//   refresh  16 x 49 152 17.8 / 12.0;  24 x 32 768 17.4 / 12.9;  256 x 3 000 19.6 / 16.8, 4 096 19.5 / 19.6, 8 192 19.6 / 28.9
//            1 024 x 700 29.3 / 22.4, 1 024 29.3 / 26.0, 1 500 30.3 / 31.6;  4 096 x 200 42.6 / 37.8, 300 42.6 / 52
//   scan     32 x 700 requests each 19.1 / 16.2 (all of them late 18.9 / 16.3), 64 x 190 17.7 / 13.8 (17.3 / 14.1), 128 x 47 16.7 / 11.4 (16.5 / 12.2)
//            64 x 256 17.0 / 16.0, 512 17.8 / 26.7;  128 x 100 17.1 / 22;  40 x 600 18.8 / 23.9
// The line is where routing on a standing status still gains, whose table has its class order already; a refresh makes it anew and
// would gain to somewhat larger batches.
bool pair_by_pair(const gr_fleet* f, int64_t n)
{
    if (f->small_batch_pairs >= 0) return n <= kDirectMax && n * f->m_pad <= f->small_batch_pairs;
    const int pairs = std::max(f->n_inst, kGroup), lanes = pairs <= 2 * kGroup ? pairs : (pairs + kWave - 1) / kWave * kWave;
    return n * pairs <= kDirectPairs || n * lanes <= kDirectLanes;
}

// Whether an infinite latency (or a NaN) of a routing batch scored pair by pair is none, as in the pass over the table: small
// batches have always taken it for a latency.
static bool pairs_finite(const gr_fleet* f, int64_t n)
{
    const bool small = n <= kDirectMax && n * f->m_pad <= kDirectInfinite;
    return f->small_batch_pairs < 0 && !small;
}

constexpr int64_t kByClassMin = int64_t(1) << 17;      // requests from which the classes are looked at first
// and from which a workgroup takes 256 of them (64 otherwise).  Whole calls, us, 64 / 256: scan of 1 024 x 400 39.95 / 38.2,
// of 1 024 x 1 000 56.1 / 53.0 (deadlines x 16 76.5 / 69.3); refresh of 4 096 instances and 262 144 requests 64.8 / 64.9, of which a batch
// with deadlines that many meet (x 16) wants the lanes for its second half: 70.3 / 77.7, 140 000 on 2 000 52.6 / 64.3.
constexpr int64_t kByClassMany[2] = {int64_t(1) << 19, int64_t(1) << 18};      // routing, risk scan
constexpr int64_t kLinesMany = int64_t(1) << 19;      // and on fleets of few runs
constexpr int64_t kLinesScanMin = int64_t(3) << 16;     // requests of a scan from which the lines are looked at first

constexpr int64_t kLaneMin = 1 << 15;      // requests from which four lanes take one, on fleets of few runs (see k_select_lanes)

constexpr int kFewInst = 16;     // instances up to which a routing batch is decided over all of them

// A launch has fewer than 2^32 threads: kernels that take many threads per request go through larger batches
// (2^28 requests at 16 lanes each, 2^24 at a workgroup each) a part at a time.
constexpr int64_t kLaunchThreads = int64_t(1) << 31;

template <bool kMigrate>
static void launch_select(const gr_fleet* f, SelectArgs a, bool by_class, bool by_lines, bool blended, hipStream_t s)
{
    const int64_t n = a.s.n;
    if (by_class) {
        // large batches: a request per lane; else a wave's worth per workgroup, so that the second half has the
        // lanes when many requests need it
        const bool many = n >= kByClassMany[kMigrate];
        const int64_t per = many ? kBlock : kBlock / kLanes;
        a.segments = (int)((n + per - 1) / per);
#define GR_LAUNCH_BY_CLASS(N) do { \
        if (f->n_class <= 2 * kLanes) hipLaunchKernelGGL((k_select_by_class<kMigrate, N, 1>), dim3(a.segments), dim3(kBlock), 0, s, a); \
        else hipLaunchKernelGGL((k_select_by_class<kMigrate, N, 2>), dim3(a.segments), dim3(kBlock), 0, s, a); } while (0)
        if (many) GR_LAUNCH_BY_CLASS(kBlock);
        else GR_LAUNCH_BY_CLASS(kBlock / kLanes);
#undef GR_LAUNCH_BY_CLASS
        return;
    }
    if (!by_lines && f->n_run <= kLaneRuns && n >= kLaneMin) {
        for (a.first = 0; a.first < n; a.first += kLaunchThreads / kLanes) {
            const int64_t here = std::min(n - a.first, kLaunchThreads / kLanes);
            const dim3 grid((unsigned)((here * kLanes + kBlock - 1) / kBlock));
#define GR_LAUNCH_LANES(R) do { \
            if (blended) hipLaunchKernelGGL((k_select_lanes<kMigrate, R, true>), grid, dim3(kBlock), 0, s, a); \
            else hipLaunchKernelGGL((k_select_lanes<kMigrate, R, false>), grid, dim3(kBlock), 0, s, a); } while (0)
            if (f->n_run <= 16) GR_LAUNCH_LANES(16);
            else GR_LAUNCH_LANES(32);
#undef GR_LAUNCH_LANES
        }
        return;
    }
    // 16 runs per lane group and chunk: as few rounds as five chunks make, and no more chunks than fill them
    // (1 024 instances of three classes are 66 runs: two rounds of four chunks for two runs more than one)
    const int all = (f->n_run + kGroup - 1) / kGroup, rounds = (all + 4) / 5, chunks = (all + rounds - 1) / rounds;
    for (a.first = 0; a.first < n; a.first += kLaunchThreads / kGroup) {
        const int64_t here = std::min(n - a.first, kLaunchThreads / kGroup);
        const dim3 grid((unsigned)((here + kBlock / kGroup - 1) / (kBlock / kGroup)));
#define GR_LAUNCH_SELECT(C) hipLaunchKernelGGL((k_select<kMigrate, C>), grid, dim3(kBlock), 0, s, a)
        if (by_lines) hipLaunchKernelGGL(k_select_lines<kMigrate>, grid, dim3(kBlock), 0, s, a);
        else if (chunks == 1) GR_LAUNCH_SELECT(1);
        else if (chunks == 2) GR_LAUNCH_SELECT(2);
        else if (chunks == 3) GR_LAUNCH_SELECT(3);
        else if (chunks == 4) GR_LAUNCH_SELECT(4);
        else GR_LAUNCH_SELECT(5);
#undef GR_LAUNCH_SELECT
    }
}

// How the latencies of out_T are written: four instances per lane where every row begins at a multiple of 16
// bytes; few lanes per request on a small fleet, whose rows are short; and whether Alg. 1 is decided there.
struct PairsPlan {
    bool four, select;
    int lanes;

    PairsPlan(const gr_fleet* f, const float* out_T)
    {
        const int M = f->n_inst;
        four = M % 4 == 0 && M >= 64 && reinterpret_cast<uintptr_t>(out_T) % 16 == 0;
        select = M <= 128;
        lanes = select ? 16 : M <= 512 ? kWave : kBlock;
    }
};

// Whether the table of a pass has a row for every length there may be, so that the list of those that there are is not
// made, and the class order is made by the table's workgroups: two launches less (three in a routing call), two
// dependent reads less, for a table that may be larger.  Where the fleet is so small that a class's order is quickly made, and
// the table no larger than the list's launches are worth, for one request too (gr_score_route_cached takes
// the table whatever the batch).  Whole calls, us, with the list / a row per length:
//   values of the table   1.2 M (256 instances, lengths up to 4 096)   3.9 M (200, 16 384)   4.7 M (256)    7.9 M (480)
//   routing one request with its prefix       20.4 / 14.4               20.7 / 17.3          20.5 / 20.2    20.5 / 20.9
//   refresh, x 400, routing 8 192             27.4 / 20.3               27.2 / 22.4          27.0 / 25.7    28.2 / 29.1
//   risk scan x 128                           25.1 / 21.3               24.4 / 22.1          25.6 / 26.6    24.9 / 28.4
//   risk scan x 512                           28.5 / 24.7               26.7 / 24.9          27.4 / 28.9    32.8 / 36.2
// (The workgroups of 2^22 values are 1 024, and one per run: the chip takes 1 792 at once.)  On larger fleets the
// order takes a launch of its own: 777 instances, 20 011 requests, 29.2 / 29.3; 1 024 x 200, 32 768 requests 66.7 / 66.9.
static bool dense_rows(const gr_fleet* f)
{
    return f->req_cap >= f->bins && f->most_of_class <= kOwnClass && f->m_pos <= kOwnSlots &&
           (int64_t)f->bins * f->m_pos <= kDenseValues;
}

// Whether the fleet and the size of a batch are for the classes first (see launch_score).
bool classes_first(const gr_fleet* f, bool migrate, int64_t n)
{
    return !dense_rows(f) && n >= kByClassMin && f->n_class <= kGroup && f->n_run >= 4 * f->n_class &&
           f->n_run >= (migrate ? 2 * kGroup : 4 * kGroup);
}

bool needs_marks(const gr_fleet* f, int64_t n) { return !pair_by_pair(f, n) && !dense_rows(f); }

// Whether the instances are expected to have few entries in most blocks of rows (see k_memo): by the room of their tables and the
// rows there may be.  (Only tables that are read whole have that way.)  The line is at eight an instance and block on average, twice
// what a wave takes it with: decode lengths have long tails, which leave most blocks with far fewer and a few with most.
// Whole scans, us, without / with it, lengths up to 16 384 (128 and 64 of them: up to 4 096), in brackets spread evenly:
//   8 an instance and block   4 096 x 512 106.3 / 100.3 (211.5 / 212)   2 000 x 512 63.0 / 61.2 (100.2 / 104.0)   4 096 x 128 77.1 / 74.8 (65.7 / 67.5)
//   4                         4 096 x 250 74.5 / 70.3 (160 / 146)       3 000 x 64 52.4 / 51.4 (52.5 / 53.1)
//   2, 1                      4 096 x 125 68.8 / 66.7 (139 / 120)       4 096 x 60 52.8 / 51.5 (118.5 / 96.9)
// and refresh of 4 096 x 512 with 262 144 requests 66.8 / 66.1 (162.4 / 162.8).  Evenly spread, eight are never few, and the reads of the segments
// and a wave per SIMD less are for nothing; half as many are.
static bool sparse_rows(const gr_fleet* f, int64_t max_rows) { return f->cap <= 512 && (int64_t)f->cap * kMemoU <= 8 * max_rows; }

// How the rows of a pass are found.  (Lines and classes first are for fleets of more runs than have a row per length.)
struct RowsOf {
    const int* totals;
    const uint16_t* len_row;     // null: a row per length
    int64_t most;
};
static_assert(kOwnSlots / kMemoP <= 2 * kGroup, "a row per length and lines exclude each other");

static RowsOf rows_of(const gr_fleet* f, int64_t n)
{
    if (dense_rows(f)) return {f->dense_totals, nullptr, f->bins};
    return {f->totals, f->len_row, std::min<int64_t>(n, f->bins)};
}

static PairsArgs pairs_args(const gr_fleet* f, const ReqSrc& src, const ScoreOut& out)
{
    const RowsOf rows = rows_of(f, src.n);
    PairsArgs p{};
    p.ctx0 = src.ctx0; p.pred_len = src.pred_len; p.budget = src.budget; p.exclude = src.exclude;
    p.totals = rows.totals; p.len_row = rows.len_row; p.order = f->order; p.memo = f->memo; p.instK = f->instK; p.hD = f->hD;
    p.turned = f->turned; p.out_T = out.T; p.out_inst = out.inst; p.out_slack = out.slack; p.out_fallback = out.fallback;
    p.pos_of = f->pos_of;
    p.n = src.n; p.rows = f->turned_rows; p.n_inst = f->n_inst; p.m_pos = f->m_pos; p.max_len = f->max_len;
    return p;
}

static void launch_few(const gr_fleet* f, const ReqSrc& src, const ScoreOut& out, hipStream_t s)
{
    PairsArgs p = pairs_args(f, src, out);
    constexpr int64_t per = kBlock / kGroup * pairs_requests(true), most = kLaunchThreads / kBlock * per;
    for (p.first = 0; p.first < p.n; p.first += most)
        hipLaunchKernelGGL(k_select_few, dim3((unsigned)((std::min(p.n - p.first, most) + per - 1) / per)), dim3(kBlock), 0, s, p);
}

static void launch_pairs(gr_fleet* f, const ReqSrc& src, const ScoreOut& out, const PairsPlan& plan, int64_t max_rows,
                         hipStream_t s)
{
    PairsArgs p = pairs_args(f, src, out);
    const int64_t per = kBlock / plan.lanes * pairs_requests(plan.select), most = kLaunchThreads / kBlock * per;
    // (parts for as many rows as there may be; those past the last row end at once)
    for (p.row0 = 0; p.row0 < max_rows; p.row0 += p.rows) {
        {
            const int64_t rows = std::min<int64_t>(max_rows - p.row0, p.rows);
            ProfScope ps(f, kPairsRoute, s);
            hipLaunchKernelGGL(k_rows, dim3((unsigned)((rows + kWave - 1) / kWave * ((f->m_pos + kWave - 1) / kWave))), dim3(kBlock), 0, s, p);
        }
        for (p.first = 0; p.first < p.n; p.first += most) {
            const dim3 grid((unsigned)((std::min(p.n - p.first, most) + per - 1) / per));
            ProfScope ps(f, kPairsRoute, s);
#define GR_LAUNCH_PAIRS(N, S) do { \
            if (plan.four) hipLaunchKernelGGL((k_pairs<N, 4, S>), grid, dim3(kBlock), 0, s, p); \
            else hipLaunchKernelGGL((k_pairs<N, 1, S>), grid, dim3(kBlock), 0, s, p); } while (0)
            if (plan.lanes == 16) GR_LAUNCH_PAIRS(16, true);
            else if (plan.lanes == kWave) GR_LAUNCH_PAIRS(kWave, false);
            else GR_LAUNCH_PAIRS(kBlock, false);
#undef GR_LAUNCH_PAIRS
        }
    }
}

int launch_score(gr_fleet* f, const ReqSrc& src, bool migrate, const ScoreOut& out, hipStream_t s,
                 bool small_batch_ok)
{
    const int64_t n = src.n;
    if (n == 0) {
        if (out.n_selected) hipLaunchKernelGGL(k_set_int, dim3(1), dim3(1), 0, s, out.n_selected, 0);
        return hipGetLastError() == hipSuccess ? GR_OK : GR_ERR_HIP;
    }
    if (small_batch_ok && pair_by_pair(f, n)) {
        return migrate ? launch_pair_by_pair<true>(f, src, out, true, s)
                       : launch_pair_by_pair<false>(f, src, out, pairs_finite(f, n), s);
    }
    // The class order of the current status, if nobody is known to have made it, comes first: always while
    // the stream is being captured (a recorded pass may be replayed after a status build that was
    // recorded elsewhere), and always once a status build has been recorded.
    const TableAccount account(f, s);
    if (!account.ok) return GR_ERR_HIP;
    const TableView view = account.view(f);
    const bool with_order = !view.ordered, blended = view.blended;
    const int off = migrate ? kScanMigrate - kScanRoute : 0;
    const bool dense = dense_rows(f);
    const RowsOf rows = rows_of(f, n);
    OrderArgs o{};
    o.key = f->slot_key; o.instK = f->instK; o.slot_inst = f->slot_inst; o.run_cls = f->run_cls;
    o.order = f->order; o.pos_of = f->pos_of; o.posK = f->posK; o.posKey = f->posKey; o.run_head = f->run_head; o.m_pos = f->m_pos;
    if (!migrate && !dense) {
        ProfScope ps(f, kMarkRoute, s);
        constexpr int per = kBlock * kMarkItems;
        hipLaunchKernelGGL(k_mark, dim3((unsigned)((n + per - 1) / per)), dim3(kBlock), 0, s, src.pred_len, n, f->seen, f->max_len);
    }
    if (!dense) {
        ScanArgs sc{};
        sc.seen = f->seen; sc.row_len = f->row_len; sc.len_row = f->len_row; sc.totals = f->totals; sc.bins = f->bins;
        sc.late_cnt = f->late_cnt; sc.n_late = migrate ? f->n_inst * f->late_parts : 0; sc.out_n = out.n_selected;
        sc.flag = src.flag; sc.act_rem = src.act_rem; sc.act_off = src.act_off; sc.n = n; sc.n_inst = f->n_inst;
        ProfScope ps(f, kScanRoute + off, s);
        hipLaunchKernelGGL(k_scan, dim3(kScanGroups + (with_order ? order_blocks(f->m_pos, kScanBlock) : 0)), dim3(kScanBlock), 0, s, sc, o);
    }
    account.v->ordered = true;
    const int64_t max_rows = rows.most;
    // Classes first in large batches on fleets of many runs.  Whole routing call, us, a group of lanes per
    // request / classes first; in brackets with deadlines that most requests can meet, where
    // the classes only say which runs to look at:
    //   instances   65 536 requests          262 144 requests
    //      512      26.1 / 25.1 (27.0 / 37.3)   49.7 / 34.3 (55.0 / 73.9)
    //    1 024      32.2 / 29.8 (33.0 / 39.0)   68.4 / 42.9 (73.1 / 77.0)
    //    4 096      54.6 / 51.6 (55.2 / 55.6)    126 / 89.9  (133 / 109)
    // A risk scan's requests are late where they are, and few can be served in time elsewhere:
    // 512 x 512 requests 57.6 / 41.2 (42.0 / 42.0), 4 096 x 512 544 / 110 (278 / 137).
    // Fleets with a row per length have four lanes per request as an alternative: four classes of 128, scan of x 300
    // 29.9 / 35.7 (27.1 / 34.3), x 512 33.1 / 38.7 (31.4 / 40.2).
    const PairsPlan pairs(f, out.T);
    const bool select = !(out.T && pairs.select);
    const bool by_class = select && !blended && classes_first(f, migrate, n);
    // The lines first where no class decides a request: with a blend (every instance has its own prefill rate), and where
    // there are more classes than a group has lanes.  Whole calls, us, a group of lanes per request over the runs / lines
    // first (weight 1; in brackets deadlines that many instances meet):
    //   262 144 requests on 4 096 instances  92 / 61 (114 / 103), on 1 024 of 64 classes, no blend, 68 / 54 (57 / 69)
    //   a scan of 1 024 x 1 000             164 / 70 (179 / 131)   4 096 x 400  355 / 107 (226 / 147)
    //   a scan of 2 048 x 100                78 / 62 (36 / 37)     1 400 x 99   56 / 49 (31 / 38)
    // Below 2^17 requests the lookup (10 to 14 us) is not won back, in a scan below 3 * 2^16, of which hardly any may be
    // late; below 81 runs a group reads all of them at once, so only the largest scans gain.
    // A scan takes a lane per request and lists the rest, as most of it may not be late at all (3 270 x 130, a
    // group of lanes per request from the lines on: 125 us, listed 92).
    const bool by_lines = select && (blended || f->n_class > kGroup) && n >= (migrate ? kLinesScanMin : kByClassMin) &&
                          f->n_run > (migrate && n >= kLinesMany ? 2 : 5) * kGroup;
    const bool listed = by_lines && migrate && f->n_run <= kRestRuns;
    // The runs' minima in blocks of rows where the classes are looked at first (6 us less for the
    // table of 7 061 rows x 4 096 instances); else row by row: a request's 16 lanes then read 16
    // runs from one cache line, not from sixteen.  (Of a routing batch many requests may get as far as the runs, see k_class.)
    const bool blocks = by_class, rows_too = by_class && !migrate;
    const bool own = dense && with_order;
    {
        MemoArgs m{};
        m.own = o; m.run_cls = f->run_cls;
        if (dense && migrate) m.count = count_args(f, src, out);
        m.totals = f->totals; m.row_len = f->row_len; m.len_row = f->len_row; m.order = f->order; m.instK = f->instK;
        m.tabR = f->tabR; m.tabGH = f->tabGH; m.memo = f->memo; m.grp_min = f->grp_min;
        m.run_k = f->run_k; m.run_rank = f->run_rank; m.pos_thr = f->pos_thr; m.run_at = f->run_at; m.posK = f->posK; m.posKey = f->posKey;
        m.run_head = f->run_head;
        m.seen = reinterpret_cast<uint4*>(f->seen); m.seen_words = dense ? 0 : (f->bins + 15) / 16;
        m.n_run = f->n_run; m.bins = f->bins; m.run_pad = f->run_pad; m.cap = f->cap;
        // (workgroups for as many rows as there may be; those past the last row end at once)
        // (a run's workgroups on one XCD: the runs rounded up to a multiple of the XCDs)
        const dim3 grid((unsigned)((f->n_run + 7) / 8 * 8), (unsigned)(1 + (max_rows + kMemoU - 1) / kMemoU));
        ProfScope ps(f, kMemoRoute + off, s);
#define GR_LAUNCH_MEMO(B, D, O) do { \
        if (f->cap > 1024) hipLaunchKernelGGL((k_memo<4, B, D, O, false>), grid, dim3(kBlock), 0, s, m); \
        else if (f->cap > 512) hipLaunchKernelGGL((k_memo<2, B, D, O, false>), grid, dim3(kBlock), 0, s, m); \
        else hipLaunchKernelGGL((k_memo<1, B, D, O, false>), grid, dim3(kBlock), 0, s, m); } while (0)
        if (blocks && sparse_rows(f, max_rows)) hipLaunchKernelGGL((k_memo<1, true, false, false, true>), grid, dim3(kBlock), 0, s, m);
        else if (blocks) GR_LAUNCH_MEMO(true, false, false);
        else if (own) GR_LAUNCH_MEMO(false, true, true);
        else if (dense) GR_LAUNCH_MEMO(false, true, false);
        else GR_LAUNCH_MEMO(false, false, false);
#undef GR_LAUNCH_MEMO
    }
    if (by_class) {
        ClassArgs c{};
        c.totals = f->totals; c.cls_run = f->cls_run; c.order = f->order; c.memo = f->memo; c.grp_min = f->grp_min;
        c.run_k = f->run_k; c.row_min = f->row_min; c.row_len = f->row_len; c.class_least = f->class_least; c.run_rank = f->run_rank; c.cls_rank = f->cls_rank;
        c.n_class = f->n_class; c.class_shift = f->class_shift; c.n_run = f->n_run; c.run_pad = f->run_pad;
        ProfScope ps(f, kClassRoute + off, s);
        const dim3 grid((unsigned)((max_rows + kWave - 1) / kWave * f->n_class));
        if (rows_too) hipLaunchKernelGGL(k_class<true>, grid, dim3(kBlock), 0, s, c);
        else hipLaunchKernelGGL(k_class<false>, grid, dim3(kBlock), 0, s, c);
    }
    if (select) {
        SelectArgs a{};
        a.s = src; a.len_row = rows.len_row; a.order = f->order; a.memo = f->memo; a.grp_min = rows_too ? f->row_min : f->grp_min; a.run_k = f->run_k;
        a.posK = f->posK; a.posKey = f->posKey; a.run_rank = f->run_rank; a.pos_thr = f->pos_thr; a.run_at = f->run_at; a.cls_run = f->cls_run; a.class_least = f->class_least; a.clsK = f->clsK; a.cls_rank = f->cls_rank;
        a.out_inst = out.inst; a.out_slack = out.slack; a.out_fallback = out.fallback;
        a.run_pad = f->run_pad; a.n_run = f->n_run; a.n_class = f->n_class; a.class_shift = f->class_shift;
        a.max_len = f->max_len; a.n_inst = f->n_inst;
        a.lines = f->lines; a.totals = f->totals; a.row_len = f->row_len; a.pos_of = f->pos_of;
        a.rest_cnt = f->rest_cnt;
        if (by_lines) {
            constexpr int per = kBlock / kWave;
            const dim3 grid((unsigned)((max_rows * kRanges + per - 1) / per));
            ProfScope ps(f, kLinesRoute + off, s);
            if (f->n_run <= 2 * kWave) hipLaunchKernelGGL(k_lines<2>, grid, dim3(kBlock), 0, s, a);
            else hipLaunchKernelGGL(k_lines<5>, grid, dim3(kBlock), 0, s, a);      // (4 096 instances of three classes are 258 runs)
        }
        if (listed) {
            // (the lists use the room for finish times of feedback routing, a word per running request)
            a.rest = reinterpret_cast<int*>(f->scratch_finish);
            a.segments = (int)((n + kBlock * kRestItems - 1) / (kBlock * kRestItems));
            {
                ProfScope ps(f, kSelectMigrate, s);
                hipLaunchKernelGGL(k_late_lines<kRestItems>, dim3(a.segments), dim3(kBlock), 0, s, a);
            }
            ProfScope ps(f, kSelectMigrate, s);
            hipLaunchKernelGGL(k_late_rest, dim3(kRestParts * kRestBlocks), dim3(kBlock), 0, s, a, kBlock * kRestItems);
        } else {
            ProfScope ps(f, kSelectRoute + off, s);
            if (!migrate && f->n_inst <= kFewInst) launch_few(f, src, out, s);
            else if (migrate) launch_select<true>(f, a, by_class, by_lines, blended, s);
            else launch_select<false>(f, a, by_class, by_lines, blended, s);
        }
    }
    if (out.T) launch_pairs(f, src, out, pairs, max_rows, s);
    return hipGetLastError() == hipSuccess ? GR_OK : GR_ERR_HIP;
}

int launch_hits(gr_fleet* f, const ReqSrc& src, const int* hit_off, const int* hit_inst, const int* hit_len,
                int64_t n_hits, const ScoreOut& out, hipStream_t s)
{
    if (src.n == 0 || n_hits == 0) return GR_OK;
    HitArgs h{};
    h.ctx0 = src.ctx0; h.pred_len = src.pred_len; h.budget = src.budget; h.exclude = src.exclude;
    h.hit_off = hit_off; h.hit_inst = hit_inst; h.hit_len = hit_len;
    h.len_row = rows_of(f, src.n).len_row; h.pos_of = f->pos_of; h.memo = f->memo; h.posK = f->posK; h.posKey = f->posKey;
    h.out_inst = out.inst; h.out_slack = out.slack; h.out_fallback = out.fallback; h.out_T = out.T;
    h.n = src.n; h.n_hits = n_hits; h.n_inst = f->n_inst; h.n_run = f->n_run; h.max_len = f->max_len;
    ProfScope ps(f, kHitsRoute, s);
    const auto groups = [&](int lanes) { return dim3((unsigned)((src.n * lanes + kBlock - 1) / kBlock)); };
    if (out.T || src.n > kLaunchThreads / kHitLanes) hipLaunchKernelGGL(k_hits<1>, groups(1), dim3(kBlock), 0, s, h);
    else hipLaunchKernelGGL(k_hits<kHitLanes>, groups(kHitLanes), dim3(kBlock), 0, s, h);
    return hipGetLastError() == hipSuccess ? GR_OK : GR_ERR_HIP;
}

}  // namespace gr
