// The planning strategies that Section 2.3 sets beside greedy_by_size:
// bump_allocation, the baseline that never reuses memory, and the optimum of
// Eq. 2.1, which the thesis reaches through a MIP solver and which here is a
// branch and bound search over placement orders for tiny traces.
#include "internal.hpp"
#include "mp_device.hpp"

namespace mp {

namespace {

constexpr int kSBlock = 256;

// ---------------------------------------------------------------------------
// bump_allocation: each allocation, in the order they happen (first op, then
// id), goes at a running offset that then grows by its size.  Per trace: a
// stable radix sort by (trace, first op), an exclusive scan of the sizes in
// that order, and each offset is its scan value minus its trace's start.

struct BumpFlags {
    uint32_t abort;  // input rejected: every later kernel does nothing
    uint32_t pad;
    unsigned long long sum;
};

__global__ void bump_init_kernel(BumpFlags* fl) {
    fl->abort = 0;
    fl->pad = 0;
    fl->sum = 0;
}

// Checks the tensors (and the trace bounds), and writes each tensor's sort
// key (trace << op_bits) | first with its id.  A grid-stride loop over a
// bounded grid: the blocks add their sums of sizes into one word, and fewer
// blocks mean fewer of those same-address atomics.
constexpr unsigned kKeysGrid = 256;
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void bump_keys_kernel(
    const int64_t* __restrict__ begin, int64_t n_seg, const int64_t* __restrict__ size,
    const int32_t* __restrict__ first, const int32_t* __restrict__ last, int64_t n,
    int32_t num_ops, int op_bits, uint64_t* __restrict__ keys, uint32_t* __restrict__ vals,
    BumpFlags* fl, int32_t* status) {
    __shared__ uint64_t red[BLOCK / kWave];
    const int64_t items = max(n, begin ? n_seg + 1 : (int64_t)0);
    uint32_t bad = 0;
    uint64_t acc = 0;
    for (int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x; i < items;
         i += (int64_t)gridDim.x * BLOCK) {
        if (begin && i <= n_seg) {  // trace bounds: 0 = begin[0] <= ... <= begin[n_seg] = n
            const int64_t b = begin[i];
            if ((i == 0 && b != 0) || (i == n_seg && b != n) || (i < n_seg && begin[i + 1] < b))
                bad = 1;
        }
        if (i < n) {
            const int64_t s = size[i];
            const int32_t f = first[i], l = last[i];
            if (s <= 0 || f < 0 || f > l || l >= num_ops) bad = 1;
            else acc = sat_add(acc, (uint64_t)s);
            int64_t seg = 0;  // the last trace whose begin is <= i
            if (begin) {
                int64_t lo = 0, hi = n_seg - 1;
                while (lo < hi) {
                    const int64_t mid = lo + (hi - lo + 1) / 2;
                    if (begin[mid] <= i) lo = mid;
                    else hi = mid - 1;
                }
                seg = lo;
            }
            keys[i] = ((uint64_t)seg << op_bits) | (uint32_t)max(f, 0);
            vals[i] = (uint32_t)i;
        }
    }
    bad = block_reduce<BLOCK>((uint64_t)bad, OpOr<uint64_t>(), red) != 0;
    acc = block_reduce<BLOCK>(acc, OpSatAdd(), red);
    if (threadIdx.x == 0) {
        if (bad) {
            raise_status(status, MP_EINVAL);
            atomicOr(&fl->abort, 1u);
        }
        const uint64_t old = atomicAdd(&fl->sum, (unsigned long long)acc);
        if (acc > (uint64_t)INT64_MAX || old > (uint64_t)INT64_MAX - acc) {
            raise_status(status, MP_EOVERFLOW);
            atomicOr(&fl->abort, 1u);
        }
    }
}

__global__ __launch_bounds__(kSBlock) void bump_gather_kernel(const int64_t* __restrict__ size,
                                                              const uint32_t* __restrict__ vals,
                                                              int64_t n, int64_t* __restrict__ sz,
                                                              const BumpFlags* fl) {
    if (fl->abort) return;
    const int64_t k = (int64_t)blockIdx.x * kSBlock + threadIdx.x;
    if (k < n) sz[k] = size[vals[k]];
}

// scan[k] = sizes before sorted position k; a trace's tensors hold sorted
// positions [begin[s], begin[s + 1]), so its start is scan[begin[s]].
__global__ __launch_bounds__(kSBlock) void bump_write_kernel(
    const int64_t* __restrict__ begin, int64_t n_seg, const uint64_t* __restrict__ keys,
    const uint32_t* __restrict__ vals, const int64_t* __restrict__ scan,
    const int64_t* __restrict__ total, int64_t n, int op_bits, int64_t* __restrict__ offset_out,
    int64_t* __restrict__ peak_out, const BumpFlags* fl) {
    if (fl->abort) return;
    const int64_t k = (int64_t)blockIdx.x * kSBlock + threadIdx.x;
    auto before = [&](int64_t e) { return e < n ? scan[e] : *total; };
    if (k < n) {
        const int64_t seg = (int64_t)(keys[k] >> op_bits);
        offset_out[vals[k]] = scan[k] - (begin ? before(begin[seg]) : 0);
    }
    const int64_t nseg = begin ? n_seg : 1;
    if (k < nseg)
        peak_out[k] = begin ? before(begin[k + 1]) - before(begin[k]) : *total;
}

struct BumpLayout {
    size_t flags, keys0, keys1, sz, partial, radix, vals0, vals1, end;
};

BumpLayout bump_layout(int64_t n) {
    const size_t nn = (size_t)(n > 0 ? n : 1);
    BumpLayout L;
    size_t at = 0;
    auto take = [&](size_t bytes) {
        const size_t here = at;
        at += (bytes + 255) & ~(size_t)255;
        return here;
    };
    L.flags = take(sizeof(BumpFlags));
    L.keys0 = take(nn * 8);
    L.keys1 = take(nn * 8);
    L.sz = take(nn * 8);
    L.partial = take(scan_workspace_bytes((int64_t)nn));
    L.radix = take(radix_workspace_bytes((int64_t)nn));
    L.vals0 = take(nn * 4);
    L.vals1 = take(nn * 4);
    L.end = at;
    return L;
}

int bit_width64(uint64_t x) { return x ? 64 - __builtin_clzll(x) : 0; }

// ---------------------------------------------------------------------------
// The optimum of Eq. 2.1 for a tiny trace.  List an optimal plan by (offset,
// tensor) and put each tensor, in that order, at the lowest offset clear of the
// ones before it: no tensor moves up, so the peak stays optimal, and repeating
// it ends (the offsets' sum falls) in a plan whose own order reproduces it.  In
// that order offsets never fall, so a tensor's place is simply the highest end
// among its neighbours placed before it (its base), and it is enough to search
// orders in which
//   - (base, tensor) does not fall from one tensor to the next, and
//   - no tensor is put at or above the end that another unplaced tensor would
//     have at its own base (nothing later could cover that place, so the other
//     one would not be at its lowest offset).
// A subtree is cut when an unplaced tensor, or the unplaced tensors alive at
// one op stacked from the last offset on, cannot end below the best peak; the
// search stops at the live-bytes lower bound.  The best starts at the greedy by
// size plan, which reaches the bound for nine in ten of the tiny ResNeXt-like
// traces, or else at the best of 128 other greedy plans.
//
// One wave per trace.  Tensors are numbered by size descending, so the masks
// below are the same for every lane and sit in scalar registers; a lane holds
// its tensors' ends in registers and searches depth first below prefixes of the
// order (the first kOptPrefix levels, dealt to the lanes as they become free).
// Each turn of the loop evaluates the lane's node and either places a tensor or
// backs up, without memory accesses: bound by instruction issue (several hundred
// vector instructions a turn) and by the longest search of the batch.  All
// lanes share the best peak through ballots, so the plan found does not depend
// on timing.  2048 traces of 10 tensors: 6.80 ms for the search over all n!
// orders in one workgroup a trace, 0.10 ms for this one.

constexpr int kOptMaxN = MP_OPT_MAX_N;
static_assert(kOptMaxN <= 15, "tensor numbers in 4 bits");

struct OptShared {
    int64_t sz[kOptMaxN];      // by rank (size descending, id)
    int32_t first[kOptMaxN], last[kOptMaxN];
    int32_t id[kOptMaxN];
    uint32_t meets[kOptMaxN];  // bit j: lifetimes of i and j meet (j != i)
    uint32_t alive[kOptMaxN];  // bit j: j is alive at i's first op
    int32_t by_area[kOptMaxN]; // numbers by size times lifetime descending
};

__device__ __forceinline__ uint32_t opt_uniform(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}
__device__ __forceinline__ uint64_t opt_uniform(uint64_t v) {
    return ((uint64_t)opt_uniform((uint32_t)(v >> 32)) << 32) | opt_uniform((uint32_t)v);
}
template <typename T>
__device__ __forceinline__ T opt_wave_min(T v) {
    return wave_reduce(v, OpMin<T>());
}

// The search over T counts of the trace's unit.  `ends`: this lane's best plan so
// far, `mine` its peak, `best` the least of them; returns the least peak found.
template <typename T, int N>
__device__ __forceinline__ T opt_search(const OptShared& S, int n, int sh, T lb, T best, T (&ends)[N],
                                        T& mine) {
    const int lane = threadIdx.x & (kWave - 1);
    const uint64_t below = (1ull << lane) - 1ull;
    const uint32_t all = (1u << n) - 1u;
    T sz[N];
    uint32_t meets[N], alive[N];
    T left0[N];  // sizes alive at i's first op, all unplaced
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int c = i < n ? i : 0;
        sz[i] = i < n ? opt_uniform((T)((uint64_t)S.sz[c] >> sh)) : T(0);
        meets[i] = i < n ? opt_uniform(S.meets[c]) : 0u;
        alive[i] = i < n ? opt_uniform(S.alive[c]) : 0u;
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        left0[i] = 0;
#pragma unroll
        for (int j = 0; j < N; ++j) left0[i] += ((alive[i] >> j) & 1u) ? sz[j] : T(0);
    }
    // prefixes of two tensors (at most 132 for 64 lanes), or of three from 11
    // tensors on, where single subtrees get long enough to idle the others
    const int d = n < 2 ? n : (n <= 10 ? 2 : 3);
    uint32_t n_pre = 1;
    for (int k = 0; k < d; ++k) n_pre *= (uint32_t)(n - k);
    uint32_t next_pre = 0;  // uniform

    T end[N];   // ends of the placed tensors, 0 while unplaced
    T left[N];  // sizes of the unplaced tensors alive at i's first op
    uint64_t order = 0;  // 4 bits a level
    uint32_t placed = 0, from = 0, forced = 0;
    int level = 0;
    bool busy = false, out = false;
    while (true) {
        // lanes without a subtree take the next prefixes, in lane order
        const uint64_t want = __ballot(!busy && !out);
        if (want) {
            const uint32_t p = next_pre + (uint32_t)__popcll(want & below);
            if (!busy && !out) {
                if (p < n_pre) {
                    busy = true;
                    uint32_t q = p, free_ids = all;
                    forced = 0;
                    for (int k = 0; k < d; ++k) {  // the p-th prefix, in mixed radix
                        const uint32_t r = (uint32_t)(n - k), digit = q % r;
                        q /= r;
                        uint32_t f = free_ids;
                        for (uint32_t t = 0; t < digit; ++t) f &= f - 1;
                        const uint32_t c = (uint32_t)__builtin_ctz(f);
                        forced |= c << (4 * k);
                        free_ids &= ~(1u << c);
                    }
                    placed = from = 0;
                    order = 0;
                    level = 0;
#pragma unroll
                    for (int i = 0; i < N; ++i) {
                        end[i] = 0;
                        left[i] = left0[i];
                    }
                } else {
                    out = true;
                }
            }
            next_pre += (uint32_t)__popcll(want);
        }
        if (!__ballot(busy)) break;
        // ---- the node: bases, the cuts, and the tensors that may come next
        const int prev = level ? (int)((order >> (4 * (level - 1))) & 15u) : -1;
        T last = 0, limit = ~T(0), need = 0;
#pragma unroll
        for (int i = 0; i < N; ++i) last = i == prev ? end[i] - sz[i] : last;
        T base[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            T b = 0;
            T top = 0;  // highest end at i's first op
            // the masks go through an empty asm each turn: hoisted out of the
            // loop, their bits became 132 lane masks and were spilled
            uint32_t mi = meets[i], ai = alive[i];
            asm volatile("" : "+s"(mi), "+s"(ai));
#pragma unroll
            for (int j = 0; j < N; ++j) {
                const T e = end[j] & (T)(int64_t)((int32_t)(mi << (31 - j)) >> 31);
                const T a = end[j] & (T)(int64_t)((int32_t)(ai << (31 - j)) >> 31);
                b = e > b ? e : b;
                top = a > top ? a : top;
            }
            base[i] = b;
            const bool un = i < n && !((placed >> i) & 1u);
            const T e = b + sz[i], h = (b > last ? b : last) + sz[i];
            limit = un && e < limit ? e : limit;
            need = un && h > need ? h : need;
            // the tensors left at i's first op, stacked on those placed there
            const T l = (top > last ? top : last) + left[i];
            need = i < n && left[i] && l > need ? l : need;
        }
        uint32_t cand = 0;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const bool ok = base[i] < limit && (base[i] > last || (base[i] == last && i > prev));
            cand |= ok ? 1u << i : 0u;
        }
        cand = need < best ? cand & all & ~placed & ~((1u << from) - 1u) : 0u;
        const bool pre = level < d;
        if (pre) cand &= 1u << ((forced >> (4 * level)) & 15u);
        const bool place = busy && cand != 0;
        // ---- place the lowest candidate, or take the last tensor back
        const int c = place ? (int)__builtin_ctz(cand) : prev;
        // a prefix that cannot be placed, or whose subtree is done, is left
        const bool drop = busy && !place && (pre || level == d);
        const bool back = busy && !place && !drop;
        const bool moves = place || back;
        uint32_t at = 0;
        T s = 0;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            s = i == c ? sz[i] : s;
            const T e = place ? base[i] + sz[i] : T(0);
            end[i] = moves && i == c ? e : end[i];
            at |= ((alive[i] >> (c & 31)) & 1u) << i;  // the first ops at which c is alive
        }
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const T v = moves && ((at >> i) & 1u) ? s : T(0);
            left[i] = place ? left[i] - v : left[i] + v;
        }
        if (place) {
            order |= (uint64_t)c << (4 * level);
            placed |= 1u << c;
            ++level;
            from = 0;
        } else if (back) {
            --level;
            order &= ~(15ull << (4 * level));
            placed &= ~(1u << c);
            from = (uint32_t)c + 1u;
        }
        if (drop) busy = false;
        if (__ballot(busy && level == n)) {  // complete orders
            T pk = ~T(0);
            if (busy && level == n) {
                pk = 0;
#pragma unroll
                for (int i = 0; i < N; ++i) pk = end[i] > pk ? end[i] : pk;
                if (pk < mine) {
                    mine = pk;
#pragma unroll
                    for (int i = 0; i < N; ++i) ends[i] = end[i];
                }
                if (n == d) busy = false;  // the prefix was the whole order
            }
            const T low = opt_wave_min(pk);
            best = low < best ? low : best;
            if (best <= lb) break;
        }
    }
    return best;
}

// Before the search: 64 greedy plans at once, lane l's with two tensors put first
// (the l-th pair) and the rest by size or by area.  Nine in ten of the tiny
// ResNeXt-like traces that greedy by size leaves above the live-bytes bound reach it
// so, whose searches made up most of the time: three sets of 400 traces of 8
// tensors, launch and all, 66, 130 and 83 us without and 61, 30 and 30 with them, of
// 9 tensors 80, 84 and 92 and 35, 35 and 44 (a workgroup a trace over all orders: 51,
// 52, 52 and 56, 698, 60).
template <typename T, int N>
__device__ __forceinline__ T opt_variants(const OptShared& S, int n, int sh, bool area, T best,
                                          T (&ends)[N], T& mine) {
    const uint32_t pair = threadIdx.x % (uint32_t)(n * (n - 1));
    const uint32_t p0 = pair % (uint32_t)n, q = pair / (uint32_t)n, p1 = q + (q >= p0 ? 1u : 0u);
    T off[N], end[N], pk = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) off[i] = end[i] = 0;
    uint32_t left = (1u << n) - 1u;  // positions of the order
    for (int t = 0; t < n; ++t) {
        const uint32_t pos = t == 0 ? p0 : (t == 1 ? p1 : (uint32_t)__builtin_ctz(left));
        left &= ~(1u << pos);
        const uint32_t c = area ? (uint32_t)S.by_area[pos] : pos;
        const T w = (T)((uint64_t)S.sz[c] >> sh);
        const uint32_t nb = S.meets[c];
        T hi[N];  // ends of the placed neighbours, 0 of the others
#pragma unroll
        for (int j = 0; j < N; ++j) hi[j] = (nb >> j) & 1u ? end[j] : T(0);
        T x = 0;
        while (true) {  // past the highest end among the ranges that overlap, until none does
            T up = 0;
#pragma unroll
            for (int j = 0; j < N; ++j) up = off[j] < x + w && x < hi[j] && hi[j] > up ? hi[j] : up;
            if (!__ballot(up != 0)) break;
            x = up ? up : x;
        }
#pragma unroll
        for (int j = 0; j < N; ++j) {
            off[j] = (uint32_t)j == c ? x : off[j];
            end[j] = (uint32_t)j == c ? x + w : end[j];
        }
        pk = x + w > pk ? x + w : pk;
    }
    if (pk < mine) {
        mine = pk;
#pragma unroll
        for (int i = 0; i < N; ++i) ends[i] = end[i];
    }
    const T low = opt_wave_min(mine);
    return low < best ? low : best;
}

// Numbers by area, for the second set of greedy plans.
__device__ __forceinline__ void opt_areas(OptShared& S, int n) {
    const int lane = threadIdx.x & (kWave - 1);
    auto area = [&](int i) { return (double)S.sz[i] * (double)(S.last[i] - S.first[i] + 1); };
    if (lane < n) {
        const double a = area(lane);
        int r = 0;
        for (int j = 0; j < n; ++j) r += area(j) > a || (area(j) == a && j < lane) ? 1 : 0;
        S.by_area[r] = lane;
    }
    __syncthreads();
}

// Greedy by size over T units (tensors in rank order, each at the lowest
// offset that fits), by one wave: lane a tries the end of tensor a, lane n
// offset 0.  Returns the peak; ends[] the same in every lane.
template <typename T, int N>
__device__ __forceinline__ T opt_greedy(const OptShared& S, int n, int sh, T (&ends)[N]) {
    const int lane = threadIdx.x & (kWave - 1);
    T pk = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) ends[i] = 0;
    T my_end = 0;  // of the tensor this lane holds
    for (int t = 0; t < n; ++t) {
        const T s = (T)((uint64_t)S.sz[t] >> sh);
        const uint32_t nb = S.meets[t] & ((1u << t) - 1u);
        bool ok = lane == n || ((nb >> (lane & 31)) & 1u && lane < t);
        const T x = lane == n ? T(0) : my_end;
        for (uint32_t m = nb; m; m &= m - 1) {
            const int j = __builtin_ctz(m);
            const T e = (T)__shfl(my_end, j, kWave), o = e - (T)((uint64_t)S.sz[j] >> sh);
            if (x < e && o < x + s) ok = false;
        }
        const T at = opt_wave_min(ok ? x : ~T(0));
        if (lane == t) my_end = at + s;
        pk = at + s > pk ? at + s : pk;
#pragma unroll
        for (int i = 0; i < N; ++i) ends[i] = i == t ? at + s : ends[i];
    }
    return pk;
}

template <typename T, int N>
__device__ __forceinline__ void opt_plan(OptShared& S, int n, int sh, uint64_t lb_bytes, int64_t b0,
                         int64_t* __restrict__ offset_out, int64_t* __restrict__ peak) {
    const int lane = threadIdx.x & (kWave - 1);
    const T lb = (T)(lb_bytes >> sh);
    T ends[N], mine;
    T best = opt_greedy<T, N>(S, n, sh, ends);
    mine = best;
#pragma unroll 1  // one copy of the code, fetched once
    for (int area = 0; area < 2 && best > lb; ++area) {
        if (area) opt_areas(S, n);
        best = opt_variants<T, N>(S, n, sh, area != 0, best, ends, mine);
    }
    if (best > lb) best = opt_search<T, N>(S, n, sh, lb, best, ends, mine);
    const uint64_t win = __ballot(mine == best);
    if (lane == (int)__builtin_ctzll(win)) {
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (i < n) offset_out[b0 + S.id[i]] = (int64_t)((uint64_t)ends[i] << sh) - S.sz[i];
        *peak = (int64_t)((uint64_t)best << sh);
    }
}

// A turn goes over all pairs of the N tensors it is written out for.
template <typename T>
__device__ __forceinline__ void opt_plan_n(OptShared& S, int n, int sh, uint64_t lb, int64_t b0,
                                           int64_t* __restrict__ offset_out,
                                           int64_t* __restrict__ peak) {
    if (n <= 8) opt_plan<T, 8>(S, n, sh, lb, b0, offset_out, peak);
    else if (n <= 10) opt_plan<T, 10>(S, n, sh, lb, b0, offset_out, peak);
    else opt_plan<T, kOptMaxN>(S, n, sh, lb, b0, offset_out, peak);
}

__global__ __launch_bounds__(kWave) void optimal_kernel(
    const int64_t* __restrict__ begin, const int32_t* __restrict__ num_ops,
    const int64_t* __restrict__ size, const int32_t* __restrict__ first,
    const int32_t* __restrict__ last, int64_t n_tensors, int64_t* __restrict__ offset_out,
    int64_t* __restrict__ peak_out, int32_t* __restrict__ status) {
    __shared__ OptShared S;
    const int lane = threadIdx.x;
    const int64_t b0 = begin[blockIdx.x], b1 = begin[blockIdx.x + 1];
    const int64_t nn = b1 - b0;
    if (b0 < 0 || b1 > n_tensors || nn < 0 || nn > kOptMaxN) {
        if (lane == 0) raise_status(status, MP_EINVAL);
        return;
    }
    const int n = (int)nn;
    int64_t s = 0;
    int32_t f = 0, l = 0;
    bool bad = false;
    if (lane < n) {
        s = size[b0 + lane];
        f = first[b0 + lane];
        l = last[b0 + lane];
        bad = s <= 0 || f < 0 || f > l || l >= num_ops[blockIdx.x];
    }
    if (__ballot(bad)) {
        if (lane == 0) raise_status(status, MP_EINVAL);
        return;
    }
    const uint64_t total = wave_reduce((uint64_t)s, OpSatAdd());
    if (total > (uint64_t)INT64_MAX) {
        if (lane == 0) raise_status(status, MP_EOVERFLOW);
        return;
    }
    if (n == 0) {
        if (lane == 0) peak_out[blockIdx.x] = 0;
        return;
    }
    // ranks, lifetimes that meet, and the live bytes at each tensor's first op
    // (the most live bytes are reached at some tensor's first op)
    int rank = 0;
    for (int j = 0; j < n; ++j) {
        const int64_t sj = __shfl(s, j, kWave);
        rank += (sj > s || (sj == s && j < lane)) ? 1 : 0;
    }
    if (lane < n) {
        S.sz[rank] = s;
        S.first[rank] = f;
        S.last[rank] = l;
        S.id[rank] = lane;
    }
    __syncthreads();
    uint64_t live = 0;
    if (lane < n) {
        uint32_t meets = 0, alive = 0;
        for (int j = 0; j < n; ++j) {
            if (j != lane && S.first[lane] <= S.last[j] && S.first[j] <= S.last[lane])
                meets |= 1u << j;
            if (S.first[j] <= S.first[lane] && S.first[lane] <= S.last[j]) {
                alive |= 1u << j;
                live += (uint64_t)S.sz[j];
            }
        }
        S.meets[lane] = meets;
        S.alive[lane] = alive;
    }
    const uint64_t lb = wave_reduce(live, OpMax<uint64_t>());
    const uint64_t orv = wave_reduce((uint64_t)s, OpOr<uint64_t>());
    __syncthreads();
    const int sh = __builtin_ctzll(orv);
    // 32-bit counts of the common unit while two sums of the sizes fit them
    if ((total >> sh) < (1ull << 31))
        opt_plan_n<uint32_t>(S, n, sh, lb, b0, offset_out, peak_out + blockIdx.x);
    else
        opt_plan_n<uint64_t>(S, n, sh, lb, b0, offset_out, peak_out + blockIdx.x);
}

}  // namespace

size_t bump_workspace_bytes(int64_t n) {
    if (n < 0 || n >= INT32_MAX) return 0;
    return bump_layout(n).end;
}

hipError_t launch_bump(const int64_t* begin, int64_t n_seg, const int64_t* size,
                       const int32_t* first, const int32_t* last, int64_t n, int32_t num_ops,
                       int64_t* offset_out, int64_t* peak_out, void* ws, int32_t* status,
                       hipStream_t st) {
    const BumpLayout L = bump_layout(n);
    char* w = static_cast<char*>(ws);
    BumpFlags* fl = reinterpret_cast<BumpFlags*>(w + L.flags);
    uint64_t* k0 = reinterpret_cast<uint64_t*>(w + L.keys0);
    uint64_t* k1 = reinterpret_cast<uint64_t*>(w + L.keys1);
    uint32_t* v0 = reinterpret_cast<uint32_t*>(w + L.vals0);
    uint32_t* v1 = reinterpret_cast<uint32_t*>(w + L.vals1);
    int64_t* sz = reinterpret_cast<int64_t*>(w + L.sz);
    int64_t* partial = reinterpret_cast<int64_t*>(w + L.partial);
    const int op_bits = bit_width64(num_ops > 1 ? (uint64_t)(num_ops - 1) : 0);
    const int seg_bits = begin ? bit_width64(n_seg > 1 ? (uint64_t)(n_seg - 1) : 0) : 0;
    const int64_t items = max(n, begin ? n_seg + 1 : (int64_t)0);
    const unsigned nb = (unsigned)((max(items, (int64_t)1) + kSBlock - 1) / kSBlock);
    hipLaunchKernelGGL(bump_init_kernel, dim3(1), dim3(1), 0, st, fl);
    if (nb <= kKeysGrid)
        hipLaunchKernelGGL(bump_keys_kernel<kSBlock>, dim3(nb), dim3(kSBlock), 0, st, begin, n_seg,
                           size, first, last, n, num_ops, op_bits, k0, v0, fl, status);
    else
        hipLaunchKernelGGL(bump_keys_kernel<1024>, dim3(kKeysGrid), dim3(1024), 0, st, begin, n_seg,
                           size, first, last, n, num_ops, op_bits, k0, v0, fl, status);
    bool alt = false;
    // An even number of digits: inputs that are in order already (recorded
    // traces are) then stay where they are, without a pass over the pairs.
    const int key_bits = min((op_bits + seg_bits + 15) / 16 * 16, 64);
    hipError_t e = radix_sort_pairs(k0, v0, k1, v1, n, 0, key_bits, w + L.radix, &alt, st,
                                    &fl->abort);
    if (e != hipSuccess) return e;
    const uint64_t* ks = alt ? k1 : k0;
    const uint32_t* vs = alt ? v1 : v0;
    const unsigned ng = (unsigned)((max(n, (int64_t)1) + kSBlock - 1) / kSBlock);
    hipLaunchKernelGGL(bump_gather_kernel, dim3(ng), dim3(kSBlock), 0, st, size, vs, n, sz,
                       (const BumpFlags*)fl);
    if (n > 0) {
        e = device_scan_i64(sz, n, false, partial, nullptr, st, &fl->abort);
        if (e != hipSuccess) return e;
    }
    // the sum of the sizes: the scan's total, or the checked sum (0) when empty
    const int64_t* total = n > 0 ? partial + (scan_workspace_bytes(n) / 8 - 1)
                                 : reinterpret_cast<const int64_t*>(&fl->sum);
    hipLaunchKernelGGL(bump_write_kernel, dim3(nb), dim3(kSBlock), 0, st, begin, n_seg, ks, vs,
                       (const int64_t*)sz, total, n, op_bits, offset_out, peak_out,
                       (const BumpFlags*)fl);
    return hipGetLastError();
}

hipError_t launch_optimal(const int64_t* begin, int64_t n_traces, const int32_t* num_ops,
                          const int64_t* size, const int32_t* first, const int32_t* last,
                          int64_t n_tensors, int64_t* offset_out, int64_t* peak_out,
                          int32_t* status, hipStream_t st) {
    if (n_traces == 0) return hipSuccess;
    hipLaunchKernelGGL(optimal_kernel, dim3((unsigned)n_traces), dim3(kWave), 0, st, begin,
                       num_ops, size, first, last, n_tensors, offset_out, peak_out, status);
    return hipGetLastError();
}

}  // namespace mp
