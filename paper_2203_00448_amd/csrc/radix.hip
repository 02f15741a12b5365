// Stable LSD radix sort of (u64 key, u32 value) pairs, 8-bit digits.
//
// Every digit's device-wide counts come from one reading of the keys; then one
// kernel a digit ranks a tile, publishes the tile's counts and adds up those of
// the tiles before it, so a digit costs one launch (and a sort of p digits p + 2)
// where counting, scanning in three kernels and scattering cost five.  The
// counting kernel also sees which digits are the same in every key and whether
// the keys are in order already: those passes are not made (their launches end
// at once).  Up to 4,096 pairs are sorted by one workgroup in LDS instead, in
// one launch.
//
// Bound by latency up to some millions of pairs: launch, tile load, eight
// ballots an element, one exchange through device memory, scatter.  Bump plans, the
// five kernels a digit -> this: 1 M tensors in op order 140 -> 71 us, in any order
// (two to three digits that differ) 175 -> 152, 4 M 456 -> 412, 16 M 1880 -> 1641; a
// plan of 5,000 tensors has 14 launches of sorts (16 beyond 16,384 pairs) where it had
// 80.
#include "internal.hpp"
#include "mp_device.hpp"

namespace mp {

namespace {

constexpr int kRadixBlock = 1024;
constexpr int kRadixItems = 4;
constexpr int kRadixWaves = kRadixBlock / kWave;
constexpr int64_t kRadixTile = (int64_t)kRadixBlock * kRadixItems;
constexpr int kDigits = 256;
constexpr int kMaxPasses = 8;
// Workgroups that count, one a CU.  Each writes its counts, which the next kernel
// adds up: as atomics on one set of counts they took 0.25 ns each, on eight sets
// too, and fewer workgroups read too slowly (4 M keys that differ in three digits:
// 68 us by 96 workgroups with atomics, 28 us so; a bump plan of 1 M 178 -> 152 us).
constexpr int kCountGrid = 256;
// Up to this many pairs one workgroup counts, in LDS alone: no clearing launch,
// no exchange (58 -> 55 us for live bytes and a bump plan of 6,000 tensors).
constexpr int64_t kCountAlone = 4 * kRadixTile;
// A tile adds up the counts of its group's tiles before it, of its block's groups
// before its own and the sum over all blocks before its own.  The last tile of a
// group publishes the group's counts before it waits for other groups, so only
// blocks (16.8 M pairs) form a chain.  (Groups of 256 tiles in a chain: a pass
// over 4 M pairs 96 -> 60 us with the above, of which 20 are a copy's.)
constexpr int kGroup = 64;       // tiles
constexpr int kBlockGroups = 64; // groups
constexpr int64_t kBlockTiles = (int64_t)kGroup * kBlockGroups;
constexpr uint32_t kPublished = 1u << 31;  // a group counts up to 2^18, a block 2^24
constexpr uint64_t kPublished64 = 1ull << 63;

struct RadixHeader {
    uint32_t ticket[kMaxPasses];  // next tile of each pass
    uint32_t differ[kMaxPasses];  // the pass's digits are not all alike
    uint32_t unordered;           // some key is smaller than the one before it
    uint32_t down[kCountGrid];    // the same, as each counting workgroup saw it
    unsigned long long base[kMaxPasses][kDigits];  // where each digit starts
};

// Published counts, twice (a move clears the other set for the next one): a row
// of 256 for each tile, each whole group and each whole block.
struct RadixRows {
    uint32_t *tile, *group;
    uint64_t* block;
};

constexpr size_t kHeaderBytes = (sizeof(RadixHeader) + 255) / 256 * 256;

__host__ __device__ __forceinline__ size_t rows_bytes(int64_t tiles) {  // of one set
    return (size_t)kDigits * (size_t)((tiles + tiles / kGroup) * 4 + tiles / kBlockTiles * 8);
}

__device__ __forceinline__ RadixRows rows_of(void* ws, int64_t tiles, int set) {
    char* p = static_cast<char*>(ws) + kHeaderBytes + set * rows_bytes(tiles);
    uint64_t* block = reinterpret_cast<uint64_t*>(p);
    uint32_t* group = reinterpret_cast<uint32_t*>(block + tiles / kBlockTiles * kDigits);
    return RadixRows{group + tiles / kGroup * kDigits, group, block};
}

// Each counting workgroup's counts, [passes][kDigits] behind the rows (none up to
// kCountAlone pairs).
__host__ __device__ __forceinline__ size_t counts_at(int64_t tiles) {
    return kHeaderBytes + 2 * rows_bytes(tiles);
}

// The passes that move the pairs, and the one among them that keeps their order.
struct RadixPlan {
    uint32_t exec, copy;
};
__device__ __forceinline__ RadixPlan plan_of(const RadixHeader* h, int passes) {
    RadixPlan r{0, 0};
    if (h->unordered)
        for (int p = 0; p < passes; ++p) r.exec |= h->differ[p] << p;
    // the result has to be in the buffer that `passes` moves end in: an odd
    // number of passes left out is made even by one that only copies
    if ((__popc(r.exec) ^ passes) & 1) {
        r.copy = ~r.exec & (r.exec + 1);  // the first pass left out
        r.exec |= r.copy;
    }
    return r;
}

template <class T>
__device__ __forceinline__ T agent_load(const T* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <class T>
__device__ __forceinline__ void agent_store(T* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void clear_rows(const RadixRows& r, int64_t tile) {
    if (threadIdx.x < kDigits) {
        r.tile[tile * kDigits + threadIdx.x] = 0;
        if (tile % kGroup == kGroup - 1) r.group[tile / kGroup * kDigits + threadIdx.x] = 0;
        if (tile % kBlockTiles == kBlockTiles - 1)
            r.block[tile / kBlockTiles * kDigits + threadIdx.x] = 0;
    }
}

// Where each digit of a pass starts, and whether the pass has work to do, from the
// digit's counts c (lane l of one wave: digits 4 l .. 4 l + 3).
__device__ __forceinline__ void plan_pass(RadixHeader* h, int pass, const uint64_t (&c)[4], int64_t n) {
    const int lane = threadIdx.x & (kWave - 1);
    uint64_t sum = 0;
    bool all = false;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        all |= (int64_t)c[k] == n;
        sum += c[k];
    }
    uint64_t inc = sum;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint64_t y = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += y;
    }
    uint64_t run = inc - sum;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        h->base[pass][4 * lane + k] = run;
        run += c[k];
    }
    const bool same = __ballot(all) != 0;
    if (lane == 0) h->differ[pass] = same ? 0u : 1u;
}

// Counts of every digit; up to kCountAlone pairs one workgroup, which plans the
// passes too.
__global__ __launch_bounds__(kRadixBlock) void radix_hist_kernel(
    const uint64_t* __restrict__ keys, int64_t n, int begin_bit, int passes, RadixHeader* h,
    uint32_t* __restrict__ counts, int64_t tiles, const uint32_t* skip, const int64_t* n_live) {
    __shared__ uint32_t hist[kMaxPasses][kDigits];
    if (skip && *skip) return;
    if (n_live) n = max(min(n, *n_live), (int64_t)0);
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x)
        clear_rows(rows_of(h, tiles, 0), t);  // the first move's
    if (blockIdx.x == 0 && tid < kMaxPasses) h->ticket[tid] = 0;
    const uint64_t mask = passes >= 8 ? ~0ull : ((1ull << (8 * passes)) - 1ull);
    for (int i = tid; i < passes * kDigits; i += kRadixBlock) hist[i / kDigits][i % kDigits] = 0;
    __syncthreads();
    bool down = false;
    for (int64_t base = blockIdx.x * kRadixTile; base < n; base += gridDim.x * kRadixTile) {
        uint64_t key[kRadixItems], ahead[kRadixItems];
#pragma unroll
        for (int k = 0; k < kRadixItems; ++k) {
            const int64_t e = base + k * kRadixBlock + tid;
            key[k] = e < n ? (keys[e] >> begin_bit) & mask : 0ull;
            ahead[k] = e < n && e > 0 ? (keys[e - 1] >> begin_bit) & mask : 0ull;
        }
#pragma unroll
        for (int k = 0; k < kRadixItems; ++k) {
            const bool in = base + k * kRadixBlock + tid < n;
            down |= in && ahead[k] > key[k];
            const uint64_t who = __ballot(in);
            if (!who) continue;
            for (int p = 0; p < passes; ++p) {
                const uint32_t d = (uint32_t)(key[k] >> (8 * p)) & 0xFF;
                // lane 0 holds an element when any lane does; one addition
                // for a digit that is the same over the wave
                if (__ballot(in && d != (uint32_t)__builtin_amdgcn_readfirstlane((int)d)) == 0) {
                    if (lane == 0) atomicAdd(&hist[p][d], (uint32_t)__popcll(who));
                } else if (in) {
                    atomicAdd(&hist[p][d], 1u);
                }
            }
        }
    }
    const bool down_any = __syncthreads_or(down);
    if (gridDim.x > 1) {
        uint32_t* mine = counts + (size_t)blockIdx.x * passes * kDigits;
        for (int i = tid; i < passes * kDigits; i += kRadixBlock)
            mine[i] = hist[i / kDigits][i % kDigits];
        if (tid == 0) h->down[blockIdx.x] = down_any ? 1u : 0u;
        return;
    }
    if (wid < passes) {
        uint64_t c[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) c[k] = hist[wid][4 * lane + k];
        plan_pass(h, wid, c, n);
    }
    if (tid == 0) h->unordered = down_any ? 1u : 0u;
}

// The counting workgroups' counts added up, one workgroup a pass.
__global__ __launch_bounds__(kRadixBlock) void radix_plan_kernel(RadixHeader* h,
                                                                 const uint32_t* __restrict__ counts,
                                                                 int groups, int64_t n,
                                                                 const uint32_t* skip,
                                                                 const int64_t* n_live) {
    constexpr int kSplit = kRadixBlock / kDigits, kBatch = 16;
    __shared__ uint64_t part[kSplit][kDigits];
    if (skip && *skip) return;
    if (n_live) n = max(min(n, *n_live), (int64_t)0);
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int d = tid % kDigits, q = tid / kDigits, pass = blockIdx.x, passes = gridDim.x;
    uint64_t sum = 0;
    for (int g = q; g < groups; g += kSplit * kBatch) {
        uint32_t x[kBatch];
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const int u = g + i * kSplit;
            x[i] = u < groups ? counts[((size_t)u * passes + pass) * kDigits + d] : 0u;
        }
#pragma unroll
        for (int i = 0; i < kBatch; ++i) sum += x[i];
    }
    part[q][d] = sum;
    const bool down = __syncthreads_or(tid < groups && h->down[tid]);
    if (tid < kWave) {
        uint64_t c[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            c[k] = 0;
#pragma unroll
            for (int i = 0; i < kSplit; ++i) c[k] += part[i][4 * lane + k];
        }
        plan_pass(h, pass, c, n);
    }
    if (pass == 0 && tid == 0) h->unordered = down ? 1u : 0u;
}

__global__ __launch_bounds__(kRadixBlock) void radix_pass_kernel(
    uint64_t* k0, uint32_t* v0, uint64_t* k1, uint32_t* v1, int64_t n, int begin_bit, int pass,
    int passes, RadixHeader* h, int64_t tiles, const uint32_t* skip, const int64_t* n_live) {
    __shared__ uint32_t wave_cnt[kRadixWaves][kDigits];
    __shared__ uint32_t part[kRadixBlock / kDigits][kDigits];
    __shared__ int64_t start[kDigits];
    __shared__ uint32_t my_tile;
    if (skip && *skip) return;
    const RadixPlan plan = plan_of(h, passes);
    const uint32_t exec = plan.exec;
    if (!((exec >> pass) & 1u)) return;
    if (n_live) n = min(n, *n_live);
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    const int moves = __popc(exec & ((1u << pass) - 1u));  // before this one
    const uint64_t* kin = (moves & 1) ? k1 : k0;
    const uint32_t* vin = (moves & 1) ? v1 : v0;
    uint64_t* kout = (moves & 1) ? k0 : k1;
    uint32_t* vout = (moves & 1) ? v0 : v1;
    const RadixRows pub = rows_of(h, tiles, moves & 1);
    // Tiles in the order their workgroups started: a workgroup waits only for
    // earlier tiles, whose workgroups run already and wait for none after them.
    if (tid == 0) my_tile = atomicAdd(&h->ticket[pass], 1u);
    __syncthreads();
    const int64_t tile = my_tile, base = tile * kRadixTile;
    clear_rows(rows_of(h, tiles, (moves + 1) & 1), tile);  // the next move's
    if (base >= n) return;
    uint64_t key[kRadixItems];
    uint32_t val[kRadixItems], rank[kRadixItems];
    // a wave takes kRadixItems * 64 consecutive elements
#pragma unroll
    for (int k = 0; k < kRadixItems; ++k) {
        const int64_t e = base + (wid * kRadixItems + k) * kWave + lane;
        key[k] = e < n ? kin[e] : 0ull;
        val[k] = (e < n && vin) ? vin[e] : 0u;
    }
    if ((plan.copy >> pass) & 1u) {
#pragma unroll
        for (int k = 0; k < kRadixItems; ++k) {
            const int64_t e = base + (wid * kRadixItems + k) * kWave + lane;
            if (e < n) {
                kout[e] = key[k];
                if (vout) vout[e] = val[k];
            }
        }
        return;
    }
    const int shift = begin_bit + 8 * pass;
    for (int i = lane; i < kDigits; i += kWave) wave_cnt[wid][i] = 0;
    const uint64_t lower = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int k = 0; k < kRadixItems; ++k) {
        const bool in = base + (wid * kRadixItems + k) * kWave + lane < n;
        const uint32_t d = (uint32_t)(key[k] >> shift) & 0xFF;
        uint64_t same = __ballot(in);
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
            const uint64_t ones = __ballot((d >> bit) & 1u);
            same &= ((d >> bit) & 1u) ? ones : ~ones;
        }
        const uint32_t before = wave_cnt[wid][d];
        rank[k] = before + (uint32_t)__popcll(same & lower);
        __builtin_amdgcn_wave_barrier();  // every lane has read
        if (in && (same & lower) == 0) wave_cnt[wid][d] = before + (uint32_t)__popcll(same);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    uint32_t mine = 0;
    if (tid < kDigits) {
#pragma unroll
        for (int w = 0; w < kRadixWaves; ++w) {
            const uint32_t c = wave_cnt[w][tid];
            wave_cnt[w][tid] = mine;
            mine += c;
        }
        agent_store(&pub.tile[tile * kDigits + tid], kPublished | mine);
    }
    // the digit's count in all earlier tiles: four threads a digit, eight rows of
    // loads in flight for each
    constexpr int kSplit = kRadixBlock / kDigits, kBatch = 8;
    const int d = tid % kDigits, q = tid / kDigits;
    auto add_rows = [&](const uint32_t* rows, int64_t from, int64_t to) {
        uint32_t sum = 0;
        for (int64_t t = from + q; t < to; t += kSplit * kBatch) {
            uint32_t x[kBatch];
            bool all;
            do {
                all = true;
#pragma unroll
                for (int i = 0; i < kBatch; ++i) {
                    const int64_t u = t + i * kSplit;
                    x[i] = u < to ? agent_load(&rows[u * kDigits + d]) : kPublished;
                    all &= (x[i] & kPublished) != 0;
                }
            } while (!all);
#pragma unroll
            for (int i = 0; i < kBatch; ++i) sum += x[i] & ~kPublished;
        }
        return sum;
    };
    const int64_t group = tile / kGroup, block = tile / kBlockTiles;
    uint32_t sum = add_rows(pub.tile, group * kGroup, tile);
    if (tile % kGroup == kGroup - 1) {
        part[q][d] = sum;
        __syncthreads();
        if (tid < kDigits) {
            uint32_t all = mine;
#pragma unroll
            for (int i = 0; i < kSplit; ++i) all += part[i][tid];
            agent_store(&pub.group[group * kDigits + tid], kPublished | all);
        }
        __syncthreads();
    }
    sum += add_rows(pub.group, block * kBlockGroups, group);
    part[q][d] = sum;
    __syncthreads();
    if (tid < kDigits) {
        uint64_t before = 0;
#pragma unroll
        for (int i = 0; i < kSplit; ++i) before += part[i][tid];
        if (block > 0) {
            uint64_t x;
            do x = agent_load(&pub.block[(block - 1) * kDigits + tid]);
            while (!(x & kPublished64));
            before += x & ~kPublished64;
        }
        if (tile % kBlockTiles == kBlockTiles - 1)
            agent_store(&pub.block[block * kDigits + tid], kPublished64 | (before + mine));
        start[tid] = (int64_t)(h->base[pass][tid] + before);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kRadixItems; ++k) {
        if (base + (wid * kRadixItems + k) * kWave + lane >= n) continue;
        const uint32_t d = (uint32_t)(key[k] >> shift) & 0xFF;
        const int64_t pos = start[d] + wave_cnt[wid][d] + rank[k];
        kout[pos] = key[k];
        if (vout) vout[pos] = val[k];
    }
}

// One workgroup sorts up to kSmallSort pairs in LDS with a bitonic network
// over (the key's digit bits, input position).  Position breaks every tie, so
// the permutation is the one the stable digit passes produce; the pairs are
// written to the buffer those passes would end in (possibly the input: every
// input is in LDS before anything is written).  Elements [m, P) are padding
// that sorts last (all-ones key, position >= m).
constexpr int kSmallSort = 4096;
constexpr int kSmallSortThreads = 1024;

__global__ __launch_bounds__(kSmallSortThreads) void small_sort_kernel(
    const uint64_t* kin, const uint32_t* vin, uint64_t* kout, uint32_t* vout, int64_t n,
    int shift, uint64_t mask, int P, const uint32_t* skip, const int64_t* n_live) {
    __shared__ uint64_t sk[kSmallSort];  // full keys, moved by the network
    __shared__ uint16_t si[kSmallSort];  // input positions, moved with them
    __shared__ uint32_t sv[kSmallSort];  // values, by input position
    if (skip && *skip) return;
    int64_t m = n;
    if (n_live) m = min(m, *n_live);
    if (m < 0) m = 0;
    const int T = (int)blockDim.x, tid = (int)threadIdx.x;
    for (int i = tid; i < P; i += T) {
        const bool in = i < m;
        sk[i] = in ? kin[i] : ~0ull;
        si[i] = (uint16_t)i;
        if (vin) sv[i] = in ? vin[i] : 0u;
    }
    __syncthreads();
    for (int k = 2; k <= P; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int t = tid; t < P / 2; t += T) {
                const int a = 2 * t - (t & (j - 1)), b = a + j;  // bit j of a clear
                const uint64_t ka = sk[a], kb = sk[b];
                const uint16_t ia = si[a], ib = si[b];
                const uint64_t da = (ka >> shift) & mask, db = (kb >> shift) & mask;
                const bool gt = da > db || (da == db && ia > ib);
                if (gt == ((a & k) == 0)) {  // ascending where bit k of a is clear
                    sk[a] = kb;
                    sk[b] = ka;
                    si[a] = ib;
                    si[b] = ia;
                }
            }
            __syncthreads();
        }
    }
    for (int r = tid; r < m; r += T) {
        kout[r] = sk[r];
        if (vout) vout[r] = sv[si[r]];
    }
}

}  // namespace

size_t radix_workspace_bytes(int64_t n) {
    if (n <= kSmallSort) return 256;
    const int64_t tiles = (n + kRadixTile - 1) / kRadixTile;
    const int64_t groups = n <= kCountAlone ? 0 : min(tiles, (int64_t)kCountGrid);
    return counts_at(tiles) + (size_t)groups * kMaxPasses * kDigits * sizeof(uint32_t);
}

// Sorts n pairs by bits [begin_bit, end_bit) of the key (in whole 8-bit
// digits), stably.  *in_alt tells where the result is: (k1, v1) for an odd
// number of digits.  v0/v1 may be null (keys only).  `ws` has radix_workspace_bytes(n).
// A non-null `skip` word that is nonzero at run time turns every kernel into
// a no-op (the buffers then stay as they were).  A non-null `n_live` is a
// device count read at run time: only the first min(n, *n_live) pairs are
// sorted (n then only bounds the launch).
hipError_t radix_sort_pairs(uint64_t* k0, uint32_t* v0, uint64_t* k1, uint32_t* v1, int64_t n,
                            int begin_bit, int end_bit, void* ws, bool* in_alt, hipStream_t st,
                            const uint32_t* skip, const int64_t* n_live) {
    *in_alt = false;
    if (n <= 1 || end_bit <= begin_bit) return hipSuccess;
    if (n <= kSmallSort) {
        const int passes = (end_bit - begin_bit + 7) / 8;
        const int width = min(8 * passes, 64 - begin_bit);  // the bits the passes order by
        const uint64_t mask = width >= 64 ? ~0ull : ((1ull << width) - 1ull);
        int P = 2;
        while (P < n) P <<= 1;
        const int threads = max(kWave, min(kSmallSortThreads, P / 2));
        const bool alt = (passes & 1) != 0;
        hipLaunchKernelGGL(small_sort_kernel, dim3(1), dim3(threads), 0, st, k0, v0,
                           alt ? k1 : k0, alt ? v1 : v0, n, begin_bit, mask, P, skip, n_live);
        *in_alt = alt;
        return hipGetLastError();
    }
    const int64_t tiles = (n + kRadixTile - 1) / kRadixTile;
    const int passes = (end_bit - begin_bit + 7) / 8;
    if (tiles > INT32_MAX || passes > kMaxPasses) return hipErrorInvalidValue;
    RadixHeader* h = static_cast<RadixHeader*>(ws);
    const int64_t count_grid = n <= kCountAlone ? 1 : min(tiles, (int64_t)kCountGrid);
    uint32_t* counts = reinterpret_cast<uint32_t*>(static_cast<char*>(ws) + counts_at(tiles));
    hipLaunchKernelGGL(radix_hist_kernel, dim3((unsigned)count_grid),
                       dim3(kRadixBlock), 0, st,
                       (const uint64_t*)k0, n, begin_bit, passes, h, counts, tiles, skip, n_live);
    if (count_grid > 1)
        hipLaunchKernelGGL(radix_plan_kernel, dim3((unsigned)passes), dim3(kRadixBlock), 0, st, h,
                           (const uint32_t*)counts, (int)count_grid, n, skip, n_live);
    for (int p = 0; p < passes; ++p)
        hipLaunchKernelGGL(radix_pass_kernel, dim3((unsigned)tiles), dim3(kRadixBlock), 0, st, k0,
                           v0, k1, v1, n, begin_bit, p, passes, h, tiles, skip, n_live);
    *in_alt = (passes & 1) != 0;
    return hipGetLastError();
}

}  // namespace mp
