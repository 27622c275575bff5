// Block path: symbolic factorisation by 64-row blocks of bit masks.
//
// A block holds 64 consecutive rows; bit r of a 64-bit mask stands for its row
// r. For every column v the block keeps one mask: the rows whose structure
// (row of L+U) contains v. By the fill-path theorem (Background) the structure
// of a row s is the smallest set that contains the row's own entries and, with
// every k < s in it, the entries of U(k,:) (split a fill path at its largest
// intermediate vertex k: s -> k puts k into L(s,:), and the rest of the path
// puts its end into U(k,:)). So a block takes its rows' entries, then merges
// the finished U rows of the earlier blocks that its masks name, 64 rows at
// once, and finally its own rows among each other. The per-source traversal
// (k_traverse) walks every vertex reachable from every source instead: on the
// 64^3 27-point stencil 51 G edge visits, where the block path makes 1.8e5 block
// merges of 2.5e6 64-column tiles: 4.0 ms instead of 221 (1000^2 9-point stencil:
// 2.8 instead of 211 ms; 512 batch members: 2.3 instead of 90 ms).
//
// What bounds it is the chain of blocks that wait for one another, not
// throughput, and four things keep that chain short:
//   * two publications per block. The rows that depend on no earlier block
//     (whole small subtrees and the first rows of a larger one) are finished
//     and published at once, before the block waits for anything. With one
//     publication a nested-dissection order would run almost serially: a block
//     that holds the end of one subtree and the start of the next would make
//     the second wait for the first (modelled on the 1000^2 9-point stencil:
//     a chain of 102 ms with one publication, 1.8 ms with two).
//   * pruning (Eisenstat and Liu's symmetric pruning). Where U(a,k) and L(k,a)
//     are both nonzero, every later row with a in its structure has k too, and
//     U(k,:) holds the rest of U(a,:): of row a only the entries up to k are
//     needed. kmatch[a] is the smallest such k found so far.
//   * several wavefronts per block that merge pending blocks, and the tiles of a
//     long list, side by side. Merging is monotone, so a block merged too early
//     is merged again when bits of it arrive later.
//   * few round trips from one block's publication to the next one's: the reader
//     polls a 128-byte header that carries its own state, the rows and the first
//     tile ids; reductions go by data-parallel moves, the elimination inside a
//     block by table lookups, and barriers between wavefronts wait for LDS only.
//     (Per block of a separator, from the last dependency's publication to its
//     own: 17.5 us with flags, shuffles and a branching elimination loop, 5.5 us.)
//
// Blocks are taken from a counter in an order in which every block comes after
// the ones it can depend on (ascending inside a matrix), so a block waits only
// for blocks that resident workgroups have already taken, and the first
// unfinished one waits for nothing: the launch always drains. Every wait also
// ends on the abort word and after kSpinLimit polls. A launch that is asked to yield
// takes no further block and finishes those it has taken (they wait for one another
// only, as before); the next launch goes on at the counter.
//
// Data that crosses workgroups (masks, columns, headers, kmatch, flags) is
// written and read with device-scope atomics, which reach memory past the
// XCD's L2; the writer waits for its stores (s_waitcnt) before the flag.
#include <algorithm>
#include "gsofa_internal.h"
#include "gsofa.h"

namespace gsofa {

typedef unsigned long long u64;

namespace {

constexpr int kThreads = 256;         // threads of the kernels after the factorisation
constexpr int kRangeTiles = 1024;     // column tiles (64 columns) listed at a time
constexpr uint32_t kSpinLimit = 1u << 22;
constexpr int32_t kNoMatch = 0x7FFFFFFF;
constexpr int kHeadTiles = 20;        // tile ids in a list's header
// Tiles of a shared merge that a wavefront takes, and of a list that it writes, at
// a time: their round trips overlap (64^3 27-point: 4.14 ms with four, 4.00 with six
// or eight; 1000^2 9-point 3.03 and 2.96; 512 batch members 2.35, with six 2.47)
constexpr int kShare = 8;
constexpr int kWrite = 8;

// word of the header that holds tiles i and i + 1 (i even), and the other way
__device__ __forceinline__ int head_word(int i) { return i < 6 ? 4 + (i >> 1) : 8 + ((i - 6) >> 1); }
__device__ __forceinline__ int head_tile(int w) { return w < 8 ? 2 * (w - 4) : 6 + 2 * (w - 8); }

__device__ __forceinline__ int lane() { return (int)(threadIdx.x & 63); }
__device__ __forceinline__ int rfl(int v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ uint32_t below_count(u64 m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ __forceinline__ u64 readlane64(u64 v, int l) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l);
    return ((u64)hi << 32) | lo;
}

// Scans and reductions over the wavefront by data-parallel-primitive moves
// (six vector instructions) rather than shuffles through LDS, whose latency six
// times over a chain of blocks pays for.
#define GSOFA_DPP_STEP(ctrl, rmask, id, op)                                                          \
    {                                                                                                \
        const int t = __builtin_amdgcn_update_dpp(id, v, ctrl, rmask, 0xf, false);                   \
        v = op(v, t);                                                                                \
    }
#define GSOFA_DPP_SCAN(id, op)              \
    GSOFA_DPP_STEP(0x111, 0xf, id, op) /* row_shr:1 */ \
    GSOFA_DPP_STEP(0x112, 0xf, id, op) /* row_shr:2 */ \
    GSOFA_DPP_STEP(0x114, 0xf, id, op) /* row_shr:4 */ \
    GSOFA_DPP_STEP(0x118, 0xf, id, op) /* row_shr:8 */ \
    GSOFA_DPP_STEP(0x142, 0xa, id, op) /* row_bcast:15 */ \
    GSOFA_DPP_STEP(0x143, 0xc, id, op) /* row_bcast:31 */

__device__ __forceinline__ int op_add(int a, int b) { return a + b; }
__device__ __forceinline__ int op_or(int a, int b) { return a | b; }
__device__ __forceinline__ int op_max(int a, int b) { return a > b ? a : b; }
__device__ __forceinline__ int op_min(int a, int b) { return a < b ? a : b; }

__device__ __forceinline__ int incl_scan(int v) {
    GSOFA_DPP_SCAN(0, op_add)
    return v;
}
// every lane gets the result
__device__ __forceinline__ int sum32(int v) {
    GSOFA_DPP_SCAN(0, op_add)
    return __builtin_amdgcn_readlane(v, 63);
}
__device__ __forceinline__ int max64(int v) {
    GSOFA_DPP_SCAN((int)0x80000000, op_max)
    return __builtin_amdgcn_readlane(v, 63);
}
// of lanes 0 to 15
__device__ __forceinline__ int min16(int v) {
    GSOFA_DPP_STEP(0x111, 0xf, 0x7FFFFFFF, op_min)
    GSOFA_DPP_STEP(0x112, 0xf, 0x7FFFFFFF, op_min)
    GSOFA_DPP_STEP(0x114, 0xf, 0x7FFFFFFF, op_min)
    GSOFA_DPP_STEP(0x118, 0xf, 0x7FFFFFFF, op_min)
    return __builtin_amdgcn_readlane(v, 15);
}
__device__ __forceinline__ int or32(int v) {
    GSOFA_DPP_SCAN(0, op_or)
    return __builtin_amdgcn_readlane(v, 63);
}
__device__ __forceinline__ u64 or64(u64 v) {
    return (u64)(uint32_t)or32((int)(uint32_t)v) | ((u64)(uint32_t)or32((int)(uint32_t)(v >> 32)) << 32);
}

__device__ __forceinline__ u64 sum64(u64 v) {
#pragma unroll
    for (int d = 32; d; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

// device scope: data published to other workgroups
template <typename T>
__device__ __forceinline__ T ld_dev(const T* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void st_dev(T* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// workgroup scope: a block's own column masks
__device__ __forceinline__ u64 ld_wg(const u64* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// LDS words that other wavefronts change
template <typename T>
__device__ __forceinline__ T ld_lds(const T* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ u64 or_wg(u64* p, u64 v) {
    return __hip_atomic_fetch_or(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Order this wavefront's earlier LDS accesses before its later ones: the LDS
// serves a wavefront's accesses in order, so only the compiler is told. (A fence
// of workgroup scope also waits for every global store to be acknowledged.)
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
// Barrier of the workgroup for what its wavefronts pass on in LDS; global stores
// may still be on their way.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// this wavefront's device-scope stores have reached memory
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ __forceinline__ u64 above(int k) { return k < 63 ? ~0ull << (k + 1) : 0ull; }
__device__ __forceinline__ u64 below(int k) { return (1ull << k) - 1ull; }

// Lane b: the OR of the lanes' words w[a] over the bits a of set[b], through
// sixteen 16-entry tables in LDS (the OR of every subset of four words): the
// lookups of a table touch 16 consecutive words, so they never conflict.
// Following the up to 63 bits of a set one by one costs several times as much.
// xs: 64 words, tab: 256 words of the wavefront's own.
__device__ __forceinline__ u64 lane_or(u64 w, u64 set, u64* xs, u64* tab) {
    const int ln = lane();
    const u64 m0 = 0ull - (u64)(ln & 1), m1 = 0ull - (u64)((ln >> 1) & 1), m2 = 0ull - (u64)((ln >> 2) & 1),
              m3 = 0ull - (u64)((ln >> 3) & 1);
    wave_sync();
    xs[ln] = w;
    wave_sync();
    u64 t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const u64* q = &xs[((ln >> 4) + 4 * i) * 4];  // entry ln & 15 of nibble (ln >> 4) + 4 i
        t[i] = (q[0] & m0) | (q[1] & m1) | (q[2] & m2) | (q[3] & m3);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) tab[ln + 64 * i] = t[i];
    wave_sync();
    u64 y = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) y |= tab[i * 16 + (int)((set >> (4 * i)) & 15ull)];
    return y;
}

__device__ __forceinline__ uint32_t lo32(u64 v) { return (uint32_t)v; }
__device__ __forceinline__ uint32_t hi32(u64 v) { return (uint32_t)(v >> 32); }
__device__ __forceinline__ uint32_t rl32(uint32_t v, int l) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, l);
}
// all ones where bit k of v is set
__device__ __forceinline__ uint32_t bit_mask(uint32_t v, int k) { return (uint32_t)__builtin_amdgcn_sbfe((int)v, k, 1); }

// One block's rows among each other. x: lane b's word is the mask of the
// block's own column b. Row k's pattern right of k goes to every row r > k that
// holds k, for the rows k of S in ascending order; with `narrow` a row that
// depends on a row outside S leaves S (S then ends as the rows finished
// without any earlier block). The 64 steps depend on one another; a step is six
// instructions without a branch (broadcast column k, spread bit k of the own
// word, and-or) and takes 40 ns all the same, the way of a word through the
// scalar registers (two rows a step, the second one's column brought up to date
// there, took longer).
template <bool narrow>
__device__ __forceinline__ void eliminate(u64& x, u64& S) {
    const u64 up = below(lane());
    const uint32_t ulo = lo32(up), uhi = hi32(up);
    uint32_t lo = lo32(x), hi = hi32(x);
#pragma unroll 8
    for (int k = 0; k < 32; ++k) {
        uint32_t Ll = rl32(lo, k) & (uint32_t)(0xFFFFFFFEull << k), Lh = rl32(hi, k);
        if (narrow) {
            const uint32_t in = (uint32_t)0 - (uint32_t)((S >> k) & 1ull);
            S &= ~(((u64)(Lh & ~in) << 32) | (Ll & ~in));
            Ll &= in;
            Lh &= in;
        }
        const uint32_t t = bit_mask(lo & ulo, k);
        lo |= t & Ll;
        hi |= t & Lh;
    }
#pragma unroll 8
    for (int k = 32; k < 64; ++k) {
        uint32_t Lh = rl32(hi, k) & (uint32_t)(0xFFFFFFFEull << (k - 32));
        if (narrow) {
            const uint32_t in = (uint32_t)0 - (uint32_t)((S >> k) & 1ull);
            S &= ~((u64)(Lh & ~in) << 32);
            Lh &= in;
        }
        hi |= bit_mask(hi & uhi, k - 32) & Lh;
    }
    x = ((u64)hi << 32) | lo;
}

// The same for all rows at once: every pass adds to each column b the rows that
// reach it through any k < b of S (the rule of a step above, for the entries
// known so far), until a pass adds nothing. Blocks deep in a separator are
// nearly full when their turn comes and need two or three passes of 0.25 us,
// those of a band five or six; one that needs more than kPasses goes step by
// step. With `narrow`, S then loses the rows that depend on one outside it.
template <bool narrow>
__device__ __forceinline__ void eliminate_all(u64& x, u64& S, u64* xs, u64* tab) {
    constexpr int kPasses = 8;
    const int ln = lane();
    const u64 up = below(ln) & S, dn = above(ln);
    int i = 0;
    for (; i < kPasses; ++i) {
        const u64 y = x | lane_or(x & dn, x & up, xs, tab);
        const bool more = y != x;
        x = y;
        if (__ballot(more) == 0ull) break;
    }
    if (i == kPasses) {
        eliminate<narrow>(x, S);
    } else if (narrow) {
        for (;;) {
            const u64 T = S & ~or64((S >> ln) & 1ull ? 0ull : x & dn);
            if (T == S) break;
            S = T;
        }
    }
}

// Transitive closure of a relation on the block's rows: lane k holds the rows
// that k leads to. A pass doubles the lengths of the chains covered, so there are
// at most seven; a full block is closed already and needs one.
__device__ __forceinline__ u64 closure(u64 c, u64* xs, u64* tab) {
    for (;;) {
        const u64 d = c | lane_or(c, c, xs, tab);
        const bool more = d != c;
        c = d;
        if (__ballot(more) == 0ull) return c;
    }
}

// Lane k: the first b with U(k,b) and L(b,k) both nonzero, or -1, for the rows
// of S of an eliminated block (x, and all its words in xw). In a full block that
// is the first row below, so the candidates are tried one by one.
__device__ __forceinline__ int first_match(u64 x, u64 S, const u64* xw) {
    const int ln = lane();
    int match = -1;
    u64 cand = ((S >> ln) & 1ull) ? x & above(ln) : 0ull;
    while (cand != 0ull) {
        const int b = __builtin_ctzll(cand);
        cand &= cand - 1ull;
        if ((xw[b] >> ln) & 1ull) {
            match = b;
            cand = 0;
        }
    }
    return match;
}

}  // namespace

// ------------------------------------------------------------- factorisation

// One workgroup of W wavefronts per block at a time.
//
// A block's result is a list of tiles, 64 columns each: tile ids and 64 masks
// per tile, U beyond the block (read by later blocks) and L before it. Whole
// tiles need no counting and no prefix sums before they are written, are read
// as 512 consecutive bytes, and hold about half set columns on the stencils.
template <int W>
__global__ __launch_bounds__(64 * W, 4) void k_bm_factor(BlockArgs a) {
    constexpr int kTasks = 4;
    extern __shared__ u64 s_bits[];  // five bitmaps: touched column tiles, blocks to merge
    __shared__ __attribute__((aligned(16))) u64 s_xs[W][64];
    __shared__ u64 s_tab[W][256];
    __shared__ u64 s_C[64], s_x[64];
    __shared__ uint16_t s_tile[kRangeTiles];
    __shared__ int32_t s_rp[65];
    // merges of long lists, shared by the wavefronts: the rows' masks, the list,
    // (tiles << 32 | next tile), tiles done, owned
    __shared__ u64 s_ty[kTasks][64];
    __shared__ u64 s_toff[kTasks], s_tuse[kTasks], s_topen[kTasks];
    __shared__ int32_t s_tblk[kTasks];
    __shared__ u64 s_tnext[kTasks];
    __shared__ int s_tdone[kTasks], s_town[kTasks], s_tstep[kTasks];
    __shared__ u64 s_ext, s_S, s_con, s_off, s_arena, s_arena_end;
    __shared__ int s_item, s_active, s_wait, s_poll, s_stop, s_ntile, s_total;

    const int tid = threadIdx.x, ln = lane(), wv = rfl(tid >> 6);
    u64* X = a.x + (int64_t)blockIdx.x * a.x_stride;
    const int nw = a.bit_words;
    u64* touch = s_bits;
    u64* pend = s_bits + nw;       // blocks to merge, not looked at yet,
    u64* ready = s_bits + 2 * nw;  // known to be published,
    u64* wait1 = s_bits + 3 * nw;  // found unpublished,
    u64* wait2 = s_bits + 4 * nw;  // without their second publication
    u64* xs = s_xs[wv];
    u64* tab = s_tab[wv];
    if (tid == 0) s_arena = s_arena_end = 0;
    if (tid < kTasks) {
        s_tnext[tid] = 0;
        s_town[tid] = 0;
    }

    for (;;) {
        if (tid == 0) {
            const uint32_t asked = a.yield ? __hip_atomic_load(a.yield, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) : 0u;
            s_stop = ld_dev(&a.ctl[kBmAbort]) != 0u;
            s_item = asked ? a.nblocks : (int)atomicAdd(&a.ctl[kBmNext], 1u);
            s_ext = 0;
            s_active = 0;
            s_poll = 0;
            s_wait = 0;
        }
        for (int i = tid; i < 5 * nw; i += 64 * W) s_bits[i] = 0ull;
        __syncthreads();
        const int item = s_item;
        if (item >= a.nblocks || s_stop) break;
        const int32_t gb = a.items ? a.items[item] : item;
        const int32_t jb = a.blk_job ? a.blk_job[gb] : 0;
        const Job* J = &a.jobs[jb];
        const int32_t n = J->n;
        const int32_t b0 = (int32_t)J->item_base;  // first block of the matrix
        const int32_t g = gb - b0;
        const int32_t nr = min(64, n - 64 * g);
        const u64 rows = nr == 64 ? ~0ull : (1ull << nr) - 1ull;
        const int32_t* rp = J->row_ptr + 64 * (int64_t)g;
        const int32_t* ci = J->col_idx;
        const int32_t ntiles = (n + 63) >> 6;
        if (tid <= nr) s_rp[tid] = rp[tid];
        __syncthreads();

        // ---- the rows' own entries
        u64 ext = 0;
        bool dup = false;
        int ndiag = 0;
        // (unsigned: a step beyond up to 2^31 - 1 entries still compares right)
        const uint32_t e1 = (uint32_t)s_rp[nr];
        for (uint32_t e = (uint32_t)s_rp[0] + tid; e < e1; e += 64 * W) {
            const int32_t w = ci[e];
            int lo = 0, hi = nr - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if ((uint32_t)s_rp[mid] <= e) lo = mid;
                else hi = mid - 1;
            }
            const u64 bit = 1ull << lo;
            const int32_t t = w >> 6;
            if (or_wg(&X[w], bit) & bit) dup = true;
            if (w == 64 * g + lo) ++ndiag;
            if (!((touch[t >> 6] >> (t & 63)) & 1ull)) atomicOr(&touch[t >> 6], 1ull << (t & 63));
            if (t < g) {
                ext |= bit;
                if (!((pend[t >> 6] >> (t & 63)) & 1ull)) atomicOr(&pend[t >> 6], 1ull << (t & 63));
            }
        }
        ext = or64(ext);
        const u64 dups = __ballot(dup);
        const u64 nd = (u64)sum32(ndiag);
        if (ln == 0) {
            if (ext) atomicOr(&s_ext, ext);
            if (dups) atomicOr(&a.jstats[jb].err, kErrDuplicate);
            if (nd) atomicAdd(&a.jstats[jb].diag, nd);
        }
        __syncthreads();
        if (tid < nr) or_wg(&X[64 * (int64_t)g + tid], 1ull << tid);
        if (tid == 0) atomicOr(&touch[g >> 6], 1ull << (g & 63));
        __syncthreads();

        // words of the touched tiles in [lo, hi)
        auto touched = [&](int wi, int lo, int hi) -> u64 {
            if (wi >= nw) return 0ull;
            u64 w = touch[wi];
            const int t0 = wi * 64;
            if (t0 < lo) w &= lo - t0 >= 64 ? 0ull : ~0ull << (lo - t0);
            if (t0 + 64 > hi) w &= hi - t0 <= 0 ? 0ull : hi - t0 >= 64 ? ~0ull : (1ull << (hi - t0)) - 1ull;
            return w;
        };
        // Lists the touched tiles of [lo, hi) (kRangeTiles ids at a time), takes
        // room in the pool and writes their ids and the bits `keep` of their
        // masks, ascending; the block's closures s_C are applied first where S is
        // not empty (rows of S pass their pattern on), and the masks cleared
        // behind a `last` list. s_off, s_total: where the list is. Unless
        // state is 0 the list is published as (part, state): the header, then the
        // flag behind all stores.
        auto write_list = [&](int lo, int hi, u64 keep, u64 S, bool last, int part, uint32_t state) -> bool {
            const int R0 = lo / kRangeTiles, R1 = hi > lo ? (hi - 1) / kRangeTiles : R0 - 1;
            u64* head = a.head + (int64_t)gb * kBmHeadWords + part * (kBmHeadWords / 2);
            // Header of a published list, one word per lane: the rows it covers, the
            // rows whose entries beyond the block others need, where the tiles
            // are, how many, and the ids of the first kHeadTiles (n of the list's
            // first range). Words 7 and 15 stay 0 until everything is stored (one per
            // 64-byte half of the line, so that a reader's two copies seldom differ).
            auto header = [&](int n, int t0) {
                wave_sync();
                n = min(n, kHeadTiles);
                if (ln < 16 && (ln & 7) != 7) {
                    u64 v;
                    if (ln == 0) v = keep;
                    else if (ln == 1) v = s_con;
                    else if (ln == 2) v = s_off;
                    else if (ln == 3) v = (u64)s_total | ((u64)n << 32);
                    else {
                        const int i = head_tile(ln);
                        v = (u64)(uint32_t)(i < n ? t0 + s_tile[i] : kNoMatch) |
                            ((u64)(uint32_t)(i + 1 < n ? t0 + s_tile[i + 1] : kNoMatch) << 32);
                    }
                    st_dev(&head[ln], v);
                }
            };
            if (wv == 0) {
                int c = 0;
                for (int wi = lo / 64 + ln; wi * 64 < hi; wi += 64) c += __popcll(touched(wi, lo, hi));
                const int total = sum32(c);
                if (ln == 0) {
                    s_total = total;
                    // room from the workgroup's own stretch of the pool, 64 tiles at a time
                    if (s_arena + (u64)total > s_arena_end) {
                        const u64 take = (u64)max(total, 64);
                        s_arena = atomicAdd(a.pool_tail, take);
                        s_arena_end = s_arena + take;
                        if (s_arena_end > (u64)a.pool_cap) {
                            s_stop = 1;
                            st_dev(&a.ctl[kBmAbort], (uint32_t)kBmOverflow);
                        }
                    }
                    s_off = s_arena;
                    s_arena += (u64)total;
                }
            }
            int64_t base = 0;
            for (int R = R0; R <= R1; ++R) {
                if (wv == 0) {
                    const u64 w0 = ln < kRangeTiles / 64 ? touched(R * (kRangeTiles / 64) + ln, lo, hi) : 0ull;
                    const int c = __popcll(w0);
                    const int inc = incl_scan(c);
                    int o = inc - c;
                    for (u64 w = w0; w; w &= w - 1ull) s_tile[o++] = (uint16_t)(ln * 64 + __builtin_ctzll(w));
                    if (ln == 63) s_ntile = inc;
                    if (state && R == R0) header(__builtin_amdgcn_readlane(inc, 63), R * kRangeTiles);
                }
                lds_barrier();
                if (s_stop) return false;
                const int nt = s_ntile;
                // several tiles of a wavefront at once: their round trips overlap
                for (int i0 = wv; i0 < nt; i0 += kWrite * W) {
                    int32_t t[kWrite];
                    u64 m[kWrite], m0[kWrite];
#pragma unroll
                    for (int j = 0; j < kWrite; ++j) {
                        m[j] = 0;
                        if (i0 + j * W < nt) {
                            t[j] = R * kRangeTiles + s_tile[i0 + j * W];
                            m[j] = ld_wg(&X[64 * (int64_t)t[j] + ln]);
                        }
                        m0[j] = m[j];
                    }
#pragma unroll
                    for (int j = 0; j < kWrite; ++j) {
                        if (i0 + j * W >= nt) break;
                        for (u64 q = m[j] & S; q;) {
                            const int k = __builtin_ctzll(q);
                            const u64 ck = s_C[k];
                            m[j] |= ck;
                            q &= ~(ck | (1ull << k));
                        }
                        u64* xp = &X[64 * (int64_t)t[j] + ln];
                        if (last) {
                            if (m0[j]) *xp = 0ull;
                        } else if (m[j] != m0[j]) {
                            *xp = m[j];
                        }
                        const int64_t q = (int64_t)s_off + base + i0 + j * W;
                        if (state) {
                            if (ln == 0) st_dev(&a.tids[q], t[j]);
                            st_dev(&a.masks[64 * q + ln], m[j] & keep);
                        } else {
                            a.masks[64 * q + ln] = m[j] & keep;
                            if (ln == 0) {
                                a.tids[q] = t[j];
                                a.slot[q] = atomicAdd(&a.tcount[b0 + t[j]], 1);
                            }
                        }
                    }
                }
                base += nt;
                if (R < R1) lds_barrier();
            }
            if (R0 > R1) {
                if (state && wv == 0) header(0, 0);
                lds_barrier();
                if (s_stop) return false;
            }
            if (state) {
                stores_done();
                lds_barrier();
                if (tid < 2) st_dev(&head[8 * tid + 7], (u64)state);
            }
            return true;
        };

        // After the elimination of rows S (own tile in s_x): what a publication
        // needs of the block's inside, a wavefront each. C in s_C (lane k: the rows
        // of the block that take in row k directly or through others; returned to
        // wavefront 0), the closure of U for the blocks that will merge this one
        // (lane b: the rows whose pattern brings in column b), the first matches.
        auto close_rows = [&](u64 S, int part, bool known) -> u64 {
            const u64 x = s_x[ln];
            u64 r = 0;
            if (wv == 0) {
                r = closure(((S >> ln) & 1ull) ? x & above(ln) : 0ull, xs, tab);
                s_C[ln] = r;
            } else if (wv == 1) {
                st_dev(&a.tcl[(int64_t)gb * 128 + 64 * part + ln], closure(x & below(ln) & S, xs, tab));
            } else if (wv == 2) {
                int32_t* km = a.kmatch + 64 * (int64_t)gb;
                const int match = first_match(x, S, s_x);
                if (!known) st_dev(&km[ln], match >= 0 ? 64 * g + match : kNoMatch);
                else if (match >= 0) atomicMin(&km[ln], 64 * g + match);
                const u64 nc = __ballot(match >= 0);
                if (ln == 0) s_con = S & ~nc;
            }
            lds_barrier();
            return r;
        };

        const u64 s_ext0 = s_ext;
        bool first_done = false;
        bool stop = false;

        // ---- rows that depend on no earlier block: finish and publish them now
        if (s_ext0 != 0ull && (rows & ~s_ext0) != 0ull) {
            if (wv == 0) {
                u64 x = ld_wg(&X[64 * (int64_t)g + ln]);
                u64 S = rows & ~s_ext0;
                eliminate_all<true>(x, S, xs, tab);
                X[64 * (int64_t)g + ln] = x;
                s_x[ln] = x;
                if (ln == 0) s_S = S;
            }
            __syncthreads();  // (the store to X too: other wavefronts OR into it next)
            const u64 S = s_S;
            if (S != 0ull) {
                (void)close_rows(S, 0, false);
                stop = !write_list(g + 1, ntiles, S, S, false, 0, 1u);
                first_done = true;
            }
        }

        // ---- merge the earlier blocks that the masks name
        uint32_t n_merge = 0, n_read = 0;
        if (!stop && s_ext0 != 0ull) {
            const int npw = (g + 63) >> 6;
            uint32_t spins = 0;
            // ORs up to kT tiles t (masks m) of a published list into this block's
            // masks: for every column the masks y of the rows in `use` that hold it
            auto merge_tiles = [&](int cnt, const auto& t, const auto& m, const u64* y, u64 use, u64 open, int64_t hb) {
                constexpr int kT = sizeof(m) / sizeof(m[0]);
                u64 z[kT], o[kT];
#pragma unroll
                for (int i = 0; i < kT; ++i) {
                    z[i] = o[i] = 0;
                    if (i < cnt) {
                        for (u64 w = m[i] & use; w; w &= w - 1ull) z[i] |= y[__builtin_ctzll(w)];
                        if (z[i]) o[i] = or_wg(&X[64 * (int64_t)t[i] + ln], z[i]);
                    }
                }
#pragma unroll
                for (int i = 0; i < kT; ++i) {
                    if (i >= cnt) break;
                    if (t[i] == g) {
                        // U(k, v) with v a row of this block: a match where L(v, k) is
                        // there too (of interest for rows k that have none yet)
                        for (u64 w = open; w; w &= w - 1ull) {
                            const int k = __builtin_ctzll(w);
                            const u64 both = __ballot(((m[i] >> k) & 1ull) && ((y[k] >> ln) & 1ull));
                            if (both != 0ull && ln == 0)
                                atomicMin(&a.kmatch[64 * hb + k], 64 * g + __builtin_ctzll(both));
                        }
                    }
                    if (__ballot((z[i] & ~o[i]) != 0ull) != 0ull && ln == 0) {
                        atomicOr(&touch[t[i] >> 6], 1ull << (t[i] & 63));
                        if (t[i] < g) atomicOr(&pend[t[i] >> 6], 1ull << (t[i] & 63));
                    }
                }
            };
            // Takes the lowest block of a bitmap. A wavefront counts itself active
            // before it clears a block's bit and no longer once it has merged it,
            // and looks again after every merge: with nothing waiting and nobody
            // active the merging is done, and whoever marks a block takes it if
            // nobody else does. (A wavefront that only looks must not count:
            // several in step would keep each other here.)
            auto take = [&](u64* bits) -> int {
                for (int w0 = 0; w0 < npw; w0 += 64) {
                    for (;;) {
                        const u64 w = w0 + ln < npw ? ld_lds(&bits[w0 + ln]) : 0ull;
                        const u64 nz = __ballot(w != 0ull);
                        if (nz == 0ull) break;
                        const int l = __builtin_ctzll(nz);
                        const int b = __builtin_ctzll(readlane64(w, l));
                        int got = 0;
                        if (ln == 0) {
                            atomicAdd(&s_active, 1);
                            got = (int)((atomicAnd(&bits[w0 + l], ~(1ull << b)) >> b) & 1ull);
                            if (!got) atomicSub(&s_active, 1);
                        }
                        if (rfl(got)) return (w0 + l) * 64 + b;
                    }
                }
                return -1;
            };
            // Moves the waiting blocks that are published by now to `ready`: the
            // states of 64 blocks per round trip.
            auto poll = [&]() -> bool {
                uint32_t* list = (uint32_t*)tab;  // 512 ids
                bool any = false;
                for (int w0 = 0; w0 < npw; w0 += 64) {
                    u64 w = 0, w2 = 0;
                    if (w0 + ln < npw) {
                        w2 = ld_lds(&wait2[w0 + ln]);
                        w = ld_lds(&wait1[w0 + ln]) | w2;
                    }
                    const int c = __popcll(w);
                    int o = incl_scan(c) - c;
                    const int total = min(sum32(c), 512);
                    for (; w && o < 512; w &= w - 1ull, ++o) {
                        const int b = __builtin_ctzll(w);
                        list[o] = (uint32_t)((w0 + ln) * 64 + b) | ((w2 >> b) & 1ull ? 0x80000000u : 0u);
                    }
                    wave_sync();
                    for (int i0 = 0; i0 < total; i0 += 64) {
                        if (i0 + ln < total) {
                            const uint32_t id = list[i0 + ln];
                            const bool second = id >= 0x80000000u;
                            const int b = (int)(id & 0x7FFFFFFFu);
                            const u64 bit = 1ull << (b & 63);
                            const u64* hd = a.head + (b0 + (int64_t)b) * kBmHeadWords;
                            const u64 s1 = ld_dev(&hd[7]), s2 = ld_dev(&hd[23]);
                            if (s2 != 0ull || (s1 != 0ull && !second)) {
                                // (another wavefront may have taken it meanwhile)
                                if (atomicAnd(second ? &wait2[b >> 6] : &wait1[b >> 6], ~bit) & bit) {
                                    any = true;
                                    atomicOr(&ready[b >> 6], bit);
                                }
                            }
                        }
                    }
                    wave_sync();
                }
                return __ballot(any) != 0ull;
            };
            for (;;) {
                // tiles of a shared merge first
                bool did = false;
#pragma unroll
                for (int k = 0; k < kTasks; ++k) {
                    const u64 peek = ld_lds(&s_tnext[k]);
                    if (rfl((int)lo32(peek)) >= rfl((int)hi32(peek))) continue;
                    u64 w = 0;
                    const int step = rfl(ld_lds(&s_tstep[k]));
                    if (ln == 0) w = atomicAdd(&s_tnext[k], (u64)step);
                    const int i = rfl((int)lo32(w)), nt = rfl((int)hi32(w));
                    if (i >= nt) continue;
                    wave_sync();
                    const int c = min(step, nt - i);
                    const int64_t q = (int64_t)s_toff[k] + i;
                    const int32_t tl = ln < c ? ld_dev(&a.tids[q + ln]) : 0;
                    u64 m[kShare];
                    int32_t t[kShare];
#pragma unroll
                    for (int j = 0; j < kShare; ++j) m[j] = j < c ? ld_dev(&a.masks[64 * (q + j) + ln]) : 0ull;
#pragma unroll
                    for (int j = 0; j < kShare; ++j) t[j] = __builtin_amdgcn_readlane(tl, j);
                    merge_tiles(c, t, m, s_ty[k], s_tuse[k], s_topen[k], b0 + s_tblk[k]);
                    wave_sync();
                    if (ln == 0 && atomicAdd(&s_tdone[k], c) + c == nt) {
                        atomicExch(&s_town[k], 0);
                        atomicSub(&s_active, 1);
                    }
                    n_read += (uint32_t)c;
                    did = true;
                }
                if (did) continue;
                // then blocks known to be published, then new ones; else half of the
                // wavefronts wait for a block each (polling its header, the shortest
                // way on) and one of the others polls all further ones that wait
                bool both = false, wait = false;
                int h = take(ready);
                if (h < 0) h = take(pend);
                if (h < 0) {
                    int c = 0;
                    for (int w0 = ln; w0 < npw; w0 += 64) c += __popcll(ld_lds(&wait1[w0])) + __popcll(ld_lds(&wait2[w0]));
                    c = sum32(c);
                    if (c > 0) {
                        int r = 0;  // 1: may wait, 2: may poll
                        if (ln == 0) {
                            if (atomicAdd(&s_wait, 1) < W / 2) {
                                r = 1;
                            } else {
                                atomicSub(&s_wait, 1);
                                atomicAdd(&s_active, 1);
                                if (atomicExch(&s_poll, 1) == 0) r = 2;
                                else atomicSub(&s_active, 1);
                            }
                        }
                        r = rfl(r);
                        if (r == 1) {
                            wait = true;
                            h = take(wait2);
                            both = h >= 0;
                            if (h < 0) h = take(wait1);
                            if (h < 0) {
                                if (ln == 0) atomicSub(&s_wait, 1);
                                continue;
                            }
                        } else {
                            bool idle = true, dead = false;
                            if (r == 2) {
                                idle = !poll();
                                if (!idle) spins = 0;
                                else if (((++spins) & 15u) == 0u) {
                                    if (spins > kSpinLimit) st_dev(&a.ctl[kBmAbort], (uint32_t)kBmStall);
                                    dead = rfl((int)ld_dev(&a.ctl[kBmAbort])) != 0;
                                }
                                if (ln == 0) {
                                    if (dead) s_stop = 1;
                                    atomicExch(&s_poll, 0);
                                    atomicSub(&s_active, 1);
                                }
                            }
                            if (dead || rfl(ld_lds(&s_stop))) break;
                            if (idle) __builtin_amdgcn_s_sleep(2);
                            continue;
                        }
                    }
                }
                if (h < 0) {
                    const int act = rfl(ld_lds(&s_active));
                    if (act == 0 || rfl(ld_lds(&s_stop))) break;
                    __builtin_amdgcn_s_sleep(2);
                    continue;
                }
                wave_sync();
                const int64_t hb = b0 + h;
                // wait until the rows this block needs of block h are published, or
                // put it back
                u64 y = 0, w = 0, m[4] = {0, 0, 0, 0};
                int part = 0, match = 0;
                bool dead = false, back = false;
                for (;;) {
                    for (;;) {
                        w = ln < kBmHeadWords ? ld_dev(&a.head[hb * kBmHeadWords + ln]) : 0ull;
                        // every lane's words of one load: a uniform view
                        if (readlane64(w, 23) != 0ull && readlane64(w, 31) != 0ull) part = 1;
                        else if (!both && readlane64(w, 7) != 0ull && readlane64(w, 15) != 0ull) part = 0;
                        else part = -1;
                        if (part >= 0) break;
                        if (!wait) {
                            back = true;
                            break;
                        }
                        ++spins;
                        if ((spins & 15u) == 0u) {
                            if (spins > kSpinLimit) st_dev(&a.ctl[kBmAbort], (uint32_t)kBmStall);
                            if (rfl((int)ld_dev(&a.ctl[kBmAbort])) != 0) {
                                dead = true;
                                break;
                            }
                        }
                        __builtin_amdgcn_s_sleep(1);
                    }
                    if (dead || back) break;
                    asm volatile("" ::: "memory");
                    // Nothing orders the words of one load: that it saw the state
                    // words says nothing about the rest. So the header is read again
                    // behind the state, and that copy counts. What the first one says
                    // about the tiles (a word is 0 or final) is good enough to load the
                    // first masks with the same round trip; where the copies differ
                    // they are loaded again.
                    const u64 seen = w;
                    w = ln < kBmHeadWords ? ld_dev(&a.head[hb * kBmHeadWords + ln]) : 0ull;
                    const u64 T = ld_dev(&a.tcl[hb * 128 + part * 64 + ln]);
                    const u64 x = ld_wg(&X[64 * (int64_t)h + ln]);
                    match = ld_dev(&a.kmatch[64 * hb + ln]);
                    auto first_tiles = [&](u64 head) {
                        const int64_t q = (int64_t)readlane64(head, 16 * part + 2);
                        const int cnt = (int)lo32(readlane64(head, 16 * part + 3));
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (i < cnt) m[i] = ld_dev(&a.masks[64 * (q + i) + ln]);
                    };
                    first_tiles(seen);
                    if (__ballot(w != seen) != 0ull) first_tiles(w);
                    y = x | lane_or(x, T, xs, tab);
                    if (part == 0 && (__ballot(y != 0ull) & ~readlane64(w, 0)) != 0ull) {
                        both = true;  // rows of the second publication are needed
                        continue;
                    }
                    if (y != x) or_wg(&X[64 * (int64_t)h + ln], y);
                    break;
                }
                if (wait && ln == 0) atomicSub(&s_wait, 1);
                if (back) {
                    if (ln == 0) {
                        atomicOr(both ? &wait2[h >> 6] : &wait1[h >> 6], 1ull << (h & 63));
                        atomicSub(&s_active, 1);
                    }
                    continue;
                }
                if (dead) {
                    if (ln == 0) {
                        s_stop = 1;
                        atomicSub(&s_active, 1);
                    }
                    break;
                }
                spins = 0;
                ++n_merge;
                const u64 use = __ballot(y != 0ull) & readlane64(w, 16 * part + 1);
                const u64 h_off = readlane64(w, 16 * part + 2);
                const u64 h_num = readlane64(w, 16 * part + 3);
                const int h_cnt = (int)lo32(h_num), h_inl = (int)hi32(h_num);
                // Tiles beyond the last first match of the rows in use are not
                // needed. Only a match below this block counts: a row takes the
                // rest from its match's row if that comes before it.
                const u64 open = use & __ballot(match >= 64 * g);
                int tmax = -1;
                if ((use >> ln) & 1ull) tmax = match >= 64 * g ? kNoMatch : match >> 6;
                tmax = (max64(tmax));
                // lane i: tile i of the list, from the header as far as it goes
                int cnt = 0;
                int32_t t = kNoMatch;
                if (tmax >= 0) {
                    const int src = 16 * part + head_word(ln & ~1);
                    const int tl = __shfl((int)lo32(w), src, 64), th = __shfl((int)hi32(w), src, 64);
                    if (ln < h_inl) t = (ln & 1) ? th : tl;
                    else if (ln < h_cnt) t = ld_dev(&a.tids[(int64_t)h_off + ln]);
                    cnt = __popcll(__ballot(t <= tmax && t != kNoMatch));
                    for (int i0 = 64; i0 < h_cnt && cnt == i0; i0 += 64) {
                        const int32_t ti = i0 + ln < h_cnt ? ld_dev(&a.tids[(int64_t)h_off + i0 + ln]) : kNoMatch;
                        cnt += __popcll(__ballot(ti <= tmax && ti != kNoMatch));
                    }
                }
                int task = -1;
                if (cnt > 4) {
                    if (ln == 0)
                        for (int k = 0; k < kTasks && task < 0; ++k)
                            if (atomicCAS(&s_town[k], 0, 1) == 0) task = k;
                    task = rfl(task);
                }
                if (task >= 0) {
                    // a long list: any wavefront takes tiles of it, all but the four
                    // that are loaded here already
                    s_ty[task][ln] = y;
                    if (ln == 0) {
                        s_toff[task] = h_off;
                        s_tuse[task] = use;
                        s_topen[task] = open;
                        s_tblk[task] = h;
                        s_tdone[task] = 0;
                        s_tstep[task] = min(kShare, (cnt - 4 + W - 1) / W);
                    }
                    wave_sync();
                    if (ln == 0) atomicExch(&s_tnext[task], ((u64)cnt << 32) | 4ull);
                }
                wave_sync();
                xs[ln] = y;
                wave_sync();
                for (int i0 = 0; i0 < (task >= 0 ? 4 : cnt); i0 += 4) {
                    const int c = min(4, cnt - i0);
                    const int64_t q = (int64_t)h_off + i0;
                    int32_t tt[4];
                    if (i0 > 0) {  // (no task free for a longer list)
                        const int32_t tl = ln < c ? ld_dev(&a.tids[q + ln]) : 0;
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            m[j] = j < c ? ld_dev(&a.masks[64 * (q + j) + ln]) : 0ull;
                            tt[j] = __builtin_amdgcn_readlane(tl, j);
                        }
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; ++j) tt[j] = __builtin_amdgcn_readlane(t, j);
                    }
                    merge_tiles(c, tt, m, xs, use, open, hb);
                }
                n_read += (uint32_t)(task >= 0 ? 4 : cnt);
                wave_sync();
                if (task < 0) {
                    if (ln == 0) atomicSub(&s_active, 1);
                } else if (ln == 0 && atomicAdd(&s_tdone[task], 4) + 4 == cnt) {
                    atomicExch(&s_town[task], 0);
                    atomicSub(&s_active, 1);
                }
            }
            lds_barrier();
            stop = s_stop != 0;
        }
        if (stop) break;

        // ---- the block's own rows among each other, then everything published
        u64 own = 0;
        if (wv == 0) {
            own = ld_wg(&X[64 * (int64_t)g + ln]);
            u64 S = rows;
            eliminate_all<false>(own, S, xs, tab);
            s_x[ln] = own;
        }
        lds_barrier();
        const u64 C = close_rows(rows, 1, first_done);
        if (wv == 0) X[64 * (int64_t)g + ln] = 0ull;
        if (!write_list(g + 1, ntiles, rows, rows, true, 1, 2u)) break;
        const u64 u_off = s_off;
        const int u_cnt = s_total;
        lds_barrier();

        // ---- what only later kernels read
        if (!write_list(0, g, rows, 0ull, true, 0, 0u)) break;
        if (wv == 0) {
            a.diag[64 * (int64_t)gb + ln] = own;
            // rows of the closure: lane r, the rows of the block that r takes in
            u64 M = 0;
            for (int r = 0; r < 64; ++r) {
                const u64 w = __ballot((C >> r) & 1ull);
                if (ln == r) M = w;
            }
            a.lcl[64 * (int64_t)gb + ln] = M;
            if (ln == 0) {
                BlockRec* r = &a.rec[gb];
                r->u_off = (int64_t)u_off;
                r->u_cnt = u_cnt;
                r->l_off = (int64_t)s_off;
                r->l_cnt = s_total;
            }
        }
        if (ln == 0) {
            if (n_merge) atomicAdd(&a.jstats[jb].iterations, (u64)n_merge);
            if (n_read) atomicAdd(&a.jstats[jb].edges_gpu, (u64)n_read * 64ull);
        }
        __syncthreads();
    }
}

// -------------------------------------------------------------- row counts

namespace {
// the factorisation neither gave up nor yielded before its last block
__device__ __forceinline__ bool all_done(const BlockArgs& a) {
    return ld_dev(&a.ctl[kBmAbort]) == 0u && ld_dev(&a.ctl[kBmNext]) >= (uint32_t)a.nblocks;
}

constexpr int kPlanes = 16;  // a wavefront counts less than 2^16 tiles

// m's bits, 64 by 64, with rows and columns exchanged
__device__ __forceinline__ u64 transpose64(u64 x) {
    const int ln = lane();
    u64 keep = 0x00000000FFFFFFFFull;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        const u64 y = __shfl_xor(x, d, 64);
        x = ln & d ? (x & ~keep) | ((y >> d) & keep) : (x & keep) | ((y << d) & ~keep);
        keep ^= keep << (d >> 1);
    }
    return x;
}
}  // namespace

// Entries of L and U per row. A lane adds its columns' masks up in bit planes
// (plane j holds bit j of 64 counters, one per row), four tiles in flight; then
// the planes change rows with columns and lane r sums row r's popcounts. A
// ballot per tile and row instead took 468 us on the 64^3 27-point stencil (204 on
// 1000^2 9-point); this way 64 (69): the tiles are
// read once.
// On the way the block's L tiles go into the lists of their columns.
__global__ __launch_bounds__(kThreads) void k_bm_count(BlockArgs a, BlockCols cl) {
    __shared__ int32_t s_cnt[2][64];
    const int ln = lane(), wv = rfl(threadIdx.x >> 6);
    if (!all_done(a)) return;
    const int32_t gb = blockIdx.x;
    const int32_t jb = a.blk_job ? a.blk_job[gb] : 0;
    const Job* J = &a.jobs[jb];
    const int32_t b0 = (int32_t)J->item_base;
    const int32_t g = gb - b0;
    const int32_t nr = min(64, J->n - 64 * g);
    const BlockRec rec = a.rec[gb];
    for (int i = threadIdx.x; i < rec.l_cnt; i += kThreads) {
        const int64_t q = rec.l_off + i;
        const int64_t e = cl.ptr[b0 + a.tids[q]] + a.slot[q];
        cl.blk[e] = g;
        cl.tile[e] = (int32_t)q;
    }
    if (threadIdx.x < 128) s_cnt[threadIdx.x >> 6][ln] = 0;
    __syncthreads();
    const u64 d = a.diag[64 * (int64_t)gb + ln];
#pragma unroll
    for (int part = 0; part < 2; ++part) {
        const int64_t off = part ? rec.u_off : rec.l_off;
        const int32_t cnt = part ? rec.u_cnt : rec.l_cnt;
        u64 c[kPlanes];
#pragma unroll
        for (int p = 0; p < kPlanes; ++p) c[p] = 0;
        int k = 0;  // masks added so far
        auto add = [&](u64 m) {
            ++k;
#pragma unroll
            for (int p = 0; p < kPlanes; ++p) {
                const u64 t = c[p] & m;
                c[p] ^= m;
                m = t;
                if (k < (2 << p)) break;
            }
        };
        if (wv == 0) add(part ? d & ~above(ln) : d & above(ln));
        for (int i0 = wv; i0 < cnt; i0 += 16) {
            u64 m[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) m[j] = i0 + 4 * j < cnt ? a.masks[64 * (off + i0 + 4 * j) + ln] : 0ull;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (i0 + 4 * j < cnt) add(m[j]);
        }
        int sum = 0;
#pragma unroll
        for (int p = 0; p < kPlanes; ++p) {
            if (k < (1 << p)) break;
            sum += __popcll(transpose64(c[p])) << p;
        }
        if (k) atomicAdd(&s_cnt[part][ln], sum);
    }
    __syncthreads();
    if (threadIdx.x < nr) {
        const int64_t row = J->row_base + 64 * (int64_t)g + threadIdx.x;
        a.row_lcnt[row] = s_cnt[0][threadIdx.x];
        a.row_ucnt[row] = s_cnt[1][threadIdx.x];
    }
}

// ---------------------------------------------------------- L by columns
//
// L's tiles seen from the columns: for every block of columns the blocks of
// rows with a tile there. k_bm_count puts each tile into its column block's list
// (in the place it took during the factorisation), k_bm_lists sorts the lists by
// row block and counts the entries of every column.

// A tile of which the reach counts need one entry stands in their lists (not in the
// blocks' records) as that entry, row and column inside their blocks, in place of its
// place in the pool: nobody loads 512 bytes for a bit, and k_bm_reach_big takes 64
// such tiles at a time, a lane each. (200,000 rows with one entry below the diagonal
// at random each, where the first block of columns reaches every row through 200,000
// such tiles: 10.5 ms four tiles at a time, 2.2 so; three entries each 41 and 11.)
__device__ __forceinline__ int32_t one_entry(int row, int col) { return ~((row << 6) | col); }
__device__ __forceinline__ int entry_row(int32_t q) { return ~q >> 6; }
__device__ __forceinline__ int entry_col(int32_t q) { return ~q & 63; }

// the masks of a list's tile (the same for all lanes)
__device__ __forceinline__ u64 listed_masks(const u64* masks, int32_t q) {
    const int ln = lane();
    if (q < 0) return ln == entry_col(q) ? 1ull << entry_row(q) : 0ull;
    return masks[64 * (int64_t)q + ln];
}

// the rows of block g up to (and with) a column's match
__device__ __forceinline__ u64 upto(u64 m, int32_t g, int32_t match) {
    if (g < (match >> 6)) return m;
    if (g > (match >> 6)) return 0ull;
    return m & ~above(match & 63);
}

namespace {
// Phase I: a row with one U entry less than the row above may extend that
// row's supernode (inside the same run of max_super rows). Phase II: a chain of
// such rows is cut before every row s without L(s, r), r the supernode's first
// row so far. A wavefront takes the chains that begin in its block and follows
// the last one into the next blocks; inside a block the next cut is the first
// bit missing from column r's mask, a few scalar instructions, where one lane
// per chain and a binary search of L per row took 344 us on the 64^3 27-point
// stencil (1000^2 9-point 298), this 11 (26).
__device__ __forceinline__ void supernodes_of(const BlockArgs& a, int32_t gb, int64_t max_super, int32_t* is_start) {
    const int ln = lane();
    const int32_t jb = a.blk_job ? a.blk_job[gb] : 0;
    const Job* J = &a.jobs[jb];
    const int32_t b0 = (int32_t)J->item_base, n = J->n;
    const int32_t* uc = a.row_ucnt + J->row_base;
    int32_t* out = is_start + J->row_base;
    int32_t r = -1;  // first row of the supernode that goes on
    for (int32_t g = gb - b0; 64 * (int64_t)g < n; ++g) {
        const int32_t v = 64 * g + ln;
        const bool in = v < n;
        const int32_t u = in ? uc[v] : 0, above_u = in && v > 0 ? uc[v - 1] : 0;
        const u64 d = a.diag[64 * (int64_t)(b0 + g) + ln];
        const u64 rows = __ballot(in);
        const u64 F = __ballot(in && v > 0 && (max_super <= 0 || v % max_super != 0) && u == above_u - 1);
        const bool first = g == gb - b0;
        // rows of chains that begin here, or of the one that goes on
        const int lead = rows & ~F ? __builtin_ctzll(rows & ~F) : 64;
        u64 todo = first ? (lead < 64 ? rows & ~below(lead) : 0ull) : lead < 64 ? rows & below(lead) : rows;
        if (todo == 0ull) break;
        const u64 mine = todo;
        u64 starts = 0;
        u64 C = 0;  // rows of this block with an entry in column r
        if (!first) {
            // the tile of r's column block, near the end of the block's L list
            const BlockRec rec = a.rec[b0 + g];
            for (int i = rec.l_cnt; i > 0; i -= 64) {
                const int32_t t = i - 64 + ln >= 0 ? a.tids[rec.l_off + i - 64 + ln] : -1;
                const u64 hit = __ballot(t == (r >> 6));
                if (hit) C = a.masks[64 * (rec.l_off + i - 64 + __builtin_ctzll(hit)) + (r & 63)];
                if (hit || __builtin_amdgcn_readlane(t, 0) < (r >> 6)) break;
            }
        }
        for (;;) {
            // (the first row of a chain is no follower and starts one here)
            const u64 cut = todo & ~(F & C);
            if (cut == 0ull) break;
            const int s = __builtin_ctzll(cut);
            starts |= 1ull << s;
            r = 64 * g + s;
            C = readlane64(d, s);
            todo &= above(s);
        }
        if ((mine >> ln) & 1ull) out[v] = (int32_t)((starts >> ln) & 1ull);
        // (a chain that reaches the block's last row may go on in the next block)
        if (!(mine >> 63)) break;
    }
}
}  // namespace

// One wavefront per block of columns. Lists of more than 64 tiles are ranked in a
// bitmap over the row blocks (dynamic LDS: one bit and one prefix per 64 blocks).
// The tiles with an entry up to their column's first match, all that the reach
// counts need and one or two in a separator, stay as (blk, tile) at the list's
// start, the first of them in the block's record.
// The block's supernodes follow (is_start; nullptr: not wanted).
__global__ __launch_bounds__(64) void k_bm_lists(BlockArgs a, BlockCols c, int32_t* col_cnt, int64_t max_super,
                                                 int32_t* is_start) {
    extern __shared__ u64 s_dyn[];
    if (!all_done(a)) return;
    const int ln = lane();
    const int32_t cb = blockIdx.x;
    const int32_t jb = a.blk_job ? a.blk_job[cb] : 0;
    const Job* J = &a.jobs[jb];
    const int32_t c0 = cb - (int32_t)J->item_base;
    const int64_t e0 = c.ptr[cb], e1 = c.ptr[cb + 1];
    const int cnt = (int)(e1 - e0);
    const int32_t match = a.kmatch[64 * (int64_t)cb + ln];
    int32_t sum = __popcll(a.diag[64 * (int64_t)cb + ln] & above(ln));
    int kept = 0;
    int32_t word = 0;  // the record: lane 0 the count, lanes 1.. row blocks, 8.. tiles
    // k tiles of a list (lane i: row block b, tile q): their entries per column,
    // and which of them the reach counts need
    auto walk = [&](int k, int32_t b, int32_t q) {
        u64 keep = 0, occ = 0;
        int32_t t = q;
        for (int i0 = 0; i0 < k; i0 += 4) {
            u64 m[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                m[j] = i0 + j < k ? a.masks[64 * (int64_t)__builtin_amdgcn_readlane(q, (i0 + j) & 63) + ln] : 0ull;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                sum += __popcll(m[j]);
                const int i = (i0 + j) & 63;
                const int32_t g = __builtin_amdgcn_readlane(b, i);
                const u64 x = upto(m[j], g, match);
                const u64 cols = __ballot(x != 0ull);
                if (cols != 0ull) keep |= 1ull << i;
                if (ln == i) occ = cols;
                if (cols != 0ull && (cols & (cols - 1ull)) == 0ull) {
                    const int k = __builtin_ctzll(cols);
                    const u64 rows = readlane64(x, k);
                    if ((rows & (rows - 1ull)) == 0ull && ln == i) t = one_entry(__builtin_ctzll(rows), k);
                }
            }
        }
        if ((keep >> ln) & 1ull) {
            const int64_t d = e0 + kept + (int)below_count(keep);
            c.blk[d] = b;
            c.tile[d] = t;
            c.occ[d] = occ;
        }
        for (u64 w = keep; w && kept < kReachInline; w &= w - 1ull) {
            const int i = __builtin_ctzll(w);
            const int32_t bi = __builtin_amdgcn_readlane(b, i), qi = __builtin_amdgcn_readlane(q, i);
            if (ln == 1 + kept) word = bi;
            if (ln == 1 + kReachInline + kept) word = qi;
            ++kept;
            keep &= keep - 1ull;
        }
        kept += __popcll(keep);
    };
    if (cnt <= 64) {
        const int32_t b = ln < cnt ? c.blk[e0 + ln] : kNoMatch;
        const int32_t q = ln < cnt ? c.tile[e0 + ln] : 0;
        int rank = 0;
        for (int i = 0; i < cnt; ++i) rank += __builtin_amdgcn_readlane(b, i) < b ? 1 : 0;
        if (ln < cnt) {
            c.blk2[e0 + rank] = b;
            c.tile2[e0 + rank] = q;
        }
        walk(cnt, b, q);
    } else {
        const int nw = a.bit_words;
        u64* bits = s_dyn;
        int32_t* pre = (int32_t*)(s_dyn + nw);
        for (int i = ln; i < nw; i += 64) bits[i] = 0ull;
        wave_sync();
        for (int64_t e = e0 + ln; e < e1; e += 64) atomicOr(&bits[c.blk[e] >> 6], 1ull << (c.blk[e] & 63));
        wave_sync();
        int run = 0;
        for (int i0 = 0; i0 < nw; i0 += 64) {
            const int p = i0 + ln < nw ? __popcll(bits[i0 + ln]) : 0;
            const int inc = incl_scan(p);
            if (i0 + ln < nw) pre[i0 + ln] = run + inc - p;
            run += __builtin_amdgcn_readlane(inc, 63);
        }
        wave_sync();
        for (int64_t f0 = e0; f0 < e1; f0 += 64) {
            const int k = (int)min((int64_t)64, e1 - f0);
            const int32_t q = ln < k ? c.tile[f0 + ln] : 0;
            const int32_t b = ln < k ? c.blk[f0 + ln] : 0;
            if (ln < k) {
                const int64_t d = e0 + pre[b >> 6] + __popcll(bits[b >> 6] & below(b & 63));
                c.blk2[d] = b;
                c.tile2[d] = q;
            }
            walk(k, b, q);  // (keeps no more than it has read: in place)
        }
    }
    if (ln == 0) word = kept;
    if (ln < kReachWords) c.reach[(int64_t)cb * kReachWords + ln] = word;
    const int64_t v = 64 * (int64_t)c0 + ln;
    if (v < J->n) col_cnt[J->row_base + v] = sum;
    if (is_start) supernodes_of(a, cb, max_super, is_start);
}

// ---------------------------------------------------------------- emission
//
// Both kernels write 16 of a block's rows (columns) per wavefront. The places of
// the 16 are scalar registers and move by scalar popcounts; a row's ids of one
// tile are the set bits of one mask, stored side by side by the lanes that hold
// them. Tiles are loaded four ahead of their turn. 64^3 27-point: rows 395 -> 288
// us, columns 489 -> 345, 130 of it without the stores; 1000^2 9-point 206 -> 124
// and 192 -> 129, 99 of it without the stores. (Collecting 64 ids per row in LDS,
// for whole aligned stores, took 377 and 421 us; masks by scalar loads as long
// as this on the first and longer on the second.)

namespace {

// Rows of U, or of L row-wise.
template <bool upper>
__device__ __forceinline__ void emit_rows(const BlockArgs& a, int32_t gb, const int64_t* ptr, int32_t* idx) {
    const int ln = lane(), wv = rfl(threadIdx.x >> 6);
    const int32_t jb = a.blk_job ? a.blk_job[gb] : 0;
    const Job* J = &a.jobs[jb];
    const int32_t g = gb - (int32_t)J->item_base;
    const int32_t nr = min(64, J->n - 64 * g);
    const BlockRec rec = a.rec[gb];
    const int r0 = 16 * wv;
    if (r0 >= nr) return;
    // (no branch on the lane: the places stay known as scalars)
    const int64_t at = ptr[J->row_base + 64 * (int64_t)g + r0 + min(ln, min(16, nr - r0) - 1)];
    int32_t* p[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) p[i] = idx + readlane64((u64)at, i);
    auto put = [&](u64 m, int32_t id) {
        const uint32_t w = (uint32_t)(m >> r0);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const u64 b = __ballot((w & (1u << i)) != 0u);
            if (__builtin_amdgcn_inverse_ballot_w64(b)) p[i][below_count(b)] = id;
            p[i] += __popcll(b);
        }
    };
    const u64 d = a.diag[64 * (int64_t)gb + ln];
    if (upper) put(d & ~above(ln), 64 * g + ln);
    const int64_t off = upper ? rec.u_off : rec.l_off;
    const int32_t cnt = upper ? rec.u_cnt : rec.l_cnt;
    u64 m[4];
    int32_t t[4];
    auto load = [&](int i, int32_t tl) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            m[j] = i + j < cnt ? a.masks[64 * (off + i + j) + ln] : 0ull;
            t[j] = __builtin_amdgcn_readlane(tl, (i + j) & 63);
        }
    };
    int32_t tl = ln < cnt ? a.tids[off + ln] : 0;
    load(0, tl);
    for (int i = 0; i < cnt; i += 4) {
        u64 m0[4];
        int32_t t0[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            m0[j] = m[j];
            t0[j] = t[j];
        }
        if (((i + 4) & 63) == 0) tl = i + 4 + ln < cnt ? a.tids[off + i + 4 + ln] : 0;
        load(i + 4, tl);
#pragma unroll
        for (int j = 0; j < 4; ++j) put(m0[j], 64 * t0[j] + ln);
    }
    if (!upper) put(d & above(ln), 64 * g + ln);
}

// Columns of L: the tiles of a block of columns by ascending row block, the rows
// of a column being the set bits of its mask. One load brings the wavefront's 16
// columns of four tiles.
__device__ __forceinline__ void emit_cols(const BlockArgs& a, const BlockCols& c, int32_t cb, const int64_t* l_ptr,
                                          int32_t* l_idx) {
    const int ln = lane(), wv = rfl(threadIdx.x >> 6);
    const int32_t jb = a.blk_job ? a.blk_job[cb] : 0;
    const Job* J = &a.jobs[jb];
    const int32_t c0 = cb - (int32_t)J->item_base;
    const int nc = min(16, J->n - 64 * c0 - 16 * wv);
    if (nc <= 0) return;
    // (no branch on the lane: the places stay known as scalars)
    const int64_t at = l_ptr[J->row_base + 64 * (int64_t)c0 + 16 * wv + min(ln, nc - 1)];
    int32_t* p[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) p[i] = l_idx + readlane64((u64)at, i);
    const int col = 16 * wv + (ln & 15);
    auto put = [&](int32_t g, u64 m, int j) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const u64 w = readlane64(m, 16 * j + i);
            if (__builtin_amdgcn_inverse_ballot_w64(w)) p[i][below_count(w)] = 64 * g + ln;
            p[i] += __popcll(w);
        }
    };
    put(c0, a.diag[64 * (int64_t)cb + col] & above(col), 0);
    const int64_t e0 = c.ptr[cb];
    const int cnt = (int)(c.ptr[cb + 1] - e0);
    int32_t bl = 0, tl = 0;
    auto ids = [&](int i) {
        const bool in = i + ln < cnt;
        bl = in ? c.blk2[e0 + i + ln] : 0;
        tl = in ? c.tile2[e0 + i + ln] : 0;
    };
    // (the shuffle before the test: it reads lanes that the test leaves out)
    auto load = [&](int i) -> u64 {
        const int32_t q = __shfl(tl, (i + (ln >> 4)) & 63, 64);
        return i + (ln >> 4) < cnt ? a.masks[64 * (int64_t)q + col] : 0ull;
    };
    ids(0);
    u64 m = load(0);
    for (int i = 0; i < cnt; i += 4) {
        const u64 m0 = m;
        int32_t g[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) g[j] = __builtin_amdgcn_readlane(bl, (i + j) & 63);
        if (((i + 4) & 63) == 0) ids(i + 4);
        m = load(i + 4);
#pragma unroll
        for (int j = 0; j < 4; ++j) put(g[j], m0, j);
    }
}

}  // namespace

// ------------------------------------------------------------------- reach
//
// edges_alg counts, for every source s, the degrees of the vertices reachable
// from s through vertices below s. Such a vertex v is in L(s,:) or reachable
// from some k of L(s,:) (the largest vertex of the path), so the sources that
// reach v are the ancestors of v in the graph of L's columns. One wavefront
// takes 64 vertices (a block c) and carries, for one block of rows after the
// other, the mask of c's vertices that each row reaches: rows of a block among
// each other through the closure lcl, later blocks through L's tiles up to
// each column's match (a row beyond the match reaches everything through it).
// Few blocks wait at a time, so they sit in a few LDS tiles; a wavefront
// that needs more hands its block to k_bm_reach_big.
// Bound by its instructions, some 300 per block of rows on the way up: what a
// block needs comes from one record, loaded while the one before it is worked on;
// few rows' words go through the closure one by one, more by table; the degrees'
// planes sit in registers.

namespace {
constexpr int kReachPlanes = 6;
constexpr int kReachRows = 12;  // rows in use up to which their words go one by one

// sum of the degrees in a mask: bit planes of the degrees, one popcount each
__device__ __forceinline__ u64 weigh(u64 z, const u64* planes, int np, int first) {
    u64 s = 0;
    for (int j = first; j < np; ++j) s += (u64)__popcll(z & planes[j]) << j;
    return s;
}

__device__ __forceinline__ int degree_planes(const Job* J, int32_t c, u64* planes) {
    const int ln = lane();
    const int64_t v = 64 * (int64_t)c + ln;
    const uint32_t deg = v < J->n ? (uint32_t)(J->row_ptr[v + 1] - J->row_ptr[v]) : 0u;
    const uint32_t top = (uint32_t)(max64((int)deg));
    const int np = top ? 32 - __builtin_clz(top) : 0;
    for (int j = 0; j < np; ++j) {
        const u64 p = __ballot((deg >> j) & 1u);
        if (ln == 0) planes[j] = p;
    }
    return np;
}
}  // namespace

namespace {
template <int kTiles>
struct ReachLds {
    __attribute__((aligned(16))) u64 xs[64];
    u64 tile[kTiles][64];
    u64 tab[256];
    u64 planes[32];
};

template <int kTiles>
__device__ __forceinline__ void reach_of(const BlockArgs& a, const BlockCols& cl, int32_t cb, ReachLds<kTiles>& S) {
    const int ln = lane();
    if (cb >= a.nblocks || ld_dev(&a.ctl[kBmAbort]) != 0u) return;
    const int32_t jb = a.blk_job ? a.blk_job[cb] : 0;
    const Job* J = &a.jobs[jb];
    const int32_t b0 = (int32_t)J->item_base;
    const int32_t c = cb - b0;
    const int np = degree_planes(J, c, S.planes);
    int32_t key = kNoMatch;  // lane i < kTiles: block waiting in tile i
    if (ln == 0) key = c;
    static_assert(kTiles <= 16 && kReachInline < 16, "min16");
    S.tile[0][ln] = 64 * (int64_t)c + ln < J->n ? 1ull << ln : 0ull;
    wave_sync();
    // the degrees' lowest planes and their counts in registers
    u64 plane[kReachPlanes];
    uint32_t hits[kReachPlanes];
#pragma unroll
    for (int j = 0; j < kReachPlanes; ++j) {
        plane[j] = j < np ? S.planes[j] : 0ull;
        hits[j] = 0;
    }
    u64 sum = 0;
    // what a block needs, loaded while the one before it is worked on
    u64 M;
    int32_t match, word, at = -1;
    auto fetch = [&](int32_t h) {
        at = h;
        const int64_t hb = b0 + h;
        M = a.lcl[64 * hb + ln];
        match = a.kmatch[64 * hb + ln];
        word = cl.reach[hb * kReachWords + (ln & (kReachWords - 1))];
    };
    for (;;) {
        const int32_t h = min16(key);
        if (h == kNoMatch) break;
        if (h != at) fetch(h);
        const int sl = __builtin_ctzll(__ballot(key == h));
        const int64_t hb = b0 + h;
        const int cnt = __builtin_amdgcn_readlane(word, 0);
        const int32_t w0 = word, match0 = match;
        u64 m[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            m[j] = j < cnt ? a.masks[64 * (int64_t)__builtin_amdgcn_readlane(w0, 1 + kReachInline + j) + ln] : 0ull;
        const u64 z0 = S.tile[sl][ln], M0 = M;
        if (ln == sl) key = kNoMatch;
        // the next one is waiting already or comes in now
        {
            const int32_t mine = ln >= 1 && ln <= min(cnt, kReachInline) ? w0 : kNoMatch;
            const int32_t next = min16(min(key, mine));
            if (next != kNoMatch) fetch(next);
        }
        u64 z = z0;
        const u64 from = __ballot(z0 != 0ull);
        if (h == c) {
            z |= M0;  // (row k starts with vertex k)
        } else if (__popcll(from) <= kReachRows) {
            for (u64 w = from; w; w &= w - 1ull) {
                const int k = __builtin_ctzll(w);
                const u64 zk = readlane64(z0, k);
                z |= (M0 >> k) & 1ull ? zk : 0ull;
            }
        } else {
            z |= lane_or(z0, M0, S.xs, S.tab);
        }
#pragma unroll
        for (int j = 0; j < kReachPlanes; ++j) hits[j] += (uint32_t)__popcll(z & plane[j]);
        if (np > kReachPlanes) sum += weigh(z, S.planes, np, kReachPlanes);
        bool over = false;
        auto push = [&](int32_t g, u64 mask) {
            const u64 x = z != 0ull ? upto(mask, g, match0) : 0ull;
            if (__ballot(x != 0ull) == 0ull) return;
            const u64 hit = __ballot(key == g);
            int s2;
            if (hit) {
                s2 = __builtin_ctzll(hit);
            } else {
                const u64 fr = __ballot(ln < kTiles && key == kNoMatch);
                if (fr == 0ull) {
                    over = true;
                    return;
                }
                s2 = __builtin_ctzll(fr);
                if (ln == s2) key = g;
                S.tile[s2][ln] = 0ull;
                wave_sync();
            }
            for (u64 t = x; t; t &= t - 1ull) atomicOr(&S.tile[s2][__builtin_ctzll(t)], z);
            wave_sync();
        };
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (j < cnt && !over) push(__builtin_amdgcn_readlane(w0, 1 + j), m[j]);
        if (cnt > 4) {
            const int64_t e0 = cl.ptr[hb];
            const u64 used = __ballot(z != 0ull);
            for (int i0 = 4; i0 < cnt && !over; i0 += 64) {
                const bool in = i0 + ln < cnt;
                const int32_t gl = in ? cl.blk[e0 + i0 + ln] : 0, tl = in ? cl.tile[e0 + i0 + ln] : 0;
                for (u64 w = __ballot(in && (cl.occ[e0 + i0 + ln] & used) != 0ull); w && !over; w &= w - 1ull) {
                    const int i = __builtin_ctzll(w);
                    push(__builtin_amdgcn_readlane(gl, i), listed_masks(a.masks, __builtin_amdgcn_readlane(tl, i)));
                }
            }
        }
        if (over) {
            if (ln == 0) cl.big[atomicAdd(cl.nbig, 1)] = cb;
            return;
        }
    }
    // (every vertex has counted itself once)
    for (int j = 0; j < np; ++j) sum -= (u64)((S.planes[j] >> ln) & 1ull) << j;
#pragma unroll
    for (int j = 0; j < kReachPlanes; ++j) sum += (u64)hits[j] << j;
    sum = sum64(sum);
    if (ln == 0 && sum) atomicAdd(&a.jstats[jb].edges_alg, sum);
}
}  // namespace

// Everything that is written once the sizes of U and L are known, in one launch
// (64^3 27-point: 980 -> 663 us; 1000^2 9-point 685 -> 558; 512 batch members 1,043 -> 729).
// Of nine workgroups one takes reach counts and eight rows and columns of four
// blocks, so that both kinds are in flight all the time.
template <bool l_csr, int kTiles>
__global__ __launch_bounds__(kThreads) void k_bm_emit(BlockArgs a, BlockCols c, const int64_t* u_ptr, int32_t* u_idx,
                                                      const int64_t* l_ptr, int32_t* l_idx) {
    __shared__ ReachLds<kTiles> s_reach[kThreads / 64];
    const int32_t k = (int32_t)(blockIdx.x / 9u), what = (int32_t)(blockIdx.x % 9u);
    const int32_t b = 4 * k + ((what - 1) >> 1);
    const int wv = rfl(threadIdx.x >> 6);
    if (what == 0) reach_of<kTiles>(a, c, 4 * k + wv, s_reach[wv]);
    else if (b >= a.nblocks) return;
    else if (what & 1) emit_rows<true>(a, b, u_ptr, u_idx);
    else if (l_csr) emit_rows<false>(a, b, l_ptr, l_idx);
    else emit_cols(a, c, b, l_ptr, l_idx);
}

// The same with the blocks' masks in a slot of X (all zero between uses) and bitmaps
// of the blocks waiting and met in LDS. A block of columns may reach most of the
// matrix here, so sixteen wavefronts share it: they take waiting blocks, lowest first,
// and whoever adds to a block's masks sets it waiting (again). A wavefront counts
// itself active from before it clears a block's bit until it has passed the block
// on, so with nothing waiting and nobody active the masks are final, and are
// weighed. (200,000 rows with an entry below the diagonal at random each, where
// nothing can be pruned: 73 ms with a wavefront per block of columns, 10 so, 2.2
// with lanes for tiles of one entry.)
namespace {
constexpr int kBigWaves = 16;
}

__global__ __launch_bounds__(64 * kBigWaves) void k_bm_reach_big(BlockArgs a, BlockCols cl) {
    extern __shared__ u64 s_bits[];
    __shared__ __attribute__((aligned(16))) u64 s_xs[kBigWaves][64];
    __shared__ u64 s_tab[kBigWaves][256];
    __shared__ u64 s_planes[32];
    __shared__ int s_np, s_active;
    if (ld_dev(&a.ctl[kBmAbort]) != 0u) return;
    const int ln = lane(), wv = rfl(threadIdx.x >> 6);
    u64* Z = a.x + (int64_t)blockIdx.x * a.x_stride;
    const int nw = a.bit_words;
    u64* wait = s_bits;
    u64* met = s_bits + nw;
    const int32_t total = *cl.nbig;
    for (int32_t q = blockIdx.x; q < total; q += gridDim.x) {
        const int32_t cb = cl.big[q];
        const int32_t jb = a.blk_job ? a.blk_job[cb] : 0;
        const Job* J = &a.jobs[jb];
        const int32_t b0 = (int32_t)J->item_base;
        const int32_t c = cb - b0;
        for (int i = threadIdx.x; i < 2 * nw; i += 64 * kBigWaves) s_bits[i] = 0ull;
        if (wv == 0) {
            const int np = degree_planes(J, c, s_planes);
            if (ln == 0) {
                s_np = np;
                s_active = 0;
            }
            if (64 * (int64_t)c + ln < J->n) or_wg(&Z[64 * (int64_t)c + ln], 1ull << ln);
        }
        __syncthreads();
        if (threadIdx.x == 0) wait[c >> 6] = met[c >> 6] = 1ull << (c & 63);
        __syncthreads();
        for (;;) {
            int32_t h = -1;
            for (int w0 = 0; w0 < nw && h < 0; w0 += 64) {
                for (;;) {
                    const u64 w = w0 + ln < nw ? ld_lds(&wait[w0 + ln]) : 0ull;
                    const u64 nz = __ballot(w != 0ull);
                    if (nz == 0ull) break;
                    const int l = __builtin_ctzll(nz);
                    const int b = __builtin_ctzll(readlane64(w, l));
                    int got = 0;
                    if (ln == 0) {
                        atomicAdd(&s_active, 1);
                        got = (int)((atomicAnd(&wait[w0 + l], ~(1ull << b)) >> b) & 1ull);
                        if (!got) atomicSub(&s_active, 1);
                    }
                    if (rfl(got)) {
                        h = (w0 + l) * 64 + b;
                        break;
                    }
                }
            }
            if (h < 0) {
                // (looked after the scan: a block set waiting before the last active
                // wavefront left would have been seen by that wavefront itself)
                if (rfl(ld_lds(&s_active)) == 0) break;
                __builtin_amdgcn_s_sleep(2);
                continue;
            }
            wave_sync();
            const int64_t hb = b0 + h;
            const u64 z0 = ld_wg(&Z[64 * (int64_t)h + ln]);
            const u64 M = a.lcl[64 * hb + ln];
            const int32_t match = a.kmatch[64 * hb + ln];
            const int64_t e0 = cl.ptr[hb];
            const int cnt = cl.reach[hb * kReachWords];
            const u64 z = z0 | lane_or(z0, M, s_xs[wv], s_tab[wv]);
            if (z != z0) or_wg(&Z[64 * (int64_t)h + ln], z);
            const u64 used = __ballot(z != 0ull);
            for (int i0 = 0; i0 < cnt; i0 += 64) {
                const bool in = i0 + ln < cnt;
                const int32_t gl = in ? cl.blk[e0 + i0 + ln] : 0, tl = in ? cl.tile[e0 + i0 + ln] : 0;
                // only the tiles with an entry in a column in use: single entries a lane
                // each, the others four at a time
                const bool need = in && (cl.occ[e0 + i0 + ln] & used) != 0ull;
                const u64 zk = __shfl(z, entry_col(tl), 64);
                if (need && tl < 0) {
                    const u64 old = or_wg(&Z[64 * (int64_t)gl + entry_row(tl)], zk);
                    if (zk & ~old) {
                        atomicOr(&met[gl >> 6], 1ull << (gl & 63));
                        atomicOr(&wait[gl >> 6], 1ull << (gl & 63));
                    }
                }
                for (u64 w = __ballot(need && tl >= 0); w;) {
                    u64 m[4];
                    int32_t g[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        m[j] = 0;
                        g[j] = 0;
                        if (w) {
                            const int i = __builtin_ctzll(w);
                            w &= w - 1ull;
                            g[j] = __builtin_amdgcn_readlane(gl, i);
                            m[j] = a.masks[64 * (int64_t)__builtin_amdgcn_readlane(tl, i) + ln];
                        }
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const u64 x = z != 0ull ? upto(m[j], g[j], match) : 0ull;
                        // lane r: what the columns in use bring to row r of block g
                        u64 add = 0;
                        for (u64 k = __ballot(x != 0ull); k; k &= k - 1ull) {
                            const int i = __builtin_ctzll(k);
                            const u64 zi = readlane64(z, i);
                            add |= (readlane64(x, i) >> ln) & 1ull ? zi : 0ull;
                        }
                        bool more = false;
                        if (add) more = (add & ~or_wg(&Z[64 * (int64_t)g[j] + ln], add)) != 0ull;
                        if (__ballot(more) != 0ull && ln == 0) {
                            atomicOr(&met[g[j] >> 6], 1ull << (g[j] & 63));
                            atomicOr(&wait[g[j] >> 6], 1ull << (g[j] & 63));
                        }
                    }
                }
            }
            wave_sync();
            if (ln == 0) atomicSub(&s_active, 1);
        }
        __syncthreads();
        u64 sum = 0;
        for (int i = wv; i < nw; i += kBigWaves)
            for (u64 w = met[i]; w; w &= w - 1ull) {
                const int32_t h = i * 64 + __builtin_ctzll(w);
                const u64 z = ld_wg(&Z[64 * (int64_t)h + ln]);
                Z[64 * (int64_t)h + ln] = 0ull;
                sum += weigh(h == c ? z & ~(1ull << ln) : z, s_planes, s_np, 0);
            }
        sum = sum64(sum);
        if (ln == 0 && sum) atomicAdd(&a.jstats[jb].edges_alg, sum);
        __syncthreads();  // (also the stores to Z, before the next block's)
    }
}

// ------------------------------------------------------- sums and results
//
// Small calls are made of launches that do next to nothing (4 to 5 us each, 33 of
// them around a factorisation of 270 us on a 40 x 40 grid), so what can share
// one does: the running sums of up to three arrays of a length, everything the
// host waits for, everything that only needs the finished sums.

namespace {
constexpr int kScanThreads = 1024;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanThreads * kScanItems;
// One workgroup per array up to a tile, 8,192 values (4.7 us; a second turn of the
// same workgroup made it 16), beyond it two launches of at least 4.5 us each.
constexpr int64_t kScanOne = kScanTile;

struct BlockScans {
    BlockScan s[3];
};

// A tile's values, kScanItems per thread; scan returns their sum, *at what comes
// before the thread's own.
struct TileScan {
    int32_t v[kScanItems];

    __device__ __forceinline__ void load(const int32_t* in, int64_t t0, int64_t n) {
        const int64_t i0 = t0 + (int64_t)threadIdx.x * kScanItems;
        if (i0 + kScanItems <= n) {  // (in: 16-byte aligned)
#pragma unroll
            for (int k = 0; k < kScanItems; k += 4) {
                const int4 w = *(const int4*)(in + i0 + k);
                v[k] = w.x;
                v[k + 1] = w.y;
                v[k + 2] = w.z;
                v[k + 3] = w.w;
            }
            return;
        }
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) v[k] = i0 + k < n ? in[i0 + k] : 0;
    }
    __device__ __forceinline__ int64_t scan(int64_t* sh, int64_t* at) {
        const int wv = threadIdx.x >> 6;
        int64_t sum = 0;
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) sum += v[k];
        int64_t x = sum;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int64_t t = __shfl_up(x, (unsigned)d, 64);
            if (lane() >= d) x += t;
        }
        if (lane() == 63) sh[wv] = x;
        __syncthreads();
        int64_t pre = 0, total = 0;
        for (int w = 0; w < kScanThreads / 64; ++w) {
            if (w < wv) pre += sh[w];
            total += sh[w];
        }
        __syncthreads();
        *at = pre + x - sum;
        return total;
    }
    __device__ __forceinline__ void store(int64_t* out, int64_t t0, int64_t n, int64_t at) const {
        const int64_t i0 = t0 + (int64_t)threadIdx.x * kScanItems;
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            if (i0 + k < n) out[i0 + k] = at;
            at += v[k];
        }
    }
};
}  // namespace

__global__ __launch_bounds__(kScanThreads) void k_bm_scan_one(BlockScans all, int64_t n) {
    __shared__ int64_t sh[kScanThreads / 64];
    const BlockScan s = all.s[blockIdx.x];
    TileScan t;
    t.load(s.in, 0, n);
    int64_t at;
    const int64_t total = t.scan(sh, &at);
    t.store(s.out, 0, n, at);
    if (threadIdx.x == 0) s.out[n] = total;
}

__global__ __launch_bounds__(kScanThreads) void k_bm_scan_sums(BlockScans all, int64_t n, int64_t* sums) {
    __shared__ int64_t sh[kScanThreads / 64];
    TileScan t;
    t.load(all.s[blockIdx.y].in, (int64_t)blockIdx.x * kScanTile, n);
    int64_t at;
    const int64_t total = t.scan(sh, &at);
    if (threadIdx.x == 0) sums[blockIdx.y * (int64_t)gridDim.x + blockIdx.x] = total;
}

// (each workgroup adds up the tiles before its own: 512 for 2^22 rows, 1,300 for the
// 10^7 rows of 4,096 batch members)
__global__ __launch_bounds__(kScanThreads) void k_bm_scan_apply(BlockScans all, int64_t n, const int64_t* sums) {
    __shared__ int64_t sh[kScanThreads / 64];
    const BlockScan s = all.s[blockIdx.y];
    sums += blockIdx.y * (int64_t)gridDim.x;
    int64_t part = 0;
    for (int i = threadIdx.x; i < (int)blockIdx.x; i += kScanThreads) part += sums[i];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) part += __shfl_xor(part, d, 64);
    if (lane() == 0) sh[threadIdx.x >> 6] = part;
    __syncthreads();
    int64_t carry = 0;
    for (int w = 0; w < kScanThreads / 64; ++w) carry += sh[w];
    __syncthreads();
    TileScan t;
    const int64_t t0 = (int64_t)blockIdx.x * kScanTile;
    t.load(s.in, t0, n);
    int64_t at;
    const int64_t total = t.scan(sh, &at);
    t.store(s.out, t0, n, carry + at);
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) s.out[n] = carry + total;
}

namespace {
// to memory that the host may read
__device__ __forceinline__ void put_host(void* dst, const void* src, int64_t bytes, int64_t i, int64_t step) {
    for (; i < bytes / 4; i += step)
        __hip_atomic_store((uint32_t*)dst + i, ((const uint32_t*)src)[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
}  // namespace

// What the host waits for: control words, totals, statistics.
__global__ __launch_bounds__(kThreads) void k_bm_status(BlockArgs a, int32_t nj, const int64_t* u_total,
                                                        const int64_t* l_total, const int64_t* s_total,
                                                        BlockStatus* out, JobStats* js) {
    const int t = threadIdx.x;
    put_host(out->ctl, a.ctl, sizeof(out->ctl), t, kThreads);
    if (u_total) put_host(&out->nnz_u, u_total, 8, t, kThreads);
    if (l_total) put_host(&out->nnz_l, l_total, 8, t, kThreads);
    if (s_total) put_host(&out->nsuper, s_total, 8, t, kThreads);
    put_host(js, a.jstats, (int64_t)sizeof(JobStats) * nj, t, kThreads);
    __threadfence_system();
}

// What is left once rows and columns are written: supernodes from their starts
// and the starts' sums, each matrix's own pointers, pointer values at the
// matrices' ends and the statistics for the host.
__global__ __launch_bounds__(256) void k_bm_finish(BlockArgs a, BlockFinish f) {
    const int64_t i0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t r = i0; r < f.nrows; r += step) {
        const int32_t j = a.blk_job ? f.row_job[r] : 0;
        const int64_t b = a.jobs[j].row_base;
        if (f.supno) {
            const int64_t k = f.start_scan[r];  // supernode starts before r, all matrices
            const int32_t start = f.is_start[r];
            if (start) f.xsup[k + j] = (int32_t)(r - b);
            f.supno[r] = (int32_t)(k + start - 1 - f.start_scan[b]);
        }
        if (f.u_loc) {
            f.u_loc[r + j] = f.u_ptr[r] - f.u_ptr[b];
            f.l_loc[r + j] = f.l_ptr[r] - f.l_ptr[b];
        }
    }
    for (int64_t j = i0; j <= f.nj; j += step) {
        const int64_t b = j < f.nj ? a.jobs[j].row_base : f.nrows;
        const int64_t v[3] = {f.u_ptr[b], f.l_ptr[b], f.supno ? f.start_scan[b] : 0};
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (f.bounds) put_host(&f.bounds[k * (int64_t)(f.nj + 1) + j], &v[k], 8, 0, 1);
        if (j == f.nj) break;
        const int32_t n = a.jobs[j].n;
        if (f.supno) f.xsup[f.start_scan[b + n] + j] = n;
        if (f.u_loc) {
            f.u_loc[b + n + j] = f.u_ptr[b + n] - v[0];
            f.l_loc[b + n + j] = f.l_ptr[b + n] - v[1];
        }
    }
    if (f.js) put_host(f.js, a.jstats, (int64_t)sizeof(JobStats) * f.nj, i0, step);
    // (the others' fence would write the whole L2 back: 250 us on 10^6 rows, not 14)
    if (i0 <= f.nj * (int64_t)(sizeof(JobStats) / 4)) __threadfence_system();
}

// ------------------------------------------------------------------ launches

// Several matrices: blocks with the same local index are taken together, so
// that the chains of all matrices advance side by side.
__global__ void k_bm_tables(const Job* jobs, const int32_t* ord, const int64_t* cum, int32_t max_blocks,
                            int32_t nblocks, int32_t* items, int32_t* blk_job) {
    for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < nblocks; i += gridDim.x * blockDim.x) {
        int32_t lo = 0, hi = max_blocks - 1;
        while (lo < hi) {
            const int32_t mid = (lo + hi + 1) >> 1;
            if (cum[mid] <= i) lo = mid;
            else hi = mid - 1;
        }
        const int32_t j = ord[i - cum[lo]];
        const int32_t b = (int32_t)jobs[j].item_base + lo;
        items[i] = b;
        blk_job[b] = j;
    }
}

hipError_t launch_block_tables(const Job* jobs, const int32_t* ord, const int64_t* cum, int32_t max_blocks,
                               int32_t nblocks, int32_t* items, int32_t* blk_job, hipStream_t st) {
    if (nblocks <= 0) return hipSuccess;
    const unsigned g = (unsigned)std::min<int64_t>((nblocks + 255) / 256, 1024);
    hipLaunchKernelGGL(k_bm_tables, dim3(g), dim3(256), 0, st, jobs, ord, cum, max_blocks, nblocks, items, blk_job);
    return hipGetLastError();
}

namespace {
using FactorKernel = void (*)(BlockArgs);
FactorKernel factor_kernel(int waves) {
    return waves >= 8 ? k_bm_factor<8> : k_bm_factor<4>;
}
}  // namespace

int32_t block_resident_groups(int cus, int waves, int bit_words) {
    int blocks = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, factor_kernel(waves), 64 * waves,
                                                     (size_t)bit_words * 40) != hipSuccess ||
        blocks <= 0) {
        (void)hipGetLastError();
        blocks = 1;
    }
    return blocks * cus;
}

hipError_t launch_block_factor(const BlockArgs& a, hipStream_t st) {
    if (a.nblocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(factor_kernel(a.waves), dim3((unsigned)a.nslots), dim3((unsigned)(64 * a.waves)),
                       (size_t)a.bit_words * 40, st, a);
    return hipGetLastError();
}

hipError_t launch_block_counts(const BlockArgs& a, const BlockCols& c, int32_t* col_cnt, int64_t max_super,
                               int32_t* is_start, hipStream_t st) {
    if (a.nblocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_bm_count, dim3((unsigned)a.nblocks), dim3(kThreads), 0, st, a, c);
    hipLaunchKernelGGL(k_bm_lists, dim3((unsigned)a.nblocks), dim3(64), (size_t)a.bit_words * 12 + 8, st, a, c,
                       col_cnt, max_super, is_start);
    return hipGetLastError();
}

int64_t block_scan_tiles(int64_t n) { return (n + kScanTile - 1) / kScanTile; }

hipError_t launch_block_scan(const BlockScan* s, int count, int64_t n, int64_t* scratch, hipStream_t st) {
    BlockScans all{};
    for (int i = 0; i < count; ++i) all.s[i] = s[i];
    if (n <= kScanOne) {
        hipLaunchKernelGGL(k_bm_scan_one, dim3((unsigned)count), dim3(kScanThreads), 0, st, all, n);
        return hipGetLastError();
    }
    const int64_t nt = block_scan_tiles(n);
    hipLaunchKernelGGL(k_bm_scan_sums, dim3((unsigned)nt, (unsigned)count), dim3(kScanThreads), 0, st, all, n, scratch);
    hipLaunchKernelGGL(k_bm_scan_apply, dim3((unsigned)nt, (unsigned)count), dim3(kScanThreads), 0, st, all, n,
                       scratch);
    return hipGetLastError();
}

hipError_t launch_block_status(const BlockArgs& a, int32_t nj, const int64_t* u_total, const int64_t* l_total,
                               const int64_t* s_total, BlockStatus* out, JobStats* js, hipStream_t st) {
    hipLaunchKernelGGL(k_bm_status, dim3(1), dim3(kThreads), 0, st, a, nj, u_total, l_total, s_total, out, js);
    return hipGetLastError();
}

hipError_t launch_block_finish(const BlockArgs& a, const BlockFinish& f, hipStream_t st) {
    const unsigned g = (unsigned)std::min<int64_t>((f.nrows + f.nj + 1 + 255) / 256, 4096);
    hipLaunchKernelGGL(k_bm_finish, dim3(std::max(g, 1u)), dim3(256), 0, st, a, f);
    return hipGetLastError();
}

hipError_t launch_block_emit(const BlockArgs& a, const BlockCols& c, const int64_t* u_ptr, int32_t* u_idx,
                             const int64_t* l_ptr, int32_t* l_idx, bool l_csr, hipStream_t st) {
    if (a.nblocks <= 0) return hipSuccess;
    static_assert(kThreads / 64 == 4, "a workgroup takes the reach counts of four blocks");
    const dim3 grid(9u * (unsigned)((a.nblocks + 3) / 4));
    // Tiles for waiting blocks: eight keep five workgroups on a CU, which one
    // matrix wants (1000^2 9-point: 638 us with eight, 704 with twelve); among
    // many matrices some block needs more, and finishing it afterwards costs the
    // launch of 220 us (512 batch members: 942 in all with eight, 733 with twelve)
    const auto kernel = a.blk_job ? (l_csr ? k_bm_emit<true, 12> : k_bm_emit<false, 12>)
                                  : (l_csr ? k_bm_emit<true, 8> : k_bm_emit<false, 8>);
    hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, st, a, c, u_ptr, u_idx, l_ptr, l_idx);
    // (as many as there are slots: 10^6 rows coupled two by two at random, where every
    // block comes here, took 24 ms with 256 workgroups and a tile at a time, now 2.3)
    hipLaunchKernelGGL(k_bm_reach_big, dim3((unsigned)a.nslots), dim3(64 * kBigWaves), (size_t)a.bit_words * 16, st, a,
                       c);
    return hipGetLastError();
}

}  // namespace gsofa
