// Exact decoding with bounded predecessor scans (gfx950).
//
// A step needs, for every destination j, the first maximum over i of
// fl(delta_i + log A(i, j)).  With cm_j = max_i log A(i, j), a predecessor
// whose fl(delta_i + cm_j) is below the best candidate found so far cannot
// attain the maximum (float addition is monotone), so scanning predecessors
// from the largest delta downwards may stop as soon as an upper bound u of
// the deltas not yet scanned gives fl(u + cm_j) < best_j.  The stop is exact:
// scores, backpointers and ties are those of the full scan.  Where scores
// spread over more than a few units (any informative emission) a small part
// of the K predecessors is read: about 160 of 1024 rows of log A per 64
// columns with Dirichlet(0.1) transitions and N(0, 2^2) emissions, 8 of 256
// for a CRF's.
//
// The decreasing order comes in kTiers lists of states, by how far their
// scores lie below the maximum; the distances follow what the last steps
// needed.  States below the last list are scanned only when the bound still
// calls for them.
//
// FILTER: a wave with its own group (as many sequences as CUs, K > 512) is
// bound by the log A rows it reads from L2 and by the two instructions a
// candidate takes, so it first drops listed states by a closer bound: with
// r_i = max_{j in H} (log A(i, j) - cm_j) over a half group H of 32 columns
// (rounded up to float16; in LDS), delta_i + log A(i, j) <= (delta_i + r_i) +
// cm_j, and states with fl(delta_i + r_i) < h lose where fl(h + cm_j) <
// best_j.  h follows what the half group's last steps needed; where the
// results do not close the bound it takes h from them and reads the rest:
// the listed states from the new h on, and of the states on no list (a bound is
// no larger than its state's score) those that may still win.  Of
// K = 1024 with Dirichlet(0.1) transitions a half group then reads about 65
// rows of 128 bytes instead of 200 of 256: 256 sequences, T ~ U[500, 8000],
// FLASH P = 64: 111.5 -> 88.3 ms.  Where several waves share a group (teams)
// the filter's own steps take longer than the rows it saves (K = 512, one
// sequence: 2.0 -> 2.6 ms; 64 sequences of K = 1000: 13.3 -> 17.3 ms).
//
// Work division.  A team of M blocks decodes one task (a vanilla pass, a FLASH
// root, a FLASH segment); each block owns up to kTeamGroups groups of 64
// columns.  After a step each group's wave publishes its scores as 64-bit
// words {score, tracked division state, step tag} with device-scope stores;
// every block polls the words of the whole row, so data and synchronisation
// are the same transfer (about 1000 clocks between any two CUs, on one XCD
// or two; a barrier and a read would be two such trips).  There is no
// grid-wide step: teams take tasks from a queue (longest roots first) and a
// finished FLASH pass appends its segments.  The blocks of a team follow each
// other in the grid, hence sit on different XCDs, so an XCD reads only its
// blocks' columns of log A and its L2 holds them.
//
// Measured against the lock-step engine (a global step of 15 to 28 us for all
// rows): K = 512 Erdos-Renyi graph, T = 512, FLASH P = 16: 7.1 -> 2.0 ms; 64
// sequences, K = 1000, T ~ U[100, 2000], vanilla: 34.6 -> 13.3 ms; 256
// sequences, K = 1024, T ~ U[500, 8000], FLASH P = 64: 244 -> 112 (now 88) ms;
// K = 16384, T = 512, vanilla: 102 -> 24.5 ms; K = 5001, T = 777, FLASH
// P = 16: 39.3 -> 16.7 ms.
#include <float.h>

#include "fv_device.h"

namespace fv {

constexpr int kTiers = 3;
// FILTER: reach of the near and the far list in distances that the block's
// groups needed, of h in those that the half group needed, and the weight of
// a new one (swept: 1.0 / 1.6 / 1.1 / 0.3 takes 2% longer, h at 0.9 needs the
// second reading in 78% instead of 35% of the steps and takes 20% longer)
constexpr float kNear = 0.9f, kFar = 1.4f, kHalf = 1.15f, kEma = 0.2f;
// Where the bound does not prune, the engine's step, which costs the same
// whatever the scores, is the shorter one, and a pass is left to it: a vanilla
// pass or a root that reads more than 3 K / 4 rows a step (FILTER; 3 K are free;
// all K rows: 37 us a step, the engine's for 256 sequences of K = 1024 24 to 30),
// any pass that reads more than K / 32 rows a step outside the first lists (FAR;
// K / 8 are free, 16 K to a segment, whose root kept within them; such a row takes
// 0.1 to 0.2 us, on the third list a quarter of that, an engine's step 30 to 200 us
// from K = 4096 to 16384).  Up to K = 512, and for a team of blocks whose lists
// have room for all states, reading every row is no slower than the engine, or
// little.
constexpr int32_t kQuitCap = 1 << 30;   // counted up to here
constexpr int32_t kBoundRetry = 77;   // sequence status: left to the lock-step engine
constexpr int kRowCap = 128;          // rows of a wave's lists (FILTER)

// A candidate and its predecessor as one float64 pattern: the float32 score
// in the high word, the state in the low word.  Finite scores and infinities
// are finite float64 patterns, ordered first by the score, so one v_max_f64
// per candidate keeps the maximum and where it came from, in any scan order.
// Equal scores are decided by the low word: the smaller one is the larger
// number for negative scores, the larger one for positive scores, so the
// state is stored as itself while scores are negative and complemented while
// they are positive.  A step that may have candidates of both signs, or zeros,
// decides it for each (`mixed`: two instructions more, and one that makes -0
// +0); `finish` handles columns of a sign that was not expected.
struct BoundEnt {
    int32_t lo;
    float v;
};
// a state, in a mixed step: as itself for a negative score, complemented for others
__device__ __forceinline__ int32_t by_sign(float score, int32_t i) { return i ^ ~(__float_as_int(score) >> 31); }
struct Mixed { static constexpr bool on = true; };
struct OneSign { static constexpr bool on = false; };

// KC: the largest K, LC: states a list holds, NB: steps whose emission rows
// are fetched, and backpointer rows stored, at once.  (Memory operations of a
// wave complete in order, so an emission load in flight holds back every
// log A row read after it for as long as HBM takes; in groups of NB rows that
// wait comes once every NB steps.)
template <int KC, int LC, int NB, bool TEAM, bool FILTER>
struct TeamLds {
    static constexpr int TC = KC < 64 * kTeamGroups ? KC : 64 * kTeamGroups;   // columns of a block, at most
    union {
        struct {
            BoundEnt list[FILTER ? 1 : kTiers][LC];   // scanned states, unordered
            BoundEnt rows[FILTER ? 16 : 1][2][FILTER ? kRowCap + 16 : 1];   // a wave's rows to read, by half of its group
            float eb[2][NB * TC];       // emission rows of the block's columns: in use, and coming
        };
        // backpointer rows being walked
        uint32_t walk[(8 * (FILTER ? 1 : kTiers) * LC + (FILTER ? 256 * (kRowCap + 16) : 16) + 8 * NB * TC) / 4];
    };
    unsigned long long part[FILTER ? 1 : TC];   // order keys of partial maxima
    uint32_t rb[FILTER ? 16 * KC : 1];   // [groups, Kp] row bounds of both halves
    float cm[TC];                  // column maxima; NaN where no scan is ever needed
    float cm_lo, cm_hi;            // the smallest and the largest of them
    uint16_t pb[2][NB * TC];       // backpointer rows: being made, being stored
    uint16_t anc[TEAM ? 1 : 2][KC];    // tracked division state of every state
    float x[TEAM ? 1 : 2][TEAM ? 1 : KC];   // a single block's scores, by step parity
    uint32_t rmax[2];                  // and the order key of the largest
    int32_t cnt[2][4];                 // by step parity: states on the lists, any finite one on none
    uint32_t need[2];                  // by step parity: the distance the groups needed (bits of a float >= 0)
    unsigned long long key;
    int32_t sv[8];
};

// ---------------------------------------------------------------- wave operations
// v, hidden from the compiler: addresses made from it are formed where they are
// used, not kept in registers across the steps
__device__ __forceinline__ int32_t fresh(int32_t v) {
    asm volatile("" : "+v"(v));
    return v;
}
// merge_group for two half groups of 32 columns (lanes equal modulo 8 scanned the
// same four columns of either): lane l ends with column 4 (l mod 8) + l / 16 of
// half (l / 8) mod 2.
__device__ __forceinline__ double merge_halves(const double (&b0)[4], const double (&b1)[4]) {
    const double m0 = merge_group(b0), m1 = merge_group(b1);
    const bool up = threadIdx.x & 8;
    const double keep = up ? m1 : m0, give = up ? m0 : m1;
    const int32_t lo = __builtin_amdgcn_update_dpp(0, __double2loint(give), 0x128, 0xf, 0xf, false);   // row_ror:8
    const int32_t hi = __builtin_amdgcn_update_dpp(0, __double2hiint(give), 0x128, 0xf, 0xf, false);
    return max64(keep, __hiloint2double(hi, lo));
}
// largest of the lanes of a half (lanes with equal bit 3), in each of them
__device__ __forceinline__ uint32_t half_max(uint32_t v) {
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int32_t)v, 0xb1, 0xf, 0xf, false));    // quad_perm: 1, 0, 3, 2
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int32_t)v, 0x4e, 0xf, 0xf, false));    // quad_perm: 2, 3, 0, 1
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int32_t)v, 0x141, 0xf, 0xf, false));   // row_half_mirror
    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = max((uint32_t)a[0], (uint32_t)a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return max((uint32_t)b[0], (uint32_t)b[1]);
}
// x + the float16 in the low (high) half of r
__device__ __forceinline__ float add_lo16(float x, uint32_t r) {
    float s;
    asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel_hi:[1,0,0]" : "=v"(s) : "v"(r), "v"(x));
    return s;
}
__device__ __forceinline__ float add_hi16(float x, uint32_t r) {
    float s;
    asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(s) : "v"(r), "v"(x));
    return s;
}
__device__ __forceinline__ uint32_t score_key(float v) {
    const uint32_t b = __float_as_uint(v);
    return b ^ ((uint32_t)((int32_t)b >> 31) | 0x80000000u);
}
__device__ __forceinline__ float score_of_key(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}
// a candidate pattern as an unsigned number of the same order, and back
__device__ __forceinline__ unsigned long long pattern_key(double b) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(b);
    return u ^ ((unsigned long long)((long long)u >> 63) | 0x8000000000000000ull);
}
__device__ __forceinline__ double pattern_of_key(unsigned long long k) {
    return __longlong_as_double((long long)(k ^ ((unsigned long long)((long long)~k >> 63) | 0x8000000000000000ull)));
}
__device__ __forceinline__ void take1(float& best, int32_t& arg, float c, int32_t i) {
    const bool up = c > best || (c == best && i < arg);
    best = up ? c : best;
    arg = up ? i : arg;
}

// Exchange buffer of a team (device-scope accesses only): the words of the
// row by step parity, the groups' maxima by step parity, the task descriptor
// and each block's completed-task counter.
struct TeamBuf {
    unsigned long long* x[2];
    unsigned long long* g[2];
    unsigned long long* desc;
    unsigned long long* done;
};
__device__ __forceinline__ TeamBuf team_buf(char* base, int32_t Kp, int32_t M) {
    unsigned long long* w = reinterpret_cast<unsigned long long*>(base);
    if (M == 1) Kp = 0;   // a single block exchanges no scores
    const int32_t ng = (Kp / 64 + 15) & -16;
    TeamBuf b;
    b.x[0] = w;
    b.x[1] = w + Kp;
    b.g[0] = w + 2 * (int64_t)Kp;
    b.g[1] = b.g[0] + ng;
    b.desc = b.g[1] + ng;
    b.done = b.desc + 16;
    return b;
}
// score | tracked division state | stop mark | step tag (15 bits)
constexpr uint32_t kTagBits = 0x7fff;
__device__ __forceinline__ unsigned long long team_word(float v, uint32_t mid, uint32_t stop, uint32_t tag) {
    return (unsigned long long)__float_as_uint(v) | ((unsigned long long)(mid | stop << 16 | tag << 17) << 32);
}

enum : int32_t { BM_VANILLA = 0, BM_DIV = 1, BM_LEAF = 2 };

// W: waves of a block.  MIX: steps that may have results of both signs scan so.
template <int KC, int LC, int NB, bool TEAM, int W, bool FILTER, bool MIX>
__device__ __forceinline__ void team_decode(cargs_t& a) {
    constexpr int kTThreads = 64 * W;
    constexpr int TC = TeamLds<KC, LC, NB, TEAM, FILTER>::TC;
    constexpr int UN = KC <= 256 ? 16 : 8;   // list entries of a unit of work
    constexpr int UL = UN / 4;               // 16 lanes across 64 columns: 4 entries side by side
    // long rows: the groups' maxima are polled first, the words then read once
    constexpr bool GATE = TEAM && KC > 4096;
    // passes that the bound does not prune are left to the engine: ones that read
    // nearly all listed states (FILTER), or many on no list for want of room (FAR)
    constexpr bool FAR = TEAM && LC < KC;
    constexpr bool QUIT = FAR || FILTER;
    __shared__ __align__(16) TeamLds<KC, LC, NB, TEAM, FILTER> s;
    const int32_t tid = threadIdx.x, lane = tid & 63, wv = uni(tid >> 6);
    const int32_t K = a.K, Kp = a.Kp, M = a.b_team;
    if (Kp > KC) return;
    const int32_t team = blockIdx.x / M, member = blockIdx.x - team * M;
    const int32_t ngt = Kp / 64;                                  // groups of the row,
    const int32_t gb = ngt * member / M;                          // this block's first one
    const int32_t ngl = ngt * (member + 1) / M - gb;              // and their number
    const int32_t cb = gb * 64, cn = min(K, cb + ngl * 64) - cb;  // its columns
    const TeamBuf tb = team_buf(a.bxch + (int64_t)team * a.bxch_bytes, Kp, M);
    typedef __attribute__((address_space(1))) const char gchar_t;
    typedef float vec_t __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(1))) const vec_t gvec_t;
    gchar_t* const A = reinterpret_cast<gchar_t*>(reinterpret_cast<uint64_t>(a.Acol));
    const int32_t pitch = Kp * 4;
    EngineState* const st = a.st;
    const int32_t n_roots = st->q_tail0;
    // waves of a group: all of them for a single group, ..., one where there
    // are more groups than half the waves
    int32_t wpg = W;
    if (FILTER) wpg = 1;
    while (wpg > 1 && wpg * ngl > W) wpg >>= 1;
    const int32_t g = wv / wpg, sub = wv - g * wpg;               // this wave's group and share of it
    const int32_t lc4 = 4 * (lane & 15);
    // the column (in the block) a lane ends with
    const int32_t jl = g * 64 + (FILTER ? 4 * (lane & 8) + 4 * (lane & 7) : lc4) + (lane >> 4);
    const bool active = g < ngl;
    for (int32_t k = tid; k < TC; k += kTThreads) {
        const float c = k < cn ? score_of_key(a.cmax[cb + k]) : -INFINITY;
        s.cm[k] = c > -INFINITY ? c : __builtin_nanf("");
    }
    if constexpr (FILTER)
        for (int32_t k = tid; k < ngl * Kp; k += kTThreads) s.rb[k] = a.rowb[k];
    float cm_lo = 0.0f, cm_hi = 0.0f;
    if constexpr (MIX) {
        __syncthreads();
        if (wv == 0) {
            uint32_t lo = 0, hi = 0;
            for (int32_t k = lane; k < cn; k += 64) {
                const float c = s.cm[k];
                if (!(c == c)) continue;
                lo = max(lo, score_key(-c));
                hi = max(hi, score_key(c));
            }
            lo = wave_max(lo);
            hi = wave_max(hi);
            if (lane == 0) {
                s.cm_lo = -score_of_key(lo);
                s.cm_hi = score_of_key(hi);
            }
        }
        __syncthreads();
        cm_lo = __int_as_float(uni(__float_as_int(s.cm_lo)));
        cm_hi = __int_as_float(uni(__float_as_int(s.cm_hi)));
    }
    const double none = __hiloint2double((int32_t)0xff800000u, 0);
    float G = 8.0f, G1 = 16.0f;   // distance below the maximum that the scans are expected to need
    float F = 8.0f, F1 = 16.0f;   // and (FILTER) those of the lane's half group
    uint32_t epoch = 1;        // tag of the scores of a task's first position
    unsigned long long task_no = 0;
    for (;;) {
        // ---- next task: the team's first block takes it and tells the others
        ++task_no;
        if (tid == 0) {
            unsigned long long w0 = 0, w1 = 0, w2 = 0;
            int32_t got = 0;
            if (member == 0) {
                const int32_t err = ld_c(&st->error);
                const uint32_t h =
                    __hip_atomic_fetch_add(&st->bq_head, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                got = h < (uint32_t)n_roots && !err ? 1 : 0;
                // spawned tasks: wait for the publication of this ticket, or for
                // the end of every task that could still spawn (each is running
                // on some team, so the wait ends)
                if (!got && !err && a.method == FV_FLASH) {
                    for (int64_t turn = 0;; ++turn) {
                        const uint32_t live = ld_c(&st->bq_live);
                        if (ld_c(&st->bq_pub) > h) { got = 1; break; }
                        if (live == 0) {
                            got = ld_c(&st->bq_pub) > h ? 1 : 0;
                            break;
                        }
                        if (wait_over(a, turn, true)) break;
                        __builtin_amdgcn_s_sleep(16);
                    }
                }
                if (got) {
                    const unsigned long long* p = reinterpret_cast<const unsigned long long*>(a.queue + h);
                    w0 = ld_c(p);
                    w1 = ld_c(p + 1);
                    const int32_t tm = (int32_t)w1, tn = (int32_t)(w1 >> 32);
                    if ((int32_t)(w0 >> 32) == KIND_SUB) {
                        const SeqInfo& sq = a.seqs[(int32_t)w0];
                        const int32_t qn = clampi(ld_c(sq.path + tn), K);
                        const int32_t qp = tm > 0 ? clampi(ld_c(sq.path + tm - 1), K) : 0;
                        const float al = tm > 0 ? ld_cf(a.alpha_at + sq.alpha_off + tm - 1) : 0.0f;
                        w2 = (unsigned long long)__float_as_uint(al) | ((unsigned long long)(qn | qp << 16) << 32);
                    }
                }
                if (M > 1) {
                    st_c(tb.desc + 1, w0);
                    st_c(tb.desc + 2, w1);
                    st_c(tb.desc + 3, w2);
                    st_c(tb.desc + 4, (unsigned long long)got);
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                    __builtin_amdgcn_s_waitcnt(0);
                    st_c(tb.desc, task_no);
                }
            } else {
                for (int64_t turn = 0;; ++turn) {
                    if (ld_c(tb.desc) == task_no) { got = 1; break; }
                    if (wait_over(a, turn, true)) break;
                    __builtin_amdgcn_s_sleep(1);
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                if (got) {
                    w0 = ld_c(tb.desc + 1);
                    w1 = ld_c(tb.desc + 2);
                    w2 = ld_c(tb.desc + 3);
                    got = (int32_t)ld_c(tb.desc + 4);
                }
            }
            s.sv[0] = got;
            s.sv[1] = (int32_t)w0;
            s.sv[2] = (int32_t)(w0 >> 32);
            s.sv[3] = (int32_t)w1;
            s.sv[4] = (int32_t)(w1 >> 32);
            s.sv[5] = (int32_t)w2;
            s.sv[6] = (int32_t)(w2 >> 32);
            s.sv[7] = 0;
        }
        __syncthreads();
        if (!s.sv[0]) break;
        const int32_t seq = uni(s.sv[1]), kind = uni(s.sv[2]), m = uni(s.sv[3]), n = uni(s.sv[4]);
        const float alpha = __int_as_float(uni(s.sv[5]));
        const int32_t q_n = uni(s.sv[6]) & 0xffff, q_prev = (uint32_t)uni(s.sv[6]) >> 16;
        SeqInfo& sq = a.seqs[seq];
        const int32_t len = n - m + 1;
        int32_t mode = BM_VANILLA, w = 1;
        if (kind == KIND_ROOT) {
            mode = BM_DIV;
            w = sq.pp;
        } else if (kind == KIND_SUB) {
            mode = len <= a.b_leaf ? BM_LEAF : BM_DIV;
            w = mode == BM_DIV ? min(a.b_split, max(2, (len + a.b_leaf - 1) / a.b_leaf)) : 1;
        }
        // Rarely used addresses are formed where they are used (from a copy of
        // the sequence index the compiler cannot see through), not kept in
        // scalar registers across the steps.
        auto seq_info = [&]() -> SeqInfo& {
            int32_t q = seq;
            asm volatile("" : "+s"(q));
            return a.seqs[q];
        };
        auto scratch = [&]() {
            int32_t b = team;
            asm volatile("" : "+s"(b));
            return a.bscr + (int64_t)b * a.bscr_bytes;
        };
        // division copies: scores and links of w - 1 divisions, pitch Kp
        auto dsnap = [&]() {
            return kind == KIND_ROOT ? a.root_copy + seq_info().root_off * (int64_t)Kp
                                     : reinterpret_cast<float*>(scratch());
        };
        auto link = [&]() { return reinterpret_cast<int32_t*>(dsnap() + (int64_t)(w - 1) * Kp); };
        // backpointer rows: the sequence's table (row t), or the leaf's (row t - m - 1)
        const int32_t tab0 = mode == BM_VANILLA ? 0 : m + 1;
        uint16_t* const psi = a.psi16 + sq.psi_off;
        auto table = [&]() {
            return mode == BM_VANILLA ? psi : reinterpret_cast<uint16_t*>(scratch());
        };
        auto div_end = [&](int32_t k) { return m + (int32_t)((((int64_t)k + 1) * len - 1) / w); };
        const float* const lb = sq.log_b + cb;
        const int64_t ld = sq.ld;
        // emission rows t0 .. t0 + NB - 1 into LDS (no registers held); 64 columns a wave and instruction
        auto fetch = [&](int32_t half, int32_t t0) {
            typedef __attribute__((address_space(3))) void lvoid_t;
            typedef __attribute__((address_space(1))) const void gvoid_t;
            for (int32_t q = wv; q < ngl * NB; q += W) {
                const int32_t r = q % NB, c = q / NB;
                lvoid_t* dst = reinterpret_cast<lvoid_t*>((uint32_t)__builtin_amdgcn_readfirstlane(
                    (int32_t)(uintptr_t)&s.eb[half][r * TC + c * 64]));
                if (t0 + r <= n && c * 64 + lane < cn)
                    __builtin_amdgcn_global_load_lds(
                        reinterpret_cast<gvoid_t*>(
                            reinterpret_cast<uintptr_t>(lb + (int64_t)(t0 + r) * ld + c * 64 + lane)),
                        dst, 4, 0, 0);
            }
        };
        // the block's part of cnt finished backpointer rows t0 ..
        auto flush = [&](int32_t half, int32_t t0, int32_t cnt) {
            const uint16_t* const rows = s.pb[half];
            uint16_t* const dst = table() + (int64_t)(t0 - tab0) * K + cb;
            if (K & 1) {
                for (int32_t k = tid; k < cnt * TC; k += kTThreads) {
                    const int32_t c = k % TC;
                    if (c < cn) st_c(dst + (int64_t)(k / TC) * K + c, rows[k]);
                }
            } else {
                for (int32_t k = tid; k < cnt * (TC / 2); k += kTThreads) {
                    const int32_t c = 2 * (k % (TC / 2));
                    if (c < cn)
                        st_c(reinterpret_cast<uint32_t*>(dst + (int64_t)(k / (TC / 2)) * K + c),
                             reinterpret_cast<const uint32_t*>(rows)[k]);
                }
            }
        };
        if (n > m) fetch(0, m + 1);

        // ---- start vector: published under the task's first tag
        int32_t d_next = 0;
        int32_t e_next = mode == BM_DIV && w > 1 ? div_end(0) : -1, e_prev = -1;
        const int32_t e_first = e_next;
        uint32_t give_up = 0;      // this group's mark: the pass is left to the engine
        // rows of log A that the group read: listed ones (FILTER), in excess of what
        // a step may take, and ones on no list (FAR), which one wave reads by itself
        int32_t listed = 0, far = 0;
        auto publish = [&](int32_t t, float xn, int32_t mid) {
            const uint32_t tag = (epoch + (uint32_t)(t - m)) & kTagBits;
            const int32_t p = (int32_t)(epoch + (uint32_t)(t - m)) & 1;
            if constexpr (TEAM) {
                if (jl < cn) st_c(tb.x[p] + cb + jl, team_word(xn, (uint32_t)mid, give_up, tag));
            } else {
                s.x[p][jl] = xn;
                if (mode == BM_DIV) s.anc[p][jl] = (uint16_t)mid;
            }
            if constexpr (!TEAM || GATE) {
                const uint32_t mk = wave_max(score_key(xn));
                if (lane == 0) {
                    if constexpr (TEAM)
                        st_c(tb.g[p] + gb + g, (unsigned long long)mk | ((unsigned long long)give_up << 32) |
                                                   ((unsigned long long)tag << 48));
                    else atomicMax(&s.rmax[p], mk);
                }
            }
        };
        if (tid < 2) {
            s.rmax[tid] = s.need[tid] = 0;
            s.cnt[tid][0] = s.cnt[tid][1] = s.cnt[tid][2] = s.cnt[tid][3] = 0;
        }
        __syncthreads();
        if (active && sub == 0) {
            float x = -INFINITY;
            if (jl < cn) {
                const int32_t j = cb + jl;
                const float b = as_global(sq.log_b)[(int64_t)m * sq.ld + j];
                if (m > 0) x = (alpha + a.Acol[(int64_t)q_prev * Kp + j]) + b;
                else x = a.log_pi ? a.log_pi[j] + b : b;
                if (e_next == m) st_cf(dsnap() + j, x);
            }
            publish(m, x, 0);
        }
        if (e_next == m) {
            e_prev = m;
            d_next = 1;
            e_next = w > 2 ? div_end(1) : -1;
        }
        bool retry = false;
        int32_t made = len;   // positions whose scores the team published
        for (int32_t t = m + 1; t <= n; ++t) {
            const int32_t step = t - m - 1, row = step % NB, half = (step / NB) & 1, par = step & 1;
            const uint32_t tag = (epoch + (uint32_t)step) & kTagBits;
            const int32_t xp = (int32_t)(epoch + (uint32_t)step) & 1;
            if (row == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's rows of the half in use
            // ---- the previous scores and the largest of them
            constexpr int NS = KC / kTThreads;   // states of a thread
            constexpr int CN = NS < 4 ? NS : 4;
            unsigned long long v[CN];
            auto poll = [&](int32_t c) {   // words of states tid + c kTThreads, ...
                for (int64_t turn = 0;; ++turn) {
                    bool bad = false;
#pragma unroll
                    for (int k = 0; k < CN; ++k) {
                        const int32_t i = tid + (c + k) * kTThreads;
                        v[k] = (unsigned long long)(tag << 17) << 32 | 0xff800000u;
                        if (i < K) v[k] = ld_c(tb.x[xp] + i);
                    }
#pragma unroll
                    for (int k = 0; k < CN; ++k) bad = bad || (uint32_t)(v[k] >> 49) != tag;
                    if (__builtin_amdgcn_ballot_w64(bad) == 0 || wait_over(a, turn, false)) break;
                }
                if constexpr (FAR && !GATE) {
                    uint32_t stop = 0;
#pragma unroll
                    for (int k = 0; k < CN; ++k) stop |= (uint32_t)(v[k] >> 48) & 1;
                    if (stop) s.sv[7] = 1;
                }
            };
            if constexpr (TEAM && !GATE) {
                poll(0);
                uint32_t mk = 0;
#pragma unroll
                for (int k = 0; k < CN; ++k) mk = max(mk, score_key(__uint_as_float((uint32_t)v[k])));
                mk = wave_max(mk);
                if (lane == 0) atomicMax(&s.rmax[xp], mk);
            }
            if constexpr (GATE) {
                if (wv == 0) {   // one wave polls the groups' maxima: more would slow what they wait for
                    uint32_t mk = 0, stop = 0;
                    for (int32_t k0 = 0; k0 < ngt; k0 += 64) {
                        const bool in = k0 + lane < ngt;
                        unsigned long long q = 0;
                        for (int64_t turn = 0;; ++turn) {
                            if (in) q = ld_c(tb.g[xp] + k0 + lane);
                            if (__builtin_amdgcn_ballot_w64(in && (uint32_t)(q >> 48) != tag) == 0 ||
                                wait_over(a, turn, false))
                                break;
                        }
                        if (in) mk = max(mk, (uint32_t)q);
                        if (in) stop |= (uint32_t)(q >> 32) & 1;
                    }
                    mk = wave_max(mk);
                    if (lane == 0) s.rmax[xp] = mk;
                    if (stop) s.sv[7] = 1;
                }
            }
            __syncthreads();
            const float D = score_of_key((uint32_t)uni((int32_t)s.rmax[xp]));
            // a task's first step, from one state's scores, needs more than the others
            if (step > 0) {
                const float u = __uint_as_float((uint32_t)uni((int32_t)s.need[par]));
                if (step == 1) G1 = fmaxf(G1 + 0.5f * (u - G1), 1e-4f);
                else G = fmaxf(G + 0.25f * (u - G), 1e-4f);
            }
            const bool neg = D < 0.0f;
            // a step that may have results of both signs: none is above D + cm_hi, most are
            // above D - 4 G + cm_lo.  (All ones or 0, in scalar arithmetic: branches
            // here and at the result cost such kernels 4%.)
            int32_t mixm = 0;
            if constexpr (MIX)
                mixm = uni(-(((int32_t)neg & (int32_t)(D + cm_hi >= 0.0f)) |
                             ((int32_t)!neg & (int32_t)(D + cm_lo <= 4.0f * (step == 0 ? G1 : G)))));
            const bool mixed = mixm != 0, plain = MIX ? neg || mixed : neg;
            const int32_t flip = plain ? 0 : -1;   // stored states
            // ---- the lists
            // scores from which a state is on the first, second, third list: the
            // first holds what all groups are expected to need, or, where each
            // wave has its own group and looks at the bound, what most of them need
            float h0, h1, h2;
            for (int32_t go = 0;; ++go) {
                const float gx = (step == 0 ? G1 : G) * __int_as_float((127 - go) << 23);
                h0 = D - (FILTER ? kNear : (wpg > 1 || KC <= 256 ? 1.0f : 0.75f)) * gx;
                h1 = D - (FILTER ? kFar : (wpg > 1 || KC <= 256 ? 1.2f : 1.0f)) * gx;
                h2 = FILTER ? h1 : D - (GATE ? 1.4f : (wpg > 1 || KC <= 256 ? 1.7f : 1.35f)) * gx;
#pragma unroll
                for (int c = 0; c < NS; c += CN) {
                    if (c * kTThreads >= K) break;
                    float x[CN];
                    if constexpr (TEAM) {
                        if constexpr (GATE) poll(c);
#pragma unroll
                        for (int k = 0; k < CN; ++k) {
                            const int32_t i = tid + (c + k) * kTThreads;
                            x[k] = i < K ? __uint_as_float((uint32_t)v[k]) : -INFINITY;
                            if (i < K && mode == BM_DIV) s.anc[0][i] = (uint16_t)(v[k] >> 32);
                        }
                    } else {
#pragma unroll
                        for (int k = 0; k < CN; ++k) {
                            const int32_t i = tid + (c + k) * kTThreads;
                            x[k] = i < K ? s.x[xp][i] : -INFINITY;
                        }
                    }
#pragma unroll
                    for (int k = 0; k < CN; ++k) {
                        const bool fin = x[k] > -INFINITY;
                        const uint64_t c0 = __builtin_amdgcn_ballot_w64(fin && x[k] >= h0);
                        const uint64_t c1 = __builtin_amdgcn_ballot_w64(fin && x[k] >= h1);
                        const uint64_t c2 = __builtin_amdgcn_ballot_w64(fin && x[k] >= h2);
                        if (__builtin_amdgcn_ballot_w64(fin) & ~c2)
                            if (lane == 0) s.cnt[par][3] = 1;
                        if (c2 == 0) continue;
                        const int32_t n0 = __popcll(c0), n1 = __popcll(c1) - n0, n2 = __popcll(c2) - n0 - n1;
                        const int32_t add = lane == 0 ? n0 : (lane == 1 ? n1 : n2);
                        int32_t at = 0;
                        if (lane < kTiers) at = atomicAdd(&s.cnt[par][lane], add);
                        const int32_t a0 = __builtin_amdgcn_readlane(at, 0), a1 = __builtin_amdgcn_readlane(at, 1),
                                      a2 = __builtin_amdgcn_readlane(at, 2);
                        const int32_t l = x[k] >= h0 ? 0 : (x[k] >= h1 ? 1 : 2);
                        const uint64_t my = l == 0 ? c0 : (l == 1 ? c1 & ~c0 : c2 & ~c1);
                        const int32_t pos = (l == 0 ? a0 : (l == 1 ? a1 : a2)) +
                                            __builtin_amdgcn_mbcnt_hi((uint32_t)(my >> 32),
                                                                      __builtin_amdgcn_mbcnt_lo((uint32_t)my, 0));
                        if (fin && x[k] >= h2 && (LC >= KC || pos < LC))
                            s.list[FILTER ? 0 : l][FILTER && l ? LC - 1 - pos : pos] =
                                BoundEnt{(tid + (c + k) * kTThreads) ^ flip, x[k]};
                    }
                }
                if (LC >= KC || go == 8) break;
                // a first list beyond its room: a shorter reach
                __syncthreads();
                const bool fits = s.cnt[par][0] <= LC;
                __syncthreads();
                if (fits) break;
                if (tid < 4) s.cnt[par][tid] = 0;
                __syncthreads();
            }
            if (wpg > 1)
                for (int32_t k = tid; k < TC; k += kTThreads) s.part[k] = 0;
            if (tid == 0) s.need[par ^ 1] = 0;   // every wave is past its reads of the step before
            if (tid == 1) s.rmax[xp ^ 1] = 0;
            const bool quit = QUIT && s.sv[7] != 0;
            __syncthreads();
            if (quit) {   // the bound does not prune these scores, and the engine's step costs the
                retry = true;                   // same whatever they are
                made = step + 1;                // (every block stops here: the mark came with this row)
                break;
            }
            if (row == 0) {
                fetch(half ^ 1, t + NB);   // the readers of that half are past the barrier
                if (mode != BM_DIV && step > 0) flush(half ^ 1, t - NB, NB);
            }
            if (tid < 4) s.cnt[par ^ 1][tid] = 0;
            // complete lists, and whether any finite score lies below them
            int32_t lists = kTiers;
            const int4 cn4 = *reinterpret_cast<const int4*>(s.cnt[par]);
            if constexpr (FILTER) lists = 2;
            if constexpr (LC < KC) lists = uni(cn4.x) > LC ? 0 : (uni(cn4.y) > LC ? 1 : (uni(cn4.z) > LC ? 2 : 3));
            const bool outside = uni(cn4.w) != 0 || (!FILTER && lists < kTiers);
            // above every score outside the first n lists
            auto below = [&](int32_t n) { return n == 0 ? INFINITY : (n == 1 ? h0 : (n == 2 ? h1 : h2)); };
            // ---- scan of the groups' columns
            const int32_t mul = plain ? pitch : -pitch;   // row offset of a list entry from its stored form
            const int32_t add0 = cb * 4 - (plain ? 0 : pitch);
            // entries of a list of cnt from `at` on (the last one repeated past its end)
            auto load = [&](auto& en, auto& av, const BoundEnt* list, int32_t at, int32_t cnt, int32_t add) {
                constexpr int N = sizeof(en) / sizeof(en[0]);
#pragma unroll
                for (int u = 0; u < N; ++u) en[u] = list[min(at + (lane >> 4) + u * 4, cnt - 1)];
#pragma unroll
                for (int u = 0; u < N; ++u)
                    av[u] = *reinterpret_cast<gvec_t*>(A + (uint32_t)(__mul24(en[u].lo, mul) + add));
                __builtin_amdgcn_sched_barrier(0);   // every load is issued before the next wait
            };
            auto scan = [&](auto mx, double (&best)[4], const auto& en, const auto& av) {
                constexpr int N = sizeof(en) / sizeof(en[0]);
#pragma unroll
                for (int u = 0; u < N; ++u)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        float x = en[u].v + av[u][c];
                        if (mx.on) x += 0.0f;   // -0: +0
                        best[c] = max64(best[c], __hiloint2double(__float_as_int(x), mx.on ? by_sign(x, en[u].lo) : en[u].lo));
                    }
            };
            // the pattern of a candidate x of state i, and the state of a pattern
            auto pattern = [&](float x, int32_t i) {
                if (mixed) x += 0.0f;
                return __hiloint2double(__float_as_int(x), i ^ flip ^ (mixm & ~(__float_as_int(x) >> 31)));
            };
            auto state_of = [&](double b) {
                return __double2loint(b) ^ flip ^ (mixm & ~(__double2hiint(b) >> 31));
            };
            auto score_at = [&](int32_t i) {
                if constexpr (TEAM) return __uint_as_float((uint32_t)ld_c(tb.x[xp] + i));
                else return s.x[xp][i];
            };
            // the best candidate of this lane's column among the states that score
            // from thr up to (not including) top_of
            auto scan_states = [&](float thr, float top_of, float& f, int32_t& q) {
                f = -INFINITY;
                q = 0;
                gfloat_t* const ak = as_global(a.Acol) + fresh(cb + jl);
#pragma unroll 1
                for (int32_t c0 = 0; c0 < K; c0 += 256) {
                    float xo[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) xo[u] = score_at(min(c0 + u * 64 + fresh(lane), K - 1));
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const bool in = c0 + u * 64 + lane < K && xo[u] >= thr && xo[u] < top_of && xo[u] > -INFINITY;
                        uint64_t mask = __builtin_amdgcn_ballot_w64(in);
                        while (mask) {   // four rows in flight
                            int32_t r[4];
                            float v[4];
#pragma unroll
                            for (int w = 0; w < 4; ++w) {
                                r[w] = mask ? (int32_t)__builtin_ctzll(mask) : r[w ? w - 1 : 0];
                                mask &= mask - 1;
                                v[w] = ak[(uint32_t)(c0 + u * 64 + r[w]) * (uint32_t)Kp];
                            }
#pragma unroll
                            for (int w = 0; w < 4; ++w)
                                take1(f, q, __int_as_float(__builtin_amdgcn_readlane(__float_as_int(xo[u]), r[w])) + v[w],
                                      c0 + u * 64 + r[w]);
                        }
                    }
                }
            };
            // the maxima top, of the states that score from thr on, with those below:
            // thr becomes a score below which none can win (checked, not derived: the
            // subtraction is rounded)
            auto beyond = [&](double top, float& thr) {
                const float bs = __int_as_float(__double2hiint(top)), cm = s.cm[jl], top_of = thr;
                const float nd = D - (bs - cm);
                const float lim = __uint_as_float(wave_max(nd > 0.0f ? __float_as_uint(nd) : 0u));
                thr = D - lim * 1.001f - 1e-6f * fabsf(D);
                if (__builtin_amdgcn_ballot_w64(cm == cm && !(thr + cm < bs))) thr = -FLT_MAX;
                float f;
                int32_t q;
                scan_states(thr, top_of, f, q);
                return max64(top, pattern(f, q));
            };
            // the result of this wave's group: the sign check, the score, the state
            // and the division state.  Scanned were (FILTER) the states from thr on
            // that may win, or the first `done` lists and, out, the states outside
            // them, whose best is fo of qo.
            auto finish = [&](double top, float thr, int32_t done, bool out, float fo, int32_t qo) {
                // scores of the other sign, or zeros, where the low word does not
                // order equal candidates: compare by value and state.  (A mixed
                // step's is in order; a zero gets its own sign back.)
                const float b0 = __int_as_float(__double2hiint(top));
                bool odd;
                if constexpr (MIX) {
                    const int32_t negm = uni(-(int32_t)neg);
                    const float odd_lo = __int_as_float(flip & __float_as_int(-FLT_MAX));
                    const float odd_hi = __int_as_float(negm & ~mixm & __float_as_int(INFINITY));
                    odd = b0 >= odd_lo && b0 <= odd_hi;
                } else {
                    odd = neg ? b0 >= 0.0f : (b0 <= 0.0f && b0 > -INFINITY);
                }
                if (__builtin_amdgcn_ballot_w64(odd)) {
                    float f = -INFINITY;
                    int32_t q = 0;
                    if (mixed) {
                        f = b0;
                        q = state_of(top);
                        if (odd) f = score_at(q) + as_global(a.Acol)[(uint32_t)q * (uint32_t)Kp + cb + jl];
                    } else if constexpr (FILTER) {
                        scan_states(thr, INFINITY, f, q);
                    } else {
                        gfloat_t* const ak = as_global(a.Acol) + cb + jl;
                        for (int32_t l = 0; l < done; ++l) {
                            const int32_t cnt = uni(s.cnt[par][l]);
                            for (int32_t p = 0; p < cnt; p += 8) {
                                BoundEnt en[8];
                                float v[8];
    #pragma unroll
                                for (int u = 0; u < 8; ++u) en[u] = s.list[l][min(p + u, cnt - 1)];
    #pragma unroll
                                for (int u = 0; u < 8; ++u) v[u] = ak[(uint32_t)(en[u].lo ^ flip) * (uint32_t)Kp];
    #pragma unroll
                                for (int u = 0; u < 8; ++u) take1(f, q, en[u].v + v[u], en[u].lo ^ flip);
                            }
                        }
                        if (out) take1(f, q, fo, qo);
                    }
                    top = __hiloint2double(__float_as_int(f), q ^ flip ^ (mixm & ~(__float_as_int(f) >> 31)));
                }
                const float b = __int_as_float(__double2hiint(top));
                const int32_t arg = b > -INFINITY ? state_of(top) : 0;
                const float xn = jl < cn ? b + s.eb[half][row * TC + jl] : -INFINITY;
                int32_t mid = 0;
                if (mode == BM_DIV) {
                    mid = e_prev == t - 1 ? arg : (t > e_first + 1 ? s.anc[TEAM ? 0 : xp][arg] : 0);
                    if (t == e_next && jl < cn) {
                        st_cf(dsnap() + (int64_t)d_next * Kp + cb + jl, xn);
                        if (d_next >= 1) st_c(link() + (int64_t)d_next * Kp + cb + jl, mid);
                    }
                } else {
                    s.pb[half][row * TC + jl] = (uint16_t)arg;
                }
                publish(t, xn, mid);
                // what the next step's lists are made from, off the path of its scores
                const float nd = D - (b - s.cm[jl]);   // NaN where nothing is needed
                const uint32_t mx = wave_max(nd > 0.0f && nd < INFINITY ? __float_as_uint(nd) : 0u);
                if (lane == 0) atomicMax(&s.need[par ^ 1], mx);
            };
            if constexpr (FILTER) {
                if (active) {
                    double b0[4] = {none, none, none, none}, b1[4] = {none, none, none, none};
                    const int32_t add = (g * 64 + 4 * (lane & 7)) * 4 + add0;
                    // rows of a half's list: 8 lanes across 32 columns, 8 rows a load
                    auto fetch_rows = [&](auto& en, auto& av, int32_t hf, int32_t at) {
                        constexpr int N = sizeof(en) / sizeof(en[0]);
#pragma unroll
                        for (int u = 0; u < N; ++u) en[u] = s.rows[wv][hf][at + (lane >> 3) + u * 8];
#pragma unroll
                        for (int u = 0; u < N; ++u)
                            av[u] = *reinterpret_cast<gvec_t*>(A + (uint32_t)(__mul24(en[u].lo, mul) + add + hf * 128));
                        __builtin_amdgcn_sched_barrier(0);   // every load is issued before the next wait
                    };
                    // both halves' lists: each half's next rows are in flight while the
                    // other's are scanned
                    auto scan_rows = [&](int32_t n0, int32_t n1) {
                        constexpr int U = 2, inc = 8 * U;
                        BoundEnt e0[U], e1[U];
                        vec_t v0[U], v1[U];
                        const int32_t most = max(n0, n1);
                        listed += most;
                        // both lists to a multiple of 16 at the longer one's end: rows that cannot win
                        for (int32_t e = min(n0, n1) + (lane & 15); e < most + 16; e += 16) {
                            if (e >= n0) s.rows[wv][0][e] = BoundEnt{flip, -INFINITY};
                            if (e >= n1) s.rows[wv][1][e] = BoundEnt{flip, -INFINITY};
                        }
                        if (mixed) {
#pragma unroll 1
                            for (int32_t e = 0; e < most; e += inc) {
                                fetch_rows(e0, v0, 0, e);
                                fetch_rows(e1, v1, 1, e);
                                scan(Mixed{}, b0, e0, v0);
                                scan(Mixed{}, b1, e1, v1);
                            }
                            return;
                        }
                        fetch_rows(e0, v0, 0, 0);
                        fetch_rows(e1, v1, 1, 0);
#pragma unroll 1
                        for (int32_t e = inc; e < most; e += inc) {
                            scan(OneSign{}, b0, e0, v0);
                            fetch_rows(e0, v0, 0, e);
                            scan(OneSign{}, b1, e1, v1);
                            fetch_rows(e1, v1, 1, e);
                        }
                        scan(OneSign{}, b0, e0, v0);
                        scan(OneSign{}, b1, e1, v1);
                    };
                    const uint32_t* const rb = s.rb + g * Kp;
                    // listed states with bounds from the lane's lo up to (not including) its hi
                    auto filter = [&](float lo, float hi, int32_t tiers) {
                        const float lo0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lo), 0));
                        const float lo1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lo), 8));
                        const float hi0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(hi), 0));
                        const float hi1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(hi), 8));
                        // near states from the list's front, far ones from its back
                        const int32_t near = uni(cn4.x), listed = near + (tiers > 1 ? uni(cn4.y) : 0);
                        int32_t n0 = 0, n1 = 0;
#pragma unroll 1
                        for (int32_t e = 0; e < listed; e += 256) {
                            BoundEnt en[4];
                            uint32_t r[4];
                            float x[4];
#pragma unroll
                            for (int c = 0; c < 4; ++c) {
                                const int32_t p = min(e + c * 64 + lane, listed - 1);
                                en[c] = s.list[0][p < near ? p : LC - 1 - (p - near)];
                            }
#pragma unroll
                            for (int c = 0; c < 4; ++c) r[c] = rb[en[c].lo ^ flip];
#pragma unroll
                            for (int c = 0; c < 4; ++c) x[c] = e + c * 64 + lane < listed ? en[c].v : -INFINITY;
                            int32_t from = 0;   // 64s that are on the lists
#pragma unroll 1
                            do {
                                bool room = true;
#pragma unroll
                                for (int c = 0; c < 4; ++c) {
                                    if (c < from || !room) continue;
                                    const float y0 = add_lo16(x[c], r[c]), y1 = add_hi16(x[c], r[c]);
                                    const uint64_t m0 = __builtin_amdgcn_ballot_w64(y0 >= lo0) &
                                                        __builtin_amdgcn_ballot_w64(y0 < hi0);
                                    const uint64_t m1 = __builtin_amdgcn_ballot_w64(y1 >= lo1) &
                                                        __builtin_amdgcn_ballot_w64(y1 < hi1);
                                    const int32_t a0 = n0 + __popcll(m0), a1 = n1 + __popcll(m1);
                                    room = max(a0, a1) <= kRowCap;
                                    if (!room) continue;
                                    if (y0 >= lo0 && y0 < hi0)
                                        s.rows[wv][0][__builtin_amdgcn_mbcnt_hi((uint32_t)(m0 >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((uint32_t)m0, n0))] = en[c];
                                    if (y1 >= lo1 && y1 < hi1)
                                        s.rows[wv][1][__builtin_amdgcn_mbcnt_hi((uint32_t)(m1 >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((uint32_t)m1, n1))] = en[c];
                                    n0 = a0;
                                    n1 = a1;
                                    from = c + 1;
                                }
                                if ((from < 4 || e + 256 >= listed) && max(n0, n1) > 0) {
                                    scan_rows(n0, n1);
                                    n0 = n1 = 0;
                                }
                            } while (from < 4);
                        }
                    };
                    const float cm = s.cm[jl];
                    // the distance that the columns of the lane's half need
                    auto reach = [&](double top) {
                        const float nd = D - (__int_as_float(__double2hiint(top)) - cm);   // NaN where nothing is needed
                        return __uint_as_float(half_max(nd > 0.0f && nd < INFINITY ? __float_as_uint(nd) : 0u));
                    };
                    auto open = [&](float lo, double top) {
                        return __builtin_amdgcn_ballot_w64(lo + cm >= __int_as_float(__double2hiint(top))) != 0;
                    };
                    float lo = fmaxf(h0, D - kHalf * (step == 0 ? F1 : F)), hi = INFINITY;
                    double top;
                    float u;
#pragma unroll 1
                    for (int round = 0;; ++round) {
                        filter(lo, hi, __builtin_amdgcn_ballot_w64(lo < h0) ? 2 : 1);
                        top = merge_halves(b0, b1);
                        u = reach(top);
                        if (round == 2 || !open(lo, top)) break;
                        // no row whose bound is below the next lo can win (checked, not
                        // derived), or every listed row with an edge is read; at first
                        // the rows with bounds from h1 on, which mostly close it
                        hi = lo;
                        lo = fminf(lo, D - u * 1.001f - 1e-6f * fabsf(D));
                        const bool bad = cm == cm && !(lo + cm < __int_as_float(__double2hiint(top)));
                        if (half_max(bad ? 1u : 0u)) lo = -FLT_MAX;
                        if (round == 0) lo = fmaxf(lo, h1);
                    }
                    float thr = fminf(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(lo), 0)),
                                      __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lo), 8)));
                    // a bound is no larger than its state's score: below h1 there may
                    // be states on no list with bounds from lo on
                    const bool more = thr < h1 && outside && open(h1, top);
                    if (more) {
                        thr = h1;
                        top = beyond(top, thr);
                        u = reach(top);
                    }
                    if (step == 0) F1 = fmaxf(F1 + 0.5f * (u - F1), 1e-4f);
                    else F = fmaxf(F + kEma * (u - F), 1e-4f);
                    finish(top, thr, 0, more, 0.0f, 0);
                    if (kind != KIND_SUB && (step & 15) == 15) {
                        listed = max(listed - 12 * K, -kQuitCap);
                        if (listed > 3 * K && lane == 0) s.sv[7] = 1;
                    }
                }
            } else {
                double best[4] = {none, none, none, none};
                const int32_t add = (g * 64 + lc4) * 4 + add0;
                // the waves of a group share its first lists (the first alone when
                // the group is one wave's) without a look at the bound
                if (active && !mixed) {
                    for (int32_t k = 0; k < min(wpg > 1 ? 2 : 1, lists); ++k) {
                        const BoundEnt* const list = s.list[k];
                        const int32_t cnt = uni(s.cnt[par][k]), inc = wpg * UN;
                        BoundEnt e0[UL], e1[UL];
                        vec_t v0[UL], v1[UL];
                        int32_t e = sub * UN;
                        if (e >= cnt) continue;
                        load(e0, v0, list, e, cnt, add);
                        for (; e + 2 * inc < cnt; e += 2 * inc) {
                            load(e1, v1, list, e + inc, cnt, add);
                            scan(OneSign{}, best, e0, v0);
                            load(e0, v0, list, e + 2 * inc, cnt, add);
                            scan(OneSign{}, best, e1, v1);
                        }
                        if (e + inc < cnt) {
                            load(e1, v1, list, e + inc, cnt, add);
                            scan(OneSign{}, best, e0, v0);
                            scan(OneSign{}, best, e1, v1);
                        } else {
                            scan(OneSign{}, best, e0, v0);
                        }
                    }
                } else if (active) {
                    for (int32_t k = 0; k < min(wpg > 1 ? 2 : 1, lists); ++k) {
                        const int32_t cnt = uni(s.cnt[par][k]), inc = 2 * wpg * UN;
#pragma unroll 1
                        for (int32_t e = 2 * sub * UN; e < cnt; e += inc) {
                            BoundEnt e0[2 * UL];
                            vec_t v0[2 * UL];
                            load(e0, v0, s.list[k], e, cnt, add);
                            scan(Mixed{}, best, e0, v0);
                        }
                    }
                }
                int32_t k = min(wpg > 1 ? 2 : 1, lists);
                double top = merge_group(best);
                if (wpg > 1) {
                    if (active) atomicMax(&s.part[jl], pattern_key(top));
                    __syncthreads();
                    if (active) top = pattern_of_key(s.part[jl]);
                }
                if (active && sub == 0) {
                    // true when nothing outside the first k lists can win a column
                    auto closed = [&]() {
                        return __builtin_amdgcn_ballot_w64(below(k) + s.cm[jl] >= __int_as_float(__double2hiint(top))) == 0;
                    };
                    bool stop = k > 0 && closed();
                    while (!stop && k < lists) {
                        const int32_t cnt = uni(s.cnt[par][k]);
                        double more[4] = {none, none, none, none};
                        for (int32_t e = 0; e < cnt; e += 2 * UN) {
                            BoundEnt e0[2 * UL];
                            vec_t v0[2 * UL];
                            load(e0, v0, s.list[k], e, cnt, add);
                            if (mixed) scan(Mixed{}, more, e0, v0);
                            else scan(OneSign{}, more, e0, v0);
                        }
                        if (FAR && K > LC) far = min(far + cnt / 4, kQuitCap);   // (by one wave, 16 rows in flight, not 4)
                        ++k;
                        top = max64(top, merge_group(more));
                        stop = closed();
                    }
                    // states outside the lists, where the bound still asks for them
                    const bool out = !stop && outside;
                    float fo = -INFINITY;
                    int32_t qo = 0;
                    // (of a first list without room for them, more than LC)
                    auto beyond_reason = [&](int32_t rows) {
                        const int64_t most = K / (K > LC ? 8 : 4) + (int64_t)step * (K / 32) + (kind == KIND_SUB ? 16 * K : 0);
                        return FAR && t < n && far + rows > min(most, (int64_t)kQuitCap);
                    };
                    bool drop = beyond_reason(out && lists == 0 ? LC : 0);
                    if (out && !drop) {
                        // none that scores below thr can win (checked, not derived: the
                        // subtraction is rounded)
                        const float bs = __int_as_float(__double2hiint(top)), cm = s.cm[jl];
                        const float nd = D - (bs - cm);
                        const float lim = __uint_as_float(wave_max(nd > 0.0f ? __float_as_uint(nd) : 0u));
                        float thr = D - lim * 1.001f - 1e-6f * fabsf(D);
                        if (__builtin_amdgcn_ballot_w64(cm == cm && !(thr + cm < bs))) thr = -FLT_MAX;
                        const float top_of = below(k);
                        gfloat_t* const ak = as_global(a.Acol) + cb + jl;
                        for (int32_t c0 = 0; c0 < K; c0 += 256) {
                            float xo[4];
#pragma unroll
                            for (int u = 0; u < 4; ++u)
                                xo[u] = score_at(min(c0 + u * 64 + lane, K - 1));
                            if constexpr (FAR) {
                                drop = beyond_reason(0);   // with the rows read so far
                                if (drop) break;
                            }
#pragma unroll
                            for (int u = 0; u < 4; ++u) {
                                const bool in = c0 + u * 64 + lane < K && xo[u] >= thr && xo[u] < top_of;
                                uint64_t mask = __builtin_amdgcn_ballot_w64(in);
                                if constexpr (FAR) far = min(far + (int32_t)__popcll(mask), kQuitCap);
                                while (mask) {   // four rows in flight
                                    int32_t r[4];
                                    float v[4];
#pragma unroll
                                    for (int q = 0; q < 4; ++q) {
                                        r[q] = mask ? (int32_t)__builtin_ctzll(mask) : r[q ? q - 1 : 0];
                                        mask &= mask - 1;
                                        v[q] = ak[(uint32_t)(c0 + u * 64 + r[q]) * (uint32_t)Kp];
                                    }
#pragma unroll
                                    for (int q = 0; q < 4; ++q)
                                        take1(fo, qo,
                                              __int_as_float(__builtin_amdgcn_readlane(__float_as_int(xo[u]), r[q])) + v[q],
                                              c0 + u * 64 + r[q]);
                                }
                            }
                        }
                        top = max64(top, pattern(fo, qo));
                    }
                    if (drop) {   // no one reads this row's scores
                        give_up = 1;
                        publish(t, -INFINITY, 0);
                    } else {
                        finish(top, 0.0f, k, out, fo, qo);
                    }
                }
            }
            if (t == e_next) {
                e_prev = t;
                ++d_next;
                e_next = d_next < w - 1 ? div_end(d_next) : -1;
            }
        }
        // ---- end of the pass: every block's stores complete, then its counter
        __syncthreads();
        if (mode != BM_DIV && n > m && !retry) {
            const int32_t cnt = (n - m - 1) % NB + 1;
            flush(((n - m - 1) / NB) & 1, n - cnt + 1, cnt);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        const int32_t xe = (int32_t)(epoch + (uint32_t)(n - m)) & 1;   // the last scores' parity
        // The next tags follow those of the last words written, also where the
        // pass was given up: what is still there of either parity is a few tags
        // back, and the tags (15 bits) come round to it in no wait.
        epoch += (uint32_t)(made + 1 + (made == 1));
        if (M > 1) {
            if (member != 0) {
                if (tid == 0) st_c(tb.done + member, task_no);
                continue;
            }
            for (int32_t k = 1 + tid; k < M; k += kTThreads)
                for (int64_t turn = 0; ld_c(tb.done + k) != task_no && !wait_over(a, turn, false); ++turn)
                    __builtin_amdgcn_s_sleep(1);
            __syncthreads();
        }
        auto last_x = [&](int32_t j) {
            if constexpr (TEAM) return __uint_as_float((uint32_t)ld_c(tb.x[xe] + j));
            else return s.x[xe][j];
        };
        int32_t q_end = q_n;
        bool feasible = true;
        if (retry) {
            if (tid == 0) st_c(&sq.status, kBoundRetry);
            feasible = false;
        } else if (kind != KIND_SUB) {
            // the largest score and its lowest state (-0 and +0 equal)
            if (tid == 0) s.key = 0;
            __syncthreads();
            unsigned long long key = 0;
            for (int32_t j = tid; j < K; j += kTThreads) {
                const unsigned long long o = order_key(last_x(j), j);
                key = o > key ? o : key;
            }
            atomicMax(&s.key, key);
            __syncthreads();
            q_end = clampi((int32_t)(0xFFFFFFFFu - (uint32_t)(s.key & 0xFFFFFFFFull)), K);
            const float score = last_x(q_end);
            feasible = score != -INFINITY;
            if (!feasible)
                for (int32_t t = tid; t <= n; t += kTThreads) st_c(sq.path + t, -1);
            if (tid == 0) {
                st_cf(sq.score, score);
                if (feasible) st_c(sq.path + n, q_end);
                else st_c(&sq.status, (int32_t)FV_E_INFEASIBLE);
            }
        }
        if (feasible && mode != BM_DIV) {
            // walk the backpointer rows t = n .. m + 1 from q_end; short rows are
            // copied to LDS in chunks, of long ones only the entries on the path
            // are read
            const uint16_t* const tab = table();
            int32_t* const path = sq.path;
            int32_t q = q_end;
            constexpr int32_t cap = (int32_t)(sizeof(s.walk) / 4);
            const int32_t w2 = (K + 1) / 2, per = KC <= 4096 && !(K & 1) ? min(cap / w2, 64) : 0;
            if (per >= 4) {
                for (int32_t hi = n; hi > m; hi -= per) {
                    const int32_t lo = max(m + 1, hi - per + 1), cnt = (hi - lo + 1) * w2;
                    const uint32_t* src = reinterpret_cast<const uint32_t*>(tab + (int64_t)(lo - tab0) * K);
                    __syncthreads();
                    for (int32_t k = tid; k < cnt; k += 8 * kTThreads) {
                        uint32_t v[8];
#pragma unroll
                        for (int u = 0; u < 8; ++u)
                            v[u] = k + u * kTThreads < cnt ? ld_c(src + k + u * kTThreads) : 0;
#pragma unroll
                        for (int u = 0; u < 8; ++u)
                            if (k + u * kTThreads < cnt) s.walk[k + u * kTThreads] = v[u];
                    }
                    __syncthreads();
                    if (tid == 0) {
                        for (int32_t t = hi; t >= lo; --t) {
                            q = clampi(reinterpret_cast<const uint16_t*>(s.walk)[(t - lo) * K + q], K);
                            st_cg(path + t - 1, q);
                        }
                        s.sv[7] = q;
                    }
                    __syncthreads();
                    q = s.sv[7];
                }
            } else if (tid == 0) {
                for (int32_t t = n; t > m; --t) {
                    q = clampi(ld_c(tab + (int64_t)(t - tab0) * K + q), K);
                    st_cg(path + t - 1, q);
                }
            }
            if (tid == 0 && mode == BM_VANILLA) st_c(&sq.walked, 1);
            __syncthreads();
        } else if (feasible && w > 1) {
            // division states and scores, last to first, then the segments between them
            if (tid == 0) {
                const float* const ds = dsnap();
                const int32_t* const dl = link();
                int32_t q;
                if constexpr (TEAM) q = clampi((int32_t)(uint16_t)(ld_c(tb.x[xe] + q_end) >> 32), K);
                else q = clampi(s.anc[xe][q_end], K);
                for (int32_t d = w - 2; d >= 0; --d) {
                    const int32_t e = div_end(d);
                    st_cg(sq.path + e, q);
                    const float al = ld_cf(ds + (int64_t)d * Kp + q);
                    if (d >= 1) q = clampi(ld_c(dl + (int64_t)d * Kp + q), K);
                    st_cf(a.alpha_at + sq.alpha_off + e, al);
                }
            }
            if (wv == 0) {
                int32_t cnt = 0;
                for (int32_t k0 = 0; k0 < w; k0 += 64) {
                    const int32_t k = k0 + lane;
                    const bool seg = k < w && (k == w - 1 ? n : div_end(k)) > (k == 0 ? m : div_end(k - 1) + 1);
                    cnt += __popcll(__builtin_amdgcn_ballot_w64(seg));
                }
                uint32_t pos = 0;
                if (lane == 0 && cnt > 0) {
                    pos = __hip_atomic_fetch_add(&st->bq_res, (uint32_t)cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_fetch_add(&st->bq_live, (uint32_t)cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                pos = (uint32_t)uni((int32_t)pos);
                uint32_t at = pos;
                for (int32_t k0 = 0; k0 < w; k0 += 64) {
                    const int32_t k = k0 + lane;
                    const int32_t lo = k == 0 ? m : div_end(k - 1) + 1, hi = k >= w - 1 ? n : div_end(k);
                    const bool seg = k < w && hi > lo;
                    const uint64_t mask = __builtin_amdgcn_ballot_w64(seg);
                    if (seg) {
                        const uint32_t p = at + (uint32_t)__popcll(mask & ((1ull << lane) - 1));
                        if ((int64_t)p < a.q_cap) {
                            uint64_t* q = reinterpret_cast<uint64_t*>(a.queue + p);
                            st_c(q, (uint64_t)(uint32_t)seq | ((uint64_t)KIND_SUB << 32));
                            st_c(q + 1, (uint64_t)(uint32_t)lo | ((uint64_t)(uint32_t)hi << 32));
                        }
                    }
                    at += (uint32_t)__popcll(mask);
                }
                // path, scores and tasks are at the memory side before the publication
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                __builtin_amdgcn_s_waitcnt(0);
                if (lane == 0 && cnt > 0) {
                    // publications follow the reservations' order (the earlier one is
                    // being written by a running block); none after a wait that gave up
                    bool next = false;
                    for (int64_t turn = 0; !(next = ld_c(&st->bq_pub) == pos) && !wait_over(a, turn, false); ++turn)
                        __builtin_amdgcn_s_sleep(1);
                    if (next)
                        __hip_atomic_fetch_add(&st->bq_pub, (uint32_t)cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
        __syncthreads();
        if (tid == 0)
            __hip_atomic_fetch_sub(&st->bq_live, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // ---- the last block leaves the sequences it could not decode to the engine
    __syncthreads();
    if (tid == 0) {
        __builtin_amdgcn_s_waitcnt(0);
        s.sv[0] = __hip_atomic_fetch_add(&st->bq_done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == gridDim.x;
    }
    __syncthreads();
    if (!s.sv[0] || wv != 0) return;
    int32_t left = 0;
    for (int32_t k0 = 0; k0 < n_roots; k0 += 64) {
        const int32_t k = k0 + lane;
        Task tk{};
        bool again = false;
        if (k < n_roots) {
            tk = a.queue[k];
            again = ld_c(&a.seqs[tk.seq].status) == kBoundRetry;
        }
        const uint64_t mask = __builtin_amdgcn_ballot_w64(again);
        if (again) {
            a.queue[left + __popcll(mask & ((1ull << lane) - 1))] = tk;
            st_c(&a.seqs[tk.seq].status, (int32_t)FV_OK);
        }
        left += __popcll(mask);
    }
    if (lane == 0) st->q_tail0 = left;
}

// One block per task for K <= 256, 512 and 1024, teams for K <= 1024, 4096
// and 16384.  Those up to K = 1024 come with MIX for short sequences (kMixT),
// which costs the common step 3 to 7% (registers), and without for others; above,
// where one wave's second scan of a step is many times the step, all have it
// (K = 1243, 93 sequences, FLASH: 27.4 ms without, 28.5 with; K = 4096, T = 100 and
// scores from above zero: 3.8 and 3.4).  A block takes a CU's 16 wavefronts (two blocks of 8 for one task
// each: 158 instead of 112 ms for 256 sequences of K = 1024, FLASH P = 64, whose
// roots then leave half of them idle); up to K = 256, with a wave for each
// group and rows enough for one or two units, three blocks of 4 share a CU:
// 512 sequences of K = 256, T ~ U[32, 512], FLASH P = 16 and the score's gradients
// take 2.6 ms (8 waves each: 2.5, 16: 3.9; 64 sequences of K = 200: 1.5, 1.7, 1.7).
#define FV_TEAM(NAME, KC, LC, NB, TEAM, W, FILTER, MIX)                                                         \
    extern "C" __global__ __launch_bounds__(64 * W, W == 4 ? 3 : 4) void NAME(const EngineArgs* __restrict__ table) {                \
        team_decode<KC, LC, NB, TEAM, W, FILTER, MIX>(*reinterpret_cast<cargs_t*>(reinterpret_cast<uint64_t>(table))); \
    }
FV_TEAM(fv_bound256_kernel, 256, 256, 8, false, 4, false, false)
FV_TEAM(fv_bound256_short_kernel, 256, 256, 8, false, 4, false, true)
FV_TEAM(fv_bound512_kernel, 1024, 1024, 4, false, 16, false, false)
FV_TEAM(fv_bound512_short_kernel, 1024, 1024, 4, false, 16, false, true)
FV_TEAM(fv_bound1k_kernel, 1024, 1024, 2, false, 16, true, false)
FV_TEAM(fv_bound1k_short_kernel, 1024, 1024, 2, false, 16, true, true)
FV_TEAM(fv_team1k_kernel, 1024, 1024, 4, true, 16, false, false)
FV_TEAM(fv_team1k_short_kernel, 1024, 1024, 4, true, 16, false, true)
FV_TEAM(fv_team4k_kernel, 4096, kBoundListK, 4, true, 16, false, true)
FV_TEAM(fv_team16k_kernel, 16384, kBoundListK, 2, true, 16, false, true)
#undef FV_TEAM

// Row bounds: rowb[g][i] (two float16) >= max over the 32 columns of either half
// of group g of log A(i, j) - (column j's maximum); -inf where no column has an
// edge from i.
// A block takes 64 rows of a group.
extern "C" __global__ __launch_bounds__(kBlock) void fv_rowbound_kernel(const float* __restrict__ Ap, int32_t K,
                                                                        int32_t Kp,
                                                                        const uint32_t* __restrict__ cmax,
                                                                        uint32_t* __restrict__ rowb) {
    __shared__ float part[64][65];
    const int32_t c = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int32_t j = blockIdx.x * 64 + c, i0 = blockIdx.y * 64;
    const float cm = j < K ? score_of_key(cmax[j]) : -INFINITY;
    for (int32_t r = w; r < 64; r += kWaves) {
        const int32_t i = i0 + r;
        float v = -INFINITY;
        // rounded towards zero, that is, up: the difference is not positive
        if (i < K && cm > -INFINITY) {
            const float x = Ap[(int64_t)i * Kp + j];
            v = (x - cm) * (1.0f - 0x1p-20f);
            if (x > -INFINITY) v = fmaxf(v, -FLT_MAX);   // an edge, whatever the difference
        }
        part[r][c] = v;
    }
    __syncthreads();
    if (threadIdx.x < 64) {
        const int32_t r = threadIdx.x;
        float v0 = -INFINITY, v1 = -INFINITY;
#pragma unroll
        for (int k = 0; k < 32; ++k) {
            v0 = fmaxf(v0, part[r][k]);
            v1 = fmaxf(v1, part[r][32 + k]);
        }
        rowb[(int64_t)blockIdx.x * Kp + i0 + r] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(v0, v1));
    }
}

// Column maxima of log A as order keys (cmax zeroed before): each block takes
// 64 columns of a share of the rows.  Also clears the teams' exchange buffers
// (nzero 16-byte words).
extern "C" __global__ __launch_bounds__(kBlock) void fv_colmax_kernel(const float* __restrict__ log_a, int32_t K,
                                                                      uint32_t* __restrict__ cmax,
                                                                      uint4* __restrict__ zero, int64_t nzero) {
    const int64_t nthreads = (int64_t)gridDim.x * gridDim.y * kBlock;
    for (int64_t k = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * kBlock + threadIdx.x; k < nzero; k += nthreads)
        zero[k] = uint4{0, 0, 0, 0};
    __shared__ float part[kWaves][64];
    const int32_t c = threadIdx.x & 63, r = threadIdx.x >> 6;
    const int32_t j = blockIdx.x * 64 + c;
    float v0 = -INFINITY, v1 = -INFINITY, v2 = -INFINITY, v3 = -INFINITY;
    const int32_t step = (int32_t)gridDim.y * kWaves;
    if (j < K) {
        int32_t i = blockIdx.y * kWaves + r;
        for (; i + 3 * step < K; i += 4 * step) {
            v0 = fmaxf(v0, log_a[(int64_t)i * K + j]);
            v1 = fmaxf(v1, log_a[(int64_t)(i + step) * K + j]);
            v2 = fmaxf(v2, log_a[(int64_t)(i + 2 * step) * K + j]);
            v3 = fmaxf(v3, log_a[(int64_t)(i + 3 * step) * K + j]);
        }
        for (; i < K; i += step) v0 = fmaxf(v0, log_a[(int64_t)i * K + j]);
    }
    part[r][c] = fmaxf(fmaxf(v0, v1), fmaxf(v2, v3));
    __syncthreads();
    if (r == 0 && j < K) {
        const float m = fmaxf(fmaxf(part[0][c], part[1][c]), fmaxf(part[2][c], part[3][c]));
        atomicMax(&cmax[j], score_key(m));
    }
}

}  // namespace fv
