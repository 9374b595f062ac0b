// FLASH-BS (beam) decoding, one block per task (gfx950).
//
// The lock-step engine takes a beam task one step per global step, its beam
// going through memory between them: 40 us a step for 64 dense sequences of
// K = 1024 (B = 64), 100 us for 64 trajectories on a graph of 99,856 states
// (B = 128), whatever few states a beam holds.  Here a block keeps a task's
// beam in LDS from the first step to the last and takes tasks (roots longest
// first, then the subtasks they spawn) from the queue of the bounded scans,
// with no step shared between tasks.
//
// A step scores the beam's successors, finds the B-th best score and lays
// the beam out again in state order:
//   dense:  a wave takes 64 columns, 16 lanes across them and 4 beam states
//           side by side (16-byte loads of log A rows, which bound the step:
//           B rows of K floats from L2 at about 62 bytes a clock and CU);
//   sparse: the beam states' out-edges go to a hash table in LDS by
//           destination, each slot keeping its best candidate (three dependent
//           reads, row pointers, edges and points, bound the step);
//   select: a histogram of the distances below the best score, 256 bins over
//           about three times the last beam's depth, then the exact ranks inside
//           the bin that holds the B-th.
// Arithmetic, ties and the subtask structure are the engine's.  A subtask whose
// beam lost its end state needs the exact re-decode, and a step with more
// candidates than the table holds needs the engine's sort: such tasks, and what
// they spawn, are left to the engine, which runs after this kernel.
//
// Measured against the engine: 64 sequences, K = 1024, T ~ U[200, 2000], B = 64,
// P = 16: 91.4 -> 14.6 ms; 64 trajectories on 99,856 states, T ~ U[200, 2000],
// B = 128, P = 16: 243 -> 14.6 ms (a step takes 8 and 6 us, half of it
// the reads named above).
#include <float.h>

#include "fv_device.h"

namespace fv {

constexpr int kBW = 16;               // waves of a block
constexpr int kBThreads = 64 * kBW;
constexpr int kHash = 2048;           // slots of the sparse step's table
constexpr int kHashFill = kBeamCands; // candidates it takes
constexpr int kInitCap = kHash - kBThreads;   // entries a sparse start holds before it selects

// A subtask's right child of at least this many positions goes to the queue, a
// shorter one, like every left child, stays with its block: a publication
// waits for the one before it (0.8 us), and 64 sequences of T ~ U[200, 2000]
// have 70,000 subtasks (K = 1024, B = 64: 44.7 ms with all of them
// queued, 14.4 with these).
constexpr int kBeamShare = 12;
constexpr int kBeamStack = 32;
constexpr int kBeamRank = 256;        // members of a bin that are ranked one by one, at most

struct BeamTask {
    int32_t m, n, q_prev, q_n;
    float alpha;
};

struct BeamBlk {
    // the beam, in state order, by step parity; the beam at t_mid
    int32_t bs[2][kBeamBlockB], ba[2][kBeamBlockB], ss[kBeamBlockB];
    float bv[2][kBeamBlockB], sv[kBeamBlockB];
    uint32_t hist[2][256];
    // members of the bin that holds the B-th score
    uint32_t ckey[kHash];
    int32_t cst[kHash];
    // sparse: table of destinations and their best candidates; kept entries
    int32_t hst[kHash];
    unsigned long long hval[kHash];
    int32_t ks[kBeamBlockB], ka[kBeamBlockB];
    float kv[kBeamBlockB];
    // by step modulo 3: order key of the best score, finite scores
    uint32_t best[3];
    int32_t fin[3];
    int32_t ncand, ncrit, nkept, snap_n;
    int32_t sv_[8];
    BeamTask stack[kBeamStack];       // this block's subtasks
    unsigned long long key;
    unsigned long long clo, chi;      // range of the bin's members
};

// Order of scores as unsigned numbers (-0 and +0 equal); 0 for none.
__device__ __forceinline__ uint32_t beam_key(float v) {
    if (v == 0.0f) v = 0.0f;
    const uint32_t b = __float_as_uint(v);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float beam_key_score(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}
// inclusive sum over the lanes up to this one
__device__ __forceinline__ int32_t wave_scan(int32_t x) {
    uint32_t v = (uint32_t)x;
    v += dpp_u<0x111, 0xf>(v);   // row_shr:1
    v += dpp_u<0x112, 0xf>(v);
    v += dpp_u<0x114, 0xf>(v);
    v += dpp_u<0x118, 0xf>(v);
    v += dpp_u<0x142, 0xa>(v);   // row_bcast:15
    v += dpp_u<0x143, 0xc>(v);   // row_bcast:31
    return (int32_t)v;
}
// position of state q in a beam of nb entries in state order, or -1
__device__ __forceinline__ int32_t beam_at(const int32_t* bs, int32_t nb, int32_t q) {
    int32_t lo = 0, hi = nb;
    while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if (bs[mid] == q) return mid;
        if (bs[mid] < q) lo = mid + 1; else hi = mid;
    }
    return -1;
}
__device__ __forceinline__ void beam_out_range(cargs_t& a, int32_t s, int32_t& e0, int32_t& e1) {
    int64_t x0 = a.row_ptr[s], x1 = a.row_ptr[s + 1];
    x0 = x0 < 0 ? 0 : (x0 > a.nnz ? a.nnz : x0);
    x1 = x1 < x0 ? x0 : (x1 > a.nnz ? a.nnz : x1);
    e0 = (int32_t)x0;
    e1 = (int32_t)x1;
}

// The bin that holds the b-th of n entries counted in hist (those counted
// nowhere belong to the last bin); the entries in front of it and in it.  The
// same in every lane.
__device__ __forceinline__ int32_t beam_bin(const uint32_t* hist, int32_t n, int32_t b, int32_t& before, int32_t& in) {
    const int32_t lane = threadIdx.x & 63;
    uint4 c = *reinterpret_cast<const uint4*>(&hist[4 * lane]);
    int32_t own = (int32_t)(c.x + c.y + c.z + c.w);
    int32_t upto = wave_scan(own);
    const int32_t others = n - __builtin_amdgcn_readlane(upto, 63);
    if (lane == 63) {
        c.w += (uint32_t)others;
        own += others;
        upto = n;
    }
    const uint64_t reach = __builtin_amdgcn_ballot_w64(upto >= b);
    const int32_t src = (int32_t)__builtin_ctzll(reach);   // n >= b: some lane reaches b
    int32_t kb = 4 * src;
    before = __builtin_amdgcn_readlane(upto - own, src);
    in = __builtin_amdgcn_readlane((int32_t)c.x, src);
    const int32_t c1 = __builtin_amdgcn_readlane((int32_t)c.y, src), c2 = __builtin_amdgcn_readlane((int32_t)c.z, src),
                  c3 = __builtin_amdgcn_readlane((int32_t)c.w, src);
    if (before + in < b) { before += in; in = c1; ++kb; }
    if (before + in < b) { before += in; in = c2; ++kb; }
    if (before + in < b) { before += in; in = c3; ++kb; }
    return kb;
}

// Many entries in the bin that holds the B-th (equal scores, or a depth unlike
// the last beam's): 256 bins over the bits of (score, state) in which they
// differ, until few are left.  1024 states' ranks inside one bin take 100 us, such
// a pass 2.  (Not inlined: the step's loads lose registers to it, 2% of the time
// of 64 sequences of K = 1024, B = 64.)
struct BeamCut {
    int32_t in, take;   // entries in the bin, and how many of them are kept
    int32_t mask;       // of this thread's: kept (bits 0, 1), in the bin (bits 2, 3)
};
__device__ __noinline__ BeamCut beam_narrow(BeamBlk& s, int32_t par, BeamCut c, unsigned long long w0,
                                            unsigned long long w1) {
    const int32_t tid = threadIdx.x, lane = tid & 63;
    unsigned long long w[2] = {w0, w1};   // score and state; 0: not in the bin
    int32_t kept = 0;
    while (c.in > kBeamRank) {
        __syncthreads();
        if (tid < 256) s.hist[par][tid] = 0;
        if (tid == 0) {
            s.ncrit = 0;
            s.clo = ~0ull;
            s.chi = 0;
        }
        __syncthreads();
        unsigned long long hi = max(w[0], w[1]);
        unsigned long long lo = min(w[0] ? w[0] : ~0ull, w[1] ? w[1] : ~0ull);
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            lo = min(lo, (unsigned long long)__shfl_xor(lo, off, 64));
            hi = max(hi, (unsigned long long)__shfl_xor(hi, off, 64));
        }
        if (lane == 0 && hi != 0) {
            atomicMin(&s.clo, lo);
            atomicMax(&s.chi, hi);
        }
        __syncthreads();
        hi = s.chi;
        const int32_t shift = max(0, 56 - __clzll((long long)(hi - s.clo)));   // (states differ)
        int32_t bin[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            bin[k] = (int32_t)((hi - w[k]) >> shift);
            if (w[k]) atomicAdd(&s.hist[par][bin[k]], 1u);
        }
        __syncthreads();
        int32_t before, in;
        const int32_t kb = beam_bin(s.hist[par], c.in, c.take, before, in);
        c.take -= before;
        c.in = in;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (!w[k]) continue;
            if (bin[k] < kb || (bin[k] == kb && in == c.take)) kept |= 1 << k;
            if (bin[k] != kb || in == c.take) w[k] = 0;
            if (w[k] && in <= kBeamRank) {
                const int32_t p = atomicAdd(&s.ncrit, 1);
                s.ckey[p] = (uint32_t)(w[k] >> 32);
                s.cst[p] = 0x7fffffff - (int32_t)(uint32_t)w[k];
            }
        }
        if (in == c.take) break;
    }
    c.mask = kept | (w[0] ? 4 : 0) | (w[1] ? 8 : 0);
    return c;
}

// The entries to keep of a block's v[0 .. NV) (-inf: none) with states st:
// the top B by (score desc, state asc).  `step` numbers the block's calls;
// best and fin of step modulo 3 are zero.  inv: bins per unit of score.
// Every barrier is on block-uniform control flow.
template <int NV>
__device__ __forceinline__ void beam_keep(BeamBlk& s, int32_t B, uint32_t step, const float (&v)[NV],
                                          const int32_t (&st)[NV], bool (&keep)[NV], float& inv) {
    const int32_t tid = threadIdx.x, lane = tid & 63;
    const int32_t s3 = (int32_t)(step % 3), par = (int32_t)(step & 1);
    uint32_t mk = 0;
    int32_t nf = 0;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const bool in = v[k] > -INFINITY;
        if (in) mk = max(mk, beam_key(v[k]));
        nf += __popcll(__builtin_amdgcn_ballot_w64(in));
    }
    mk = wave_max(mk);
    if (lane == 0 && nf > 0) {
        atomicMax(&s.best[s3], mk);
        atomicAdd(&s.fin[s3], nf);
    }
    __syncthreads();
    const uint32_t top = (uint32_t)uni((int32_t)s.best[s3]);
    const int32_t n = uni(s.fin[s3]);
    // the step after next's, which every wave is past the reads of
    if (tid == 0) {
        s.best[(step + 2) % 3] = 0;
        s.fin[(step + 2) % 3] = 0;
        s.ncrit = s.nkept = s.ncand = 0;
    }
    if (tid < 256) s.hist[par ^ 1][tid] = 0;
    const float D = beam_key_score(top);
    int32_t bin[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        keep[k] = v[k] > -INFINITY;
        bin[k] = 0;
    }
    if (n > B) {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            if (!keep[k]) continue;
            bin[k] = (int32_t)fminf((D - v[k]) * inv, 255.0f);
            if (bin[k] < 255) atomicAdd(&s.hist[par][bin[k]], 1u);   // (the last bin: all others)
        }
    }
    __syncthreads();
    if (n <= B) return;
    // the bin that holds the B-th score (each wave finds it)
    int32_t before, cb, kb = beam_bin(s.hist[par], n, B, before, cb);
    int32_t rem = B - before;
    bool crit[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        crit[k] = keep[k] && bin[k] == kb && cb != rem;
        keep[k] = keep[k] && (bin[k] < kb || (bin[k] == kb && cb == rem));
        if (crit[k]) {
            const int32_t p = atomicAdd(&s.ncrit, 1);
            s.ckey[p] = beam_key(v[k]);
            s.cst[p] = st[k];
        }
    }
    // bins of about 1/80 of this beam's depth next
    inv = fminf(fmaxf(80.0f * inv / (float)(kb + 1), 1e-30f), 1e30f);
    if (cb == rem) return;
    if (__builtin_expect(cb > kBeamRank, 0)) {
        unsigned long long w[2];
        static_assert(NV == 2, "entries per thread");
#pragma unroll
        for (int k = 0; k < NV; ++k)
            w[k] = crit[k] ? (unsigned long long)beam_key(v[k]) << 32 | (uint32_t)(0x7fffffff - st[k]) : 0ull;
        const BeamCut c = beam_narrow(s, par, BeamCut{cb, rem, 0}, w[0], w[1]);
        cb = uni(c.in);
        rem = uni(c.take);
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            keep[k] = keep[k] || (c.mask >> k & 1);
            crit[k] = c.mask >> (2 + k) & 1;
        }
        if (cb == rem) return;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        if (!crit[k]) continue;
        const uint32_t u = beam_key(v[k]);
        int32_t rank = 0;
        for (int32_t p = 0; p < cb; p += 8) {
            uint32_t o[8];
            int32_t os[8];
#pragma unroll
            for (int w = 0; w < 8; ++w) {
                o[w] = s.ckey[min(p + w, cb - 1)];
                os[w] = s.cst[min(p + w, cb - 1)];
            }
#pragma unroll
            for (int w = 0; w < 8; ++w) rank += p + w < cb && (o[w] > u || (o[w] == u && os[w] < st[k]));
        }
        keep[k] = rank < rem;
    }
}

// The kept entries, in any order, as the beam of parity q in state order;
// returns their number.
template <int NV>
__device__ __forceinline__ int32_t beam_lay_out(BeamBlk& s, int32_t B, int32_t q, const float (&v)[NV],
                                                const int32_t (&st)[NV], const int32_t (&an)[NV],
                                                const bool (&keep)[NV]) {
    const int32_t tid = threadIdx.x, lane = tid & 63;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const uint64_t m = __builtin_amdgcn_ballot_w64(keep[k]);
        if (m == 0) continue;
        int32_t at = 0;
        if (lane == 0) at = atomicAdd(&s.nkept, (int32_t)__popcll(m));
        const int32_t p = uni(at) + (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                 __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
        if (keep[k] && p < kBeamBlockB) {
            s.ks[p] = st[k];
            s.kv[p] = v[k];
            s.ka[p] = an[k];
        }
    }
    __syncthreads();
    const int32_t nb = min(uni(s.nkept), B);
    // ranks by state, 8 (4) threads an entry
    const int32_t per = B <= kBThreads / 8 ? 8 : 4, e = tid / per;
    int32_t rank = 0;
    const int32_t mine = e < nb ? s.ks[e] : 0;
    if (e < nb)
        for (int32_t p = tid % per; p < nb; p += 8 * per) {
            int32_t o[8];
#pragma unroll
            for (int w = 0; w < 8; ++w) o[w] = s.ks[min(p + w * per, nb - 1)];
#pragma unroll
            for (int w = 0; w < 8; ++w) rank += p + w * per < nb && o[w] < mine;
        }
    rank += __builtin_amdgcn_update_dpp(0, rank, 0xb1, 0xf, 0xf, false);   // quad_perm: 1, 0, 3, 2
    rank += __builtin_amdgcn_update_dpp(0, rank, 0x4e, 0xf, 0xf, false);   // quad_perm: 2, 3, 0, 1
    if (per == 8) rank += __builtin_amdgcn_update_dpp(0, rank, 0x141, 0xf, 0xf, false);   // row_half_mirror
    if (e < nb && tid % per == 0) {
        s.bs[q][rank] = mine;
        s.bv[q][rank] = s.kv[e];
        s.ba[q][rank] = s.ka[e];
    }
    __syncthreads();
    return nb;
}

struct BeamRecord {
    int32_t* hdr;
    int32_t* s;
    float* v;
    int32_t* a;
};
// a division's record in the root copies: header (word 0: entries), states, scores, anchors
__device__ __forceinline__ BeamRecord beam_record(cargs_t& a, int64_t root_off, int32_t d) {
    float* const base = a.root_copy + (root_off + d) * a.brec;
    BeamRecord r;
    r.hdr = reinterpret_cast<int32_t*>(base);
    r.s = reinterpret_cast<int32_t*>(base + 64);
    r.v = base + 64 + a.Bc;
    r.a = reinterpret_cast<int32_t*>(base + 64 + 2 * (int64_t)a.Bc);
    return r;
}

template <bool SPARSE>
__device__ __forceinline__ void beam_decode(cargs_t& a) {
    __shared__ __align__(16) BeamBlk s;
    constexpr int NV = 2;   // entries of a thread: kBeamBlockK = kHash = 2 kBThreads
    static_assert(NV * kBThreads == kHash && NV * kBThreads == kBeamBlockK, "entries per thread");
    const int32_t tid = threadIdx.x, lane = tid & 63, wv = uni(tid >> 6);
    const int32_t K = a.K, Kp = a.Kp, B = a.B;
    EngineState* const st = a.st;
    const int32_t n_roots = st->q_tail0;
    const int32_t ngt = Kp / 64;
    typedef __attribute__((address_space(1))) const char gchar_t;
    typedef float vec_t __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(1))) const vec_t gvec_t;
    gchar_t* const A = reinterpret_cast<gchar_t*>(reinterpret_cast<uint64_t>(a.Acol));
    if (tid < 256) s.hist[0][tid] = s.hist[1][tid] = 0;
    if (tid < 3) s.best[tid] = s.fin[tid] = 0;
    if (tid == 0) s.ncand = s.ncrit = s.nkept = 0;
    if constexpr (SPARSE)
        for (int32_t k = tid; k < kHash; k += kBThreads) {
            s.hst[k] = -1;
            s.hval[k] = 0;
        }
    uint32_t call = 0;     // selections so far
    float inv = 16.0f;
    int32_t sp = 0;
    for (;;) {
        // ---- next task
        __syncthreads();
        if (sp > 0) --sp;   // of the same sequence
        else if (tid == 0) {
            const int32_t err = ld_c(&st->error);
            const uint32_t h = __hip_atomic_fetch_add(&st->bq_head, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            int32_t got = h < (uint32_t)n_roots && !err ? 1 : 0;
            // spawned tasks: wait for the publication of this ticket, or for the
            // end of every task that could still spawn (each is running on some
            // block, so the wait ends)
            for (int64_t turn = 0; !got && !err; ++turn) {
                const uint32_t live = ld_c(&st->bq_live);
                if (ld_c(&st->bq_pub) > h) { got = 1; break; }
                if (live == 0) {
                    got = ld_c(&st->bq_pub) > h ? 1 : 0;
                    break;
                }
                if (wait_over(a, turn, true)) break;
                __builtin_amdgcn_s_sleep(16);
            }
            unsigned long long w0 = 0, w1 = 0;
            BeamTask& tk = s.stack[0];
            if (got) {
                const unsigned long long* p = reinterpret_cast<const unsigned long long*>(a.queue + h);
                w0 = ld_c(p);
                w1 = ld_c(p + 1);
                const SeqInfo& sq = a.seqs[(int32_t)w0];
                const int32_t tm = (int32_t)w1, tn = (int32_t)(w1 >> 32);
                tk.m = tm;
                tk.n = tn;
                if ((int32_t)(w0 >> 32) == KIND_BSUB) {
                    tk.q_prev = tm > 0 ? ld_c(sq.path + tm - 1) : -1;
                    tk.q_n = ld_c(sq.path + tn);
                    tk.alpha = tm > 0 ? ld_cf(a.alpha_at + sq.alpha_off + tm - 1) : 0.0f;
                }
            }
            s.sv_[0] = got;
            s.sv_[1] = (int32_t)w0;
            s.sv_[2] = (int32_t)(w0 >> 32);
        }
        __syncthreads();
        if (!s.sv_[0]) break;
        SeqInfo& sq = a.seqs[uni(s.sv_[1])];
        const int32_t seq = uni(s.sv_[1]), m = uni(s.stack[sp].m), n = uni(s.stack[sp].n);
        const bool root = uni(s.sv_[2]) != KIND_BSUB;
        const int32_t T = sq.T, pp = sq.pp, tmid = (m + n) >> 1;
        const int32_t q_prev = uni(s.stack[sp].q_prev), q_n = root ? 0 : uni(s.stack[sp].q_n);
        const float alpha = s.stack[sp].alpha;
        bool retry = !root && (q_n < 0 || q_n >= K || (m > 0 && (q_prev < 0 || q_prev >= K)));
        bool lost = false;        // retry, since the beam has no edge to the end state
        int32_t nb = 0, q = 0;    // the beam's entries and parity
        gfloat_t* const lb = as_global(sq.log_b);
        const int64_t ld = sq.ld;
        // this thread's entries: dense columns, or sparse table slots
        float v[NV];
        int32_t sx[NV], an[NV];
        bool keep[NV];
        // scores of the out-edges of the nb states of parity q at step t
        auto push = [&](int32_t t, int32_t mode) {
            const int32_t per = nb <= kBThreads / 8 ? 8 : 4, e = tid / per;
            int32_t e0 = 0, e1 = 0;
            float x = -INFINITY;
            if (e < nb) {
                beam_out_range(a, clampi(s.bs[q][e], K), e0, e1);
                x = s.bv[q][e];
            }
            // every candidate counts against the table's room
            if (tid % per == 0 && e1 > e0) atomicAdd(&s.ncand, min(e1 - e0, kHash));
            __syncthreads();
            const bool full = uni(s.ncand) > kHashFill;
            if (!full) {
                for (int32_t k = e0 + tid % per; k < e1; k += per) {
                    const int32_t j = a.col[k];
                    const float c = x + a.val[k];
                    if (j < 0 || j >= K || !(c > -INFINITY)) continue;
                    // best score first, then the lowest beam entry
                    const unsigned long long w = (unsigned long long)beam_key(c) << 32 | (uint32_t)(0x7fffffff - e);
                    uint32_t hslot = ((uint32_t)j * 2654435761u) >> 21;
                    for (;;) {   // ends: fewer candidates than slots
                        const int32_t old = atomicCAS(&s.hst[hslot], -1, j);
                        if (old == -1 || old == j) break;
                        hslot = (hslot + 1) & (kHash - 1);
                    }
                    atomicMax(&s.hval[hslot], w);
                }
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                const int32_t p = tid + k * kBThreads;
                const int32_t j = s.hst[p];
                const unsigned long long w = s.hval[p];
                s.hst[p] = -1;
                s.hval[p] = 0;
                v[k] = -INFINITY;
                sx[k] = j;
                an[k] = -1;
                if (j >= 0) {
                    const int32_t b = min(0x7fffffff - (int32_t)(uint32_t)w, kBeamBlockB - 1);
                    v[k] = beam_key_score((uint32_t)(w >> 32)) + emission(a, sq.log_b, ld, t, j);
                    an[k] = mode == 1 ? s.bs[q][b] : (mode == 2 ? s.ba[q][b] : -1);
                }
            }
            return full;
        };
        auto select = [&]() {
            beam_keep<NV>(s, B, call, v, sx, keep, inv);
            ++call;
            nb = beam_lay_out<NV>(s, B, q ^ 1, v, sx, an, keep);
            q ^= 1;
        };
        if (!retry) {
            // ---- start: pi + log B_0, or the anchored boundary state's row
            if constexpr (SPARSE) {
                if (m == 0) {
                    // every state, kBThreads at a time: those above the running B-th
                    // score join the beam's entries until a selection makes room
                    uint32_t floor_key = 0;
                    int32_t held = 0;   // entries in s.ckey / s.cst
                    for (int32_t c0 = 0; c0 < K; c0 += kBThreads) {
                        const int32_t j = c0 + tid;
                        float x = -INFINITY;
                        if (j < K) {
                            const float e = emission(a, sq.log_b, ld, 0, j);
                            x = a.log_pi ? a.log_pi[j] + e : e;
                        }
                        const bool in = x > -INFINITY && beam_key(x) > floor_key;
                        if (in) {
                            const int32_t p = atomicAdd(&s.ncand, 1);
                            s.hst[p] = j;      // p < kHash: see below
                            s.hval[p] = (unsigned long long)__float_as_uint(x);
                        }
                        __syncthreads();
                        held = uni(s.ncand);
                        const bool last = c0 + kBThreads >= K;
                        if (held <= kInitCap && !last) {
                            __syncthreads();
                            continue;
                        }
#pragma unroll
                        for (int k = 0; k < NV; ++k) {
                            const int32_t p = tid + k * kBThreads;
                            v[k] = p < held ? __uint_as_float((uint32_t)s.hval[p]) : -INFINITY;
                            sx[k] = p < held ? s.hst[p] : -1;
                            an[k] = -1;
                        }
                        select();   // clears ncand
                        if (!last) {
                            // what is kept, back on the list; later equal scores lose to
                            // these lower states
                            if (nb == B) {
                                uint32_t lo = 0xffffffffu;
                                for (int32_t p = lane; p < nb; p += 64) lo = min(lo, beam_key(s.bv[q][p]));
                                floor_key = ~wave_max(~lo);
                            }
                            if (tid < nb) {
                                s.hst[tid] = s.bs[q][tid];
                                s.hval[tid] = (unsigned long long)__float_as_uint(s.bv[q][tid]);
                            }
                            if (tid == 0) s.ncand = nb;
                        }
                        __syncthreads();
                    }
                    for (int32_t k = tid; k < kHash; k += kBThreads) {
                        s.hst[k] = -1;
                        s.hval[k] = 0;
                    }
                    __syncthreads();
                } else {
                    if (tid == 0) {
                        s.bs[q][0] = q_prev;
                        s.bv[q][0] = alpha;
                        s.ba[q][0] = -1;
                    }
                    nb = 1;
                    __syncthreads();
                    retry = push(m, 0);
                    select();
                }
            } else {
#pragma unroll
                for (int k = 0; k < NV; ++k) {
                    const int32_t j = tid + k * kBThreads;
                    v[k] = -INFINITY;
                    sx[k] = j;
                    an[k] = -1;
                    if (j < K) {
                        const float b = lb[(int64_t)m * ld + j];
                        if (m == 0) v[k] = a.log_pi ? a.log_pi[j] + b : b;
                        else v[k] = (alpha + a.Acol[(int64_t)q_prev * Kp + j]) + b;
                    }
                }
                select();
            }
            // ---- steps
            const int32_t last = root ? T - 1 : n - 1;
            int32_t d_next = 0, e_prev = -1;
            int32_t e_next = root && pp >= 2 ? (int32_t)seg_end(T, pp, 0) : -1;
            const int32_t e_first = e_next;
            // dense: the next step's emission scores of this thread's columns, a step ahead
            float em[NV];
            auto emissions = [&](int32_t t) {
#pragma unroll
                for (int k = 0; k < NV; ++k) {
                    const int32_t j = (wv + k * kBW) * 64 + 4 * (lane & 15) + (lane >> 4);
                    em[k] = !SPARSE && j < K && t <= last ? lb[(int64_t)t * ld + j] : 0.0f;
                }
            };
            if (!SPARSE) emissions(m + 1);
            for (int32_t t = m; !retry; ++t) {
                // the beam of step t is complete
                if (root && t == e_next) {
                    const BeamRecord r = beam_record(a, sq.root_off, d_next);
                    if (tid < nb) {
                        r.s[tid] = s.bs[q][tid];
                        r.v[tid] = s.bv[q][tid];
                        r.a[tid] = s.ba[q][tid];
                    }
                    if (tid == 0) r.hdr[0] = nb;
                    e_prev = t;
                    ++d_next;
                    e_next = d_next < pp - 1 ? (int32_t)seg_end(T, pp, d_next) : -1;
                }
                if (!root && t == tmid) {
                    if (tid < nb) {
                        s.ss[tid] = s.bs[q][tid];
                        s.sv[tid] = s.bv[q][tid];
                    }
                    if (tid == 0) s.snap_n = nb;
                }
                if (t >= last) break;
                const int32_t u = t + 1;   // the step being made
                int32_t mode;   // anchor: 0 none, 1 the predecessor, 2 the predecessor's anchor
                if (root) mode = pp >= 2 && e_prev == t ? 1 : (pp >= 2 && u > e_first + 1 ? 2 : 0);
                else mode = u == tmid + 1 ? 1 : (u > tmid + 1 ? 2 : 0);
                if constexpr (SPARSE) {
                    retry = push(u, mode);
                    if (retry) break;
                } else {
                    const bool neg = nb > 0 && s.bv[q][0] < 0.0f;
                    const int32_t flip = neg ? 0 : -1;
#pragma unroll
                    for (int k = 0; k < NV; ++k) {
                        const int32_t g = wv + k * kBW;
                        const int32_t j = g * 64 + 4 * (lane & 15) + (lane >> 4);
                        v[k] = -INFINITY;
                        sx[k] = j;
                        an[k] = -1;
                        if (g >= ngt || nb == 0) continue;
                        const double none = __hiloint2double((int32_t)0xff800000u, 0);
                        double best[4] = {none, none, none, none};
                        const uint32_t cbyte = (uint32_t)(g * 64 + 4 * (lane & 15)) * 4;
                        for (int32_t b0 = 0; b0 < nb; b0 += 32) {
                            vec_t av[8];
                            float bv[8];
#pragma unroll
                            for (int w = 0; w < 8; ++w) {
                                // a candidate's pattern: score, then beam entry (complemented
                                // for scores that are not negative), see below
                                const int32_t e = min(b0 + 4 * w + (lane >> 4), nb - 1);
                                bv[w] = s.bv[q][e];
                                av[w] = *reinterpret_cast<gvec_t*>(
                                    A + ((uint32_t)__mul24(s.bs[q][e], Kp * 4) + cbyte));
                            }
#pragma unroll
                            for (int w = 0; w < 8; ++w) {
                                const int32_t lo = min(b0 + 4 * w + (lane >> 4), nb - 1) ^ flip;
#pragma unroll
                                for (int c = 0; c < 4; ++c)
                                    best[c] = max64(best[c], __hiloint2double(__float_as_int(bv[w] + av[w][c]), lo));
                            }
                        }
                        const double top = merge_group(best);
                        float c = __int_as_float(__double2hiint(top));
                        int32_t w = __double2loint(top) ^ flip;
                        // zeros and scores of the other sign, which the low word does not order
                        const bool odd = neg ? c >= 0.0f : (c <= 0.0f && c > -INFINITY);
                        if (odd) {
                            c = -INFINITY;
                            w = 0;
                            for (int32_t e = 0; e < nb; ++e) {
                                const float y = s.bv[q][e] + a.Acol[(int64_t)s.bs[q][e] * Kp + j];
                                if (y > c) { c = y; w = e; }
                            }
                        }
                        if (j < K && c > -INFINITY) {
                            v[k] = c + em[k];
                            w = clampi(w, nb);
                            an[k] = mode == 1 ? s.bs[q][w] : (mode == 2 ? s.ba[q][w] : -1);
                        }
                    }
                }
                if (!SPARSE) emissions(u + 1);
                select();
            }
        }
        // ---- end of the task: the block's stores complete (the chain reads them)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (!retry && !root) {
            // only the known end state is scored
            if (tid == 0) s.key = 0;
            __syncthreads();
            unsigned long long key = 0;
            if (tid < nb) {
                float x = -INFINITY;
                if constexpr (SPARSE) {
                    int32_t e0, e1;
                    beam_out_range(a, clampi(s.bs[q][tid], K), e0, e1);
                    for (int32_t e = e0; e < e1; ++e)
                        if (a.col[e] == q_n) x = fmaxf(x, s.bv[q][tid] + a.val[e]);
                } else {
                    x = s.bv[q][tid] + a.Acol[(int64_t)s.bs[q][tid] * Kp + q_n];
                }
                if (x != -INFINITY) key = order_key(x, tid);
            }
            if (key) atomicMax(&s.key, key);
            __syncthreads();
            retry = lost = s.key == 0;   // the beam lost q*_n
        }
        __syncthreads();
        // a subtask's children: the right one on the queue if it is long
        const bool right = !retry && !root && n - m > 2, share = right && n - tmid >= kBeamShare;
        const int32_t base = sp;
        if (!retry && !root) sp += (n - m >= 2 ? 1 : 0) + (right && !share ? 1 : 0);
        if (wv == 0) {
            int32_t cnt = 0;
            if (retry) {
                // the engine's tasks: the second half of the queue (this kernel's take
                // at most the first)
                if (lane == 0) {
                    if (lost) st_c(&sq.status, (int32_t)FV_W_BEAM_FALLBACK);
                    const int64_t p = a.q_cap / 2 + __hip_atomic_fetch_add(&st->bq_left, 1u, __ATOMIC_RELAXED,
                                                                           __HIP_MEMORY_SCOPE_AGENT);
                    const int32_t kind = root ? KIND_BROOT : (lost ? KIND_FSUB : KIND_BSUB);
                    if (p < a.q_cap) {
                        uint64_t* qe = reinterpret_cast<uint64_t*>(a.queue + p);
                        st_c(qe, (uint64_t)(uint32_t)seq | ((uint64_t)(uint32_t)kind << 32));
                        st_c(qe + 1, (uint64_t)(uint32_t)m | ((uint64_t)(uint32_t)n << 32));
                    }
                }
            } else if (!root) {
                if (lane == 0) {
                    const int32_t w = clampi((int32_t)(0xFFFFFFFFu - (uint32_t)(s.key & 0xFFFFFFFFull)), nb);
                    const int32_t qmid = n == tmid + 1 ? s.bs[q][w] : s.ba[q][w];
                    const int32_t at = n - 1 == tmid ? beam_at(s.bs[q], nb, qmid) : beam_at(s.ss, s.snap_n, qmid);
                    float am = __builtin_nanf("");
                    if (at >= 0) am = n - 1 == tmid ? s.bv[q][at] : s.sv[at];
                    st_c(sq.path + tmid, qmid);
                    st_cf(a.alpha_at + sq.alpha_off + tmid, am);
                    if (n - m >= 2) s.stack[sp - 1] = BeamTask{m, tmid, q_prev, qmid, alpha};
                    if (right && !share) s.stack[base] = BeamTask{tmid + 1, n, qmid, q_n, am};
                    // the next of this block's subtasks is of this sequence's kind
                    s.sv_[2] = KIND_BSUB;
                }
                cnt = share ? 1 : 0;
            } else if (nb == 0) {
                for (int32_t k = lane; k < T; k += 64) st_c(sq.path + k, -1);
                if (lane == 0) {
                    st_cf(sq.score, -INFINITY);
                    st_c(&sq.status, (int32_t)FV_E_INFEASIBLE);
                }
            } else {
                // the best end state, and the division chain below it
                unsigned long long key = 0;
                for (int32_t k = lane; k < nb; k += 64) {
                    const unsigned long long o = order_key(s.bv[q][k], s.bs[q][k]);
                    key = o > key ? o : key;
                }
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) {
                    const unsigned long long o = __shfl_xor(key, off, 64);
                    key = o > key ? o : key;
                }
                const int32_t qT = (int32_t)(0xFFFFFFFFu - (uint32_t)(key & 0xFFFFFFFFull));
                if (lane == 0) st_c(sq.path + T - 1, qT);
                int32_t x = s.ba[q][clampi(beam_at(s.bs[q], nb, qT), nb)];
                for (int32_t d = pp - 2; d >= 0; --d) {
                    const BeamRecord r = beam_record(a, sq.root_off, d);
                    const int32_t nr = clampi(ld_c(r.hdr), B + 1);
                    int32_t at = -1;
                    for (int32_t k = lane; k < nr; k += 64)
                        if (ld_c(r.s + k) == x) at = k;
                    const uint64_t hit = __builtin_amdgcn_ballot_w64(at >= 0);
                    at = hit ? __builtin_amdgcn_readlane(at, (int32_t)__builtin_ctzll(hit)) : -1;
                    if (lane == 0) {
                        const int32_t e = (int32_t)seg_end(T, pp, d);
                        st_c(sq.path + e, x);
                        st_cf(a.alpha_at + sq.alpha_off + e, at >= 0 ? ld_cf(r.v + at) : __builtin_nanf(""));
                    }
                    if (d >= 1) x = at >= 0 ? ld_c(r.a + at) : -1;
                }
                for (int32_t k0 = 0; k0 < pp; k0 += 64) {
                    const int32_t k = k0 + lane;
                    const bool seg = k < pp && seg_end(T, pp, k) > (k == 0 ? 0 : seg_end(T, pp, k - 1) + 1);
                    cnt += __popcll(__builtin_amdgcn_ballot_w64(seg));
                }
            }
            cnt = uni(cnt);
            if (cnt > 0) {
                uint32_t pos = 0;
                if (lane == 0) {
                    pos = __hip_atomic_fetch_add(&st->bq_res, (uint32_t)cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_fetch_add(&st->bq_live, (uint32_t)cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                pos = (uint32_t)uni((int32_t)pos);
                uint32_t at = pos;
                const int32_t parts = root ? pp : 1;
                for (int32_t k0 = 0; k0 < parts; k0 += 64) {
                    const int32_t k = k0 + lane;
                    int32_t lo, hi;
                    if (root) {
                        lo = k == 0 ? 0 : (int32_t)seg_end(T, pp, min(k, pp) - 1) + 1;
                        hi = (int32_t)seg_end(T, pp, min(k, pp - 1));
                    } else {
                        lo = tmid + 1;
                        hi = n;
                    }
                    const bool seg = k < parts && hi > lo;
                    const uint64_t mask = __builtin_amdgcn_ballot_w64(seg);
                    if (seg) {
                        const uint32_t p = at + (uint32_t)__popcll(mask & ((1ull << lane) - 1));
                        if ((int64_t)p < a.q_cap) {
                            uint64_t* qe = reinterpret_cast<uint64_t*>(a.queue + p);
                            st_c(qe, (uint64_t)(uint32_t)seq | ((uint64_t)KIND_BSUB << 32));
                            st_c(qe + 1, (uint64_t)(uint32_t)lo | ((uint64_t)(uint32_t)hi << 32));
                        }
                    }
                    at += (uint32_t)__popcll(mask);
                }
                // path, scores and tasks are at the memory side before the publication
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                __builtin_amdgcn_s_waitcnt(0);
                if (lane == 0) {
                    // publications follow the reservations' order (the earlier one is
                    // being written by a running block); none after a wait that gave up
                    bool next = false;
                    for (int64_t turn = 0; !(next = ld_c(&st->bq_pub) == pos) && !wait_over(a, turn, false); ++turn)
                        __builtin_amdgcn_s_sleep(1);
                    if (next)
                        __hip_atomic_fetch_add(&st->bq_pub, (uint32_t)cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            } else {
                __builtin_amdgcn_s_waitcnt(0);
            }
            if (lane == 0 && sp == 0)
                __hip_atomic_fetch_sub(&st->bq_live, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if constexpr (SPARSE)
            if (retry) {   // a push that found no room leaves its count
                __syncthreads();
                if (tid == 0) s.ncand = 0;
            }
    }
    // ---- the last block hands the engine its tasks
    __syncthreads();
    if (tid == 0) {
        __builtin_amdgcn_s_waitcnt(0);
        s.sv_[0] = __hip_atomic_fetch_add(&st->bq_done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == gridDim.x;
    }
    __syncthreads();
    if (!s.sv_[0]) return;
    const int64_t half = a.q_cap / 2;
    const int32_t left = (int32_t)min((int64_t)ld_c(&st->bq_left), a.q_cap - half);
    for (int32_t k = tid; k < left; k += kBThreads) {
        const unsigned long long* p = reinterpret_cast<const unsigned long long*>(a.queue + half + k);
        uint64_t* qe = reinterpret_cast<uint64_t*>(a.queue + k);
        st_c(qe, (uint64_t)ld_c(p));
        st_c(qe + 1, (uint64_t)ld_c(p + 1));
    }
    if (tid == 0) st->q_tail0 = left;
}

extern "C" __global__ __launch_bounds__(kBThreads, 4) void fv_beam_dense_kernel(const EngineArgs* __restrict__ table) {
    beam_decode<false>(*reinterpret_cast<cargs_t*>(reinterpret_cast<uint64_t>(table)));
}
extern "C" __global__ __launch_bounds__(kBThreads, 4) void fv_beam_sparse_kernel(const EngineArgs* __restrict__ table) {
    beam_decode<true>(*reinterpret_cast<cargs_t*>(reinterpret_cast<uint64_t>(table)));
}

}  // namespace fv
