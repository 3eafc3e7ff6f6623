// Schedule "rows": every (target, draft) row pair is read from HBM once, by workgroups that each keep one row pair
// (or one of its P parts) in registers.
//
//   k_rows : workgroup (prefix, draft, row, part), part fastest:
//                    1. loads its part of the row pair (every load issued before the first is used)
//                    2. sweep 1: the part's soft-max statistics, log2 sum_x 2^(c z[x]) of either row, which it leaves in
//                       the workspace (two 64-bit device-scope words per row, which say by themselves that they are there)
//                    3. collects the statistics of its draft's rows 0 .. i from the workgroups that own them
//                    4. sweep 2, from the registers: the part's share of the vocabulary sum of Eq. (hik)
//                         s_i = sum_x q_i[x] max(1 - p_i[x] / (nu_i q_i[x]), 0)^K
//
// What bounds it: the chain schedule walks a draft's rows in one workgroup per compute unit, which is right where a
// row pair fills the compute unit; shorter rows leave it waiting on the row's own latencies (9.4 us per row of 32000
// bfloat16 entries, of which 5 us are arithmetic), and a number of drafts that is not a multiple of the compute units
// leaves some idle for a whole draft.  Here a row is the unit of work, two to four workgroups share a compute unit,
// and one's loads run beside another's arithmetic.
//
// A normaliser is there when the exclusive or of its two words is the call's own number (call_nonce: no two calls of a process
// have the same, so whatever the workspace held before, words of an earlier call among it, is not taken for one).  A call
// captured in a graph has the same number in every replay; the final-token kernel, which runs behind this one and reads none
// of the words, therefore clears them.  (A kernel in front that marks the words as not there yet, which this one had before,
// cost 2 - 5 us a call.)  The four words of a part, two of either model, share 32 bytes, so that they are looked for in as many
// memory accesses as two words in places of their own were: one prompt of 3 drafts, V = 128256 28.8 us a call with the models'
// words apart, 28.0 now; 128 x 16 of 8, V = 4000 bfloat16 212.2 / 211.1; 64 x 8 of 8, V = 8000 78.4 / 77.8.  (All words of a
// draft without gaps: whole rows' words then share lines between workgroups, V = 4000 219.)
//
// Step 3 waits for workgroups with a lower index only (the same draft's earlier rows) or with the same row (its other
// parts); workgroups are dispatched in index order, so what is waited for is running or has run.  Nothing relies on
// it: after `polls` looks a workgroup computes what is missing itself, from memory, by the code of steps 1 and 2 (the
// same bits).
//
// Rows may start at any address and have any length of at least one vector: 16-byte loads need no alignment on this
// hardware, and a last vector that is not whole is loaded from the row's last 16 bytes with the entries that belong
// to the vector before it masked.
#include "specgbv_internal.hpp"

namespace specgbv {
namespace {

constexpr int kRowsMaxL = 64;                          // rows of a draft (L <= 62)
static_assert(sizeof(Row0Part) == kWordsPerPart * sizeof(unsigned long long), "the words take the room of a part's statistics");

struct RowsArgs {
    const int32_t *tokens;
    unsigned long long *words;     // [n_rows][kRowParts][2][2] log2-normalisers of the parts: float64 bits, and those ^ nonce
    unsigned long long nonce;
    int32_t *final_counter;        // [batch] arrival counters of the final-token kernel, cleared here
    RowStat *stats;
    double *s_out, *e_out;         // P = 1: the row's sum, and nu^2 (s - g) where it is needed (else -1)
    double *s_part, *e_part;       // P > 1: the parts' sums; the final-token kernel's parts of E start as "not there yet"
    int K, L, V, logP, polls;      // P = 1 << logP parts per row
    float c;
    double c_rel;
};

constexpr unsigned long long kNotThere = ~0ull;        // a word that has not been found yet (a NaN that no sum produces)

// This thread's vectors of units [lo, lo + n) of a row pair, n <= NS * TH.  Every slot is loaded, without a
// branch (a load under one is waited for where the branch ends): lanes and slots past the part's end read masked
// entries, so that the sweeps need not look at the lane, and a row's last vector that is not whole is loaded from the
// row's last 16 bytes, with the entries that belong to the vector before it masked (Slots::unpack).
template <typename T, int TH, int NS>
__device__ __forceinline__ void rows_load(const T *rq, const T *rp, int lo, int n, int V, U4 (&q)[NS], U4 (&p)[NS])
{
    constexpr int PV = Elem<T>::kPerVec;
    const int tid = threadIdx.x;
    const T *dead = masked_vector<T>();
#pragma unroll
    for (int j = 0; j < NS; ++j) {
        const int v = j * TH + tid;
        const bool live = v < n;
        int e = (lo + v) * PV;
        e = e < V - PV ? e : V - PV;
        q[j] = load16_stream_any(live ? rq + e : dead);
        p[j] = load16_stream_any(live ? rp + e : dead);
    }
}

// Which of the loaded entries count.
template <typename T, int TH>
struct Slots {
    int n, before;           // vectors of the part; entries of its last vector that belong to the one before (0: it is whole)
    __device__ __forceinline__ Slots(int lo, int n_, int V)
    {
        constexpr int PV = Elem<T>::kPerVec;
        const int rem = V % PV;
        n = n_;
        before = (rem != 0 && lo + n_ == (V + PV - 1) / PV) ? PV - rem : 0;
    }
    __device__ __forceinline__ bool used(int j) const { return j * TH < n; }          // uniform
    template <int N>
    __device__ __forceinline__ void unpack(const U4 &v, int j, float (&z)[N]) const
    {
        Elem<T>::unpack(v, z);
        if (before > 0) {                                  // uniform
            asm volatile("");
            if (j * TH + static_cast<int>(threadIdx.x) == n - 1) {
#pragma unroll
                for (int e = 0; e < N; ++e) z[e] = e < before ? -__builtin_inff() : z[e];
            }
        }
    }
};

// A slot's registers (and a running value) pass through a point in program order: the floats unpacked from a slot are
// neither formed ahead of time nor kept for the next sweep, which would double the registers the slots take.
__device__ __forceinline__ void rows_touch(U4 &v, float &acc)
{
    asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w), "+v"(acc));
}

// Sum over this wave's vectors (the drafted token's entry left out) of 2^(c z - ref), ref integral.  Every lane keeps a
// running reference, the largest entry so far, updated once per vector: the entries that make up a row's mass then
// have small exponents, which float32 rounds little, and the largest weigh exactly 1.  A workgroup of 256 threads does so for
// either half of its slots by itself, so that as many entries share a reference as with 512.  Error of ln Z, rms, bfloat16 rows
// of 8000 / 16000 entries at T = 0.7: 3.05e-8 / 3.1e-8, as on the two-pass schedule; updated once per 16 entries, without the
// halves, 4.0e-8 / 4.1e-8, and no faster.  (A reference taken from the wave's first vectors alone saves a tenth of the sweep
// and costs five times the error at T = 0.4: 2.7e-7 instead of 6e-8 in ln nu.)
struct WaveSum { float ref; double Z; };
struct TokenAt { int slot, elem; bool mine; };             // where the drafted token lies: slot (uniform, -1: not here), entry, this lane?

template <typename T, int TH, int NS>
__device__ __forceinline__ WaveSum rows_wave_sum(U4 (&v)[NS], const Slots<T, TH> &sl, float c, const TokenAt &tk)
{
    constexpr int PV = Elem<T>::kPerVec, A = 512 / TH;
    static_assert(A == 1 || A == 2, "workgroups of 256 or 512 threads");
    float m2[A], Z[A];
#pragma unroll
    for (int x = 0; x < A; ++x) {
        float m = -3.0e38f, zs = 0.0f;
#pragma unroll
        for (int j = x * (NS / A); j < (x + 1) * (NS / A); ++j) {
            if (sl.used(j)) {
                rows_touch(v[j], zs);
                float z[PV], vm = -3.0e38f;
                sl.unpack(v[j], j, z);
                if (j == tk.slot) {                        // uniform
                    asm volatile("");
                    leave_out(z, tk.mine, tk.elem);
                }
#pragma unroll
                for (int e = 0; e < PV; ++e) vm = fmaxf(vm, z[e]);
                const float n2 = fmaxf(m, vm * c);
                float a = 0.0f;
#pragma unroll
                for (int e = 0; e < PV; ++e) a += exp2_fast(fmaf(z[e], c, -n2));
                zs = fmaf(zs, exp2_fast(m - n2), a);
                m = n2;
            }
        }
        m2[x] = m; Z[x] = zs;
    }
    float top = m2[0];
#pragma unroll
    for (int x = 1; x < A; ++x) top = fmaxf(top, m2[x]);
    WaveSum s;
    s.ref = ceilf(fmaxf(wave_max(top), -3.0e38f));
    double lane = 0.0;
#pragma unroll
    for (int x = 0; x < A; ++x)
        lane += Z[x] > 0.0f ? static_cast<double>(Z[x]) * exp2_small(static_cast<double>(m2[x]) - static_cast<double>(s.ref)) : 0.0;
    s.Z = wave_sum(lane);
    return s;
}

// E = nu^2 (s - g) of a whole row pair, from memory (rare rows; see excess_needed), by the whole workgroup.
template <typename T, int TH>
__device__ __forceinline__ double rows_excess(const T *rq, const T *rp, int V, double lse2_q, double lse2_p, double log2nu, int K,
                                           float c, double *sh_d)
{
    constexpr int PV = Elem<T>::kPerVec;
    constexpr int kAhead = 2;
    const ExcessConst ec = make_excess_const(lse2_q, lse2_p, log2nu, K, c);
    const int nv = (V + PV - 1) / PV, rem = V % PV;
    float acc = 0.0f;
    for (int v0 = threadIdx.x; v0 < nv; v0 += kAhead * TH) {
        U4 q[kAhead], p[kAhead];
#pragma unroll
        for (int a = 0; a < kAhead; ++a) {
            const int v = v0 + a * TH;
            int e = (v < nv ? v : v0) * PV;
            e = e < V - PV ? e : V - PV;
            q[a] = load16_stream_any(rq + e);
            p[a] = load16_stream_any(rp + e);
        }
#pragma unroll
        for (int a = 0; a < kAhead; ++a) {
            const int v = v0 + a * TH;
            float zq[PV], zp[PV];
            Elem<T>::unpack(q[a], zq);
            Elem<T>::unpack(p[a], zp);
            if (rem != 0 && v == nv - 1) {
#pragma unroll
                for (int e = 0; e < PV; ++e)
                    if (e < PV - rem) { zq[e] = -__builtin_inff(); zp[e] = -__builtin_inff(); }
            }
            if (v < nv) acc += excess_terms(zq, zp, ec);
        }
    }
    return block_sum(static_cast<double>(acc), sh_d) * ec.scale;
}

// Registers: the tile of two vectors needs all 80 of its six waves per SIMD, and what it cannot keep costs more than anything
// else here.  With the drafted tokens' addresses kept around the loop, and the counters cleared behind sweep 1, four of them and
// eight scalars more were spilled: 128 x 16 drafts of 8, V = 4000 bfloat16 225.6 us a call, 212.2 without; 128 x 8 of 4, V = 8000
// 80.9 / 77.2; float32 128 x 16 of 8, V = 4000 228.4 / 215.7.
template <typename T, int TH, int NS>
__global__ void __launch_bounds__(TH, NS >= 4 ? 4 : 6)
k_rows(const T *__restrict__ target, const T *__restrict__ draft, RowsArgs ar)
{
    constexpr int kRowsWaves = TH / kWave;
    __shared__ double sh_word[2 * kRowsMaxL * kRowParts];  // the parts' log2-normalisers of rows 0 .. i
    __shared__ double sh_lse[2 * kRowsMaxL], sh_tok[2 * kRowsMaxL];
    __shared__ double sh_Z[2 * kRowsWaves], sh_own[2];
    __shared__ float sh_ref[2 * kRowsWaves];
    __shared__ int sh_missing, sh_again;
    constexpr int PV = Elem<T>::kPerVec;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    const int K = ar.K, L = ar.L, V = ar.V, logP = ar.logP, P = 1 << logP;
    const float c = ar.c;
    const unsigned pair_u = blockIdx.x >> logP;
    const int part = static_cast<int>(blockIdx.x & (P - 1));
    const long long pair = pair_u, bk = pair_u / static_cast<unsigned>(L);
    const int i = static_cast<int>(pair - bk * L);
    const int nv = (V + PV - 1) / PV, per = (nv + P - 1) >> logP;
    if (tid == 0) {
        sh_missing = 0x7fffffff;
        if (part == 0 && pair_u % static_cast<unsigned>(K * L) == 0u) ar.final_counter[pair_u / static_cast<unsigned>(K * L)] = 0;
    }

    // the drafted tokens of rows 0 .. i: thread 2 j + m looks after row j of the target (m = 0) or the draft (1)
    const int nstat = 2 * (i + 1);
    const int mt = tid & 1;
    uint32_t ztok = 0;
    U4 q[NS], p[NS];
    int r_now = i, part_now = part;                        // whose vectors q, p hold (uniform)
    unsigned long long *const words = ar.words + bk * L * (2 * kRowParts * kWordsPerPart);
    const int nwords = nstat * P;                          // word w: row w / (2 P), model w / P % 2, part w % P
    auto word_at = [&](int w) {
        return words + (((w >> (logP + 1)) * kRowParts + (w & (P - 1))) * 2 + ((w >> logP) & 1)) * kWordsPerPart;
    };
    for (bool first = true;; first = false) {
        const T *rq = target + (bk * (L + 1) + r_now) * static_cast<long long>(V);
        const T *rp = draft + (bk * L + r_now) * static_cast<long long>(V);
        const int lo = part_now * per, hi = lo + per < nv ? lo + per : nv, n = hi > lo ? hi - lo : 0;
        // (threads beyond nstat repeat the last row's: a load under a branch is waited for where the branch ends.  Opaque, so that
        // the addresses are made here and not kept in registers around the loop)
        int jt = (tid >> 1) < i ? (tid >> 1) : i;
        asm volatile("" : "+v"(jt));
        const int tok_raw = token_index_queued(ar.tokens, bk * L + r_now), tok_t = ar.tokens[bk * L + jt];
        rows_load<T, TH, NS>(rq, rp, lo, n, V, q, p);
        {                                                  // (behind the row's loads, needed after sweep 1 only)
            const int x = token_index_used(tok_t, V);
            ztok = Elem<T>::bits(mt ? draft + (bk * L + jt) * static_cast<long long>(V) + x
                                    : target + (bk * (L + 1) + jt) * static_cast<long long>(V) + x);
        }
        const Slots<T, TH> sl(lo, n, V);
        const int tok = token_index_used(tok_raw, V), tok_v = tok / PV - lo;   // the token's vector, counted from the part's first
        const bool tok_here = tok_v >= 0 && tok_v < n;
        TokenAt tk;
        tk.slot = __builtin_amdgcn_readfirstlane(tok_here ? tok_v / TH : -1);
        tk.mine = tok_here && tid == tok_v % TH;
        tk.elem = tok - (tok / PV * PV < V - PV ? tok / PV * PV : V - PV);     // counted from where that vector was loaded
        // sweep 1
        const WaveSum sq = rows_wave_sum<T, TH, NS>(q, sl, c, tk), sp = rows_wave_sum<T, TH, NS>(p, sl, c, tk);
        if (lane == 0) {
            sh_ref[wid] = sq.ref; sh_ref[kRowsWaves + wid] = sp.ref;
            sh_Z[wid] = sq.Z; sh_Z[kRowsWaves + wid] = sp.Z;
        }
        __syncthreads();
        if (tid < 2) {                                     // thread m: the waves' sums and, where it lies here, the token's weight
            float M = -3.0e38f;
#pragma unroll
            for (int w = 0; w < kRowsWaves; ++w) M = fmaxf(M, sh_Z[tid * kRowsWaves + w] > 0.0 ? sh_ref[tid * kRowsWaves + w] : -3.0e38f);
            double Z = 0.0;
#pragma unroll
            for (int w = 0; w < kRowsWaves; ++w)
                Z += ldexp(sh_Z[tid * kRowsWaves + w], reference_shift(sh_ref[tid * kRowsWaves + w], M));
            double ref = static_cast<double>(M);
            if (tok_here) {
                const double t = static_cast<double>(Elem<T>::scalar((tid ? rp : rq) + tok)) * static_cast<double>(c);
                const double top = Z > 0.0 ? fmax(ref, t) : t;
                Z = (Z > 0.0 ? Z * exp2_small(ref - top) : 0.0) + (t - top == 0.0 ? 1.0 : exp2_small(t - top));
                ref = top;
            }
            const double l = (Z > 0.0 && ref > -1.0e300) ? ref + log2_series(Z) : -static_cast<double>(__builtin_inff());
            sh_own[tid] = l;
            if (first) {
                unsigned long long *const dst = words + ((r_now * kRowParts + part_now) * 2 + tid) * kWordsPerPart;
                const unsigned long long bits = static_cast<unsigned long long>(__double_as_longlong(l));
                __hip_atomic_store(dst, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(dst + 1, bits ^ ar.nonce, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        if (first && i == 0 && L > 1) return;              // row 0 has no sum; the workgroup of row 1 stores its statistics
        __syncthreads();
        // collect (first pass), or put what this pass has computed in its place; then look for what is still missing
        for (int w = tid; w < nwords; w += TH) {
            const int m = (w >> logP) & 1;
            unsigned long long bits;
            if ((w >> (logP + 1)) == r_now && (w & (P - 1)) == part_now) bits = static_cast<unsigned long long>(__double_as_longlong(sh_own[m]));
            else if (first) {
                bits = kNotThere;
                const unsigned long long *const src = word_at(w);
                for (int look = 0; look < ar.polls && bits == kNotThere; ++look) {
                    const unsigned long long v = __hip_atomic_load(src, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    const unsigned long long x = __hip_atomic_load(src + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if ((v ^ x) == ar.nonce) bits = v;     // (one word of this call beside one of another is not)
                    else __builtin_amdgcn_s_sleep(2);
                }
            } else bits = static_cast<unsigned long long>(__double_as_longlong(sh_word[w]));
            sh_word[w] = __longlong_as_double(static_cast<long long>(bits));
            if (bits == kNotThere) atomicMin(&sh_missing, w);
        }
        __syncthreads();
        const int miss = __builtin_amdgcn_readfirstlane(sh_missing);
        __syncthreads();
        if (tid == 0) sh_missing = 0x7fffffff;
        if (miss == 0x7fffffff) break;
        r_now = miss >> (logP + 1); part_now = miss & (P - 1);       // computed here, both models of it, in the next pass
    }
    const T *rq = target + (bk * (L + 1) + i) * static_cast<long long>(V);
    const T *rp = draft + pair * static_cast<long long>(V);
    const int lo = part * per, hi = lo + per < nv ? lo + per : nv, n = hi > lo ? hi - lo : 0;
    if (r_now != i || part_now != part) {                  // (uniform) the registers hold another row's part: this one's again
        rows_load<T, TH, NS>(rq, rp, lo, n, V, q, p);
    }
    // the parts of each normaliser meet (groups of P lanes, P a power of two: the same bits in every workgroup)
    for (int w0 = 0; w0 < nwords; w0 += TH) {    // uniform
        const int w = w0 + tid;
        const double l = w < nwords ? sh_word[w] : -static_cast<double>(__builtin_inff());
        double top = l;
        for (int o = 1; o < P; o <<= 1) top = fmax(top, __shfl_xor(top, o));
        double lse = l;
        if (P > 1) {
            double Z = l > -1.0e300 ? exp2_small(l - top) : 0.0;
            for (int o = 1; o < P; o <<= 1) Z += __shfl_xor(Z, o);
            lse = top > -1.0e300 ? top + log2_series(Z) : top;
        }
        if (w < nwords && (w & (P - 1)) == 0) sh_lse[w >> logP] = lse;
    }
    __syncthreads();
    if (tid < nstat) sh_tok[tid] = token_scaled(static_cast<double>(Elem<T>::from_bits(ztok)) * static_cast<double>(c), sh_lse[tid], ar.c_rel);
    __syncthreads();
    RowStat st;
    st.lse2_q = sh_lse[2 * i]; st.lse2_p = sh_lse[2 * i + 1];
    st.tok2_q = sh_tok[2 * i]; st.tok2_p = sh_tok[2 * i + 1];
    if (part == 0 && tid == 0) {
        ar.stats[pair] = st;
        if (i == 1) {
            RowStat s0;
            s0.lse2_q = sh_lse[0]; s0.lse2_p = sh_lse[1]; s0.tok2_q = sh_tok[0]; s0.tok2_p = sh_tok[1];
            ar.stats[bk * L] = s0;
        }
    }
    if (i == 0) return;                                    // (L = 1)
    double log2nu = 0.0, log2P = 0.0;
    for (int j = 0; j < i; ++j) {
        const double lp = sh_tok[2 * j + 1] - sh_lse[2 * j + 1];
        log2nu += (sh_tok[2 * j] - sh_lse[2 * j]) - lp;
        log2P += lp;
    }
    // sweep 2
    const float shift_q = static_cast<float>(st.lse2_q);
    const RatioConst rc(ratio_const(st.lse2_p, st.lse2_q, log2nu, ar.c_rel));
    const Slots<T, TH> sl(lo, n, V);
    float acc = 0.0f;
#pragma unroll
    for (int j = 0; j < NS; ++j) {
        if (sl.used(j)) {
            rows_touch(q[j], acc);
            rows_touch(p[j], acc);
            // (the terms of ot_weights, the last product taken with the sum)
            float zq[PV], zp[PV], t[PV], a = 0.0f;
            sl.unpack(q[j], j, zq);
            sl.unpack(p[j], j, zp);
#pragma unroll
            for (int e = 0; e < PV; ++e) t[e] = rc.one_minus_ratio(zp[e] - zq[e], c);
            pow_array(t, K);
#pragma unroll
            for (int e = 0; e < PV; ++e) a = fmaf(exp2_fast(fmaf(zq[e], c, -shift_q)), t[e], a);
            acc += a;
        }
    }
    double total = block_sum(static_cast<double>(acc), sh_Z);
    if (tid == 0) {
        total = with_token_term<T, true>(total, st, log2nu, rq, rp, ar.tokens + pair, V, lo * PV, hi * PV < V ? hi * PV : V, c, shift_q, rc, K);
        const double s = total * exp2_small(static_cast<double>(shift_q) - st.lse2_q);
        if (P > 1) {
            ar.s_part[pair * kPendParts + part] = s;
        } else {
            ar.s_out[pair] = s;
            // where s and g nearly cancel, Eq. (hik) needs nu^2 (s - g) summed term by term (see excess_wanted)
            const bool again = excess_wanted(static_cast<float>(log2nu), static_cast<float>(s), K) && excess_needed(log2nu, log2P, s, K);
            sh_again = again ? 1 : 0;
            if (!again) ar.e_out[pair] = -1.0;
        }
    }
    if (P > 1) {                                           // only the sum over all parts can tell: the final-token kernel looks at it
        if (part == 0 && tid < kPendParts) ar.e_part[pair * kPendParts + tid] = -1.0;
        return;
    }
    __syncthreads();
    if (sh_again) {                                        // uniform
        const double e = rows_excess<T, TH>(rq, rp, V, st.lse2_q, st.lse2_p, log2nu, K, c, sh_Z);
        if (tid == 0) ar.e_out[pair] = e;
    }
}

// Short rows (short_rows): one workgroup per draft, one wave per row pair, both sweeps in one launch.
// A row is a few loads per lane here, and what such a call takes is launches and barriers: K = 2, L = 4, V = 1000 float32
// took 4.3 + 3.6 us in two kernels and the gap between them (19.1 us a call), and takes 17.5 us a call.
constexpr int kShortRows = 16;                         // waves of a workgroup, and rows of a draft

// The range of k_short_rows.  Its terms of sweep 1 are summed in float64 (a lane adds up to 32 entries of a row, and in
// float32 the error of ln nu would be 3e-7 where the other schedules' lanes, with fewer entries each, have 1.2e-7).  With
// few drafts the time of one row counts: one prompt, L = 8, bfloat16, a call takes 18.0 us with V = 1024 and 22.8 with
// V = 2048, on the other schedules 19.0 and 19.5.  With a draft for every compute unit, the workgroups and barriers per
// row count: 64 x 4 drafts of 8, V = 2048, 32.5 us and 46.5, 500 x 8 of 16 355 and 820; 40 x 2 of 16 still 37.3 and 35.0.
bool short_rows(const Problem &p)
{
    const long long drafts = static_cast<long long>(p.batch) * p.K;
    return (p.V <= 1024 && p.L <= 8) || (p.V <= 2048 && p.L <= kShortRows && drafts >= compute_units());
}

template <typename T>
__global__ void __launch_bounds__(kShortRows * kWave)
k_short_rows(const T *__restrict__ target, const T *__restrict__ draft, const int32_t *__restrict__ tokens, int K, int L, int V,
             float c, double c_rel, RowStat *__restrict__ stats, double *__restrict__ s_out, double *__restrict__ e_out,
             int32_t *__restrict__ final_counter)
{
    __shared__ double sh_lse[2 * kShortRows], sh_tok[2 * kShortRows];
    constexpr int PV = Elem<T>::kPerVec;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), r = __builtin_amdgcn_readfirstlane(tid / kWave);   // wave r: row pair r
    const int nv = row_vectors<T>(V);
    const long long bk = blockIdx.x;
    if (tid == 0 && bk % K == 0) final_counter[bk / K] = 0;              // arrival counter of the final-token kernel
    const T *const rq = target + (bk * (L + 1) + r) * static_cast<long long>(V);
    const T *const rp = draft + (bk * L + r) * static_cast<long long>(V);
    // f(v, z_q, z_p) for this lane's vectors of the row pair
    auto sweep = [&](auto f) {
        for (int v = lane; v < nv; v += 2 * kWave) {
            const int w = v + kWave < nv ? v + kWave : v;                // (no branch around a load)
            const U4 q0 = load16_stream_any(rq + vector_entry<T>(v, V)), p0 = load16_stream_any(rp + vector_entry<T>(v, V));
            const U4 q1 = load16_stream_any(rq + vector_entry<T>(w, V)), p1 = load16_stream_any(rp + vector_entry<T>(w, V));
            float zq[PV], zp[PV];
            Elem<T>::unpack(q0, zq); Elem<T>::unpack(p0, zp);
            mask_repeated<T>(zq, v, V); mask_repeated<T>(zp, v, V);
            f(v, zq, zp);
            if (w != v) {
                Elem<T>::unpack(q1, zq); Elem<T>::unpack(p1, zp);
                mask_repeated<T>(zq, w, V); mask_repeated<T>(zp, w, V);
                f(w, zq, zp);
            }
        }
    };
    int tok = tokens[bk * L + r];
    tok = tok < 0 ? 0 : (tok >= V ? V - 1 : tok);
    const float ztok = Elem<T>::scalar((lane & 1) ? rp + tok : rq + tok);
    RunningSum64 aq, ap;                               // the drafted token is left out (leave_out)
    const int tok_v = tok / PV, tok_e = tok - vector_entry<T>(tok / PV, V);
    sweep([&](int v, float (&zq)[PV], float (&zp)[PV]) {
        leave_out(zq, v == tok_v, tok_e);
        leave_out(zp, v == tok_v, tok_e);
        aq.add(zq, c);
        ap.add(zp, c);
    });
    const float Mq = wave_max(aq.m2), Mp = wave_max(ap.m2);
    const double Zq = wave_sum(aq.Z > 0.0 ? aq.Z * exp2_small(static_cast<double>(aq.m2) - static_cast<double>(Mq)) : 0.0);
    const double Zp = wave_sum(ap.Z > 0.0 ? ap.Z * exp2_small(static_cast<double>(ap.m2) - static_cast<double>(Mp)) : 0.0);
    {                                                  // even lanes: the target's row, odd lanes: the draft's
        const double Z0 = (lane & 1) ? Zp : Zq, ref = static_cast<double>((lane & 1) ? Mp : Mq);
        const double t = static_cast<double>(ztok) * static_cast<double>(c);
        const double top = Z0 > 0.0 ? fmax(ref, t) : t;
        const double Z = (Z0 > 0.0 ? Z0 * exp2_small(ref - top) : 0.0) + (t - top == 0.0 ? 1.0 : exp2_small(t - top));
        const double lse = top + log2_series(Z);
        if (lane < 2) { sh_lse[2 * r + lane] = lse; sh_tok[2 * r + lane] = token_scaled(t, lse, c_rel); }
    }
    __syncthreads();
    RowStat st;
    st.lse2_q = sh_lse[2 * r]; st.lse2_p = sh_lse[2 * r + 1];
    st.tok2_q = sh_tok[2 * r]; st.tok2_p = sh_tok[2 * r + 1];
    if (lane == 0) stats[bk * L + r] = st;
    if (r == 0) return;
    const int j = lane < r ? lane : 0;                 // lane j: row j of the rows before this one
    const double lp = lane < r ? sh_tok[2 * j + 1] - sh_lse[2 * j + 1] : 0.0;
    const double log2P = wave_sum(lp);
    const double log2nu = wave_sum(lane < r ? sh_tok[2 * j] - sh_lse[2 * j] - lp : 0.0);
    const float shift_q = static_cast<float>(st.lse2_q);
    const RatioConst rc(ratio_const(st.lse2_p, st.lse2_q, log2nu, c_rel));
    double acc = 0.0;
    sweep([&](int, float (&zq)[PV], float (&zp)[PV]) {
        float wq[PV], w[PV];
        ot_weights(zq, zp, c, shift_q, rc, K, wq, w);
#pragma unroll
        for (int e = 0; e < PV; ++e) acc += static_cast<double>(w[e]);
    });
    const double total = with_token_term<T>(wave_sum(acc), st, log2nu, rq, rp, tokens + (bk * L + r), V, 0, V,
                                            c, shift_q, rc, K);
    const double s = total * exp2_small(static_cast<double>(shift_q) - st.lse2_q);
    double e = -1.0;
    // where s and g nearly cancel, Eq. (hik) needs nu^2 (s - g) summed term by term (see excess_wanted; wave-uniform)
    if (excess_wanted(static_cast<float>(log2nu), static_cast<float>(s), K) && excess_needed(log2nu, log2P, s, K)) {
        const ExcessConst ec = make_excess_const(st.lse2_q, st.lse2_p, log2nu, K, c);
        double ex = 0.0;
        sweep([&](int, float (&zq)[PV], float (&zp)[PV]) {
#pragma unroll
            for (int x = 0; x < PV; ++x) {
                const float q1[1] = {zq[x]}, p1[1] = {zp[x]};
                ex += static_cast<double>(excess_terms(q1, p1, ec));
            }
        });
        e = wave_sum(ex) * ec.scale;
    }
    if (lane == 0) { s_out[bk * L + r] = s; e_out[bk * L + r] = e; }
}

template <typename T>
hipError_t launch_rows_typed(const Problem &p)
{
    constexpr int PV = Elem<T>::kPerVec;
    const long long pairs = static_cast<long long>(p.batch) * p.K * p.L;
    const int P = p.rows_parts;
    if (short_rows(p)) {
        hipLaunchKernelGGL((k_short_rows<T>), dim3(static_cast<unsigned>(p.batch) * static_cast<unsigned>(p.K)),
                           dim3(static_cast<unsigned>(p.L) * kWave), 0, p.stream,
                           static_cast<const T *>(p.target), static_cast<const T *>(p.draft), p.tokens, p.K, p.L, p.V, p.c, p.c_rel,
                           reinterpret_cast<RowStat *>(p.ws + p.lay.stats), reinterpret_cast<double *>(p.ws + p.lay.s),
                           reinterpret_cast<double *>(p.ws + p.lay.excess), reinterpret_cast<int32_t *>(p.ws + p.lay.counter));
        return hipGetLastError();
    }
    RowsArgs ar;
    ar.tokens = p.tokens;
    ar.words = reinterpret_cast<unsigned long long *>(p.ws + p.lay.stat_part);
    ar.stats = reinterpret_cast<RowStat *>(p.ws + p.lay.stats);
    ar.s_out = reinterpret_cast<double *>(p.ws + p.lay.s);
    ar.e_out = reinterpret_cast<double *>(p.ws + p.lay.excess);
    ar.s_part = reinterpret_cast<double *>(p.ws + p.lay.pend_part);
    ar.e_part = reinterpret_cast<double *>(p.ws + p.lay.excess_part);
    ar.K = p.K; ar.L = p.L; ar.V = p.V; ar.logP = __builtin_ctz(static_cast<unsigned>(P)); ar.polls = wait_polls();
    ar.c = p.c; ar.c_rel = p.c_rel;
    ar.nonce = p.nonce;
    ar.final_counter = reinterpret_cast<int32_t *>(p.ws + p.lay.counter);
    const T *target = static_cast<const T *>(p.target), *draft = static_cast<const T *>(p.draft);
    const int nv = (p.V + PV - 1) / PV, per = (nv + P - 1) / P;
    const dim3 grid(static_cast<unsigned>(pairs * P));
#define SPECGBV_ROWS_LAUNCH(TH, NS) hipLaunchKernelGGL((k_rows<T, TH, NS>), grid, dim3(TH), 0, p.stream, target, draft, ar)
    if (per <= 1024) SPECGBV_ROWS_LAUNCH(512, 2);
    else if (per <= 1536) SPECGBV_ROWS_LAUNCH(256, 6);
    else if (per <= 2048) SPECGBV_ROWS_LAUNCH(256, 8);
    else SPECGBV_ROWS_LAUNCH(512, 8);
#undef SPECGBV_ROWS_LAUNCH
    return hipGetLastError();
}

}  // namespace

int rows_schedule_parts(const Problem &p)
{
    const int pv = p.dtype == 1 ? 8 : 4;
    const long long pairs = static_cast<long long>(p.batch) * p.K * p.L;
    if (p.V < pv || p.L >= kRowsMaxL) return 0;
    const int nv = (p.V + pv - 1) / pv;
    if (short_rows(p)) return 1;                           // (k_short_rows: whole rows)
    if (!(p.dtype == 1 ? read_by_vectors<uint16_t>(p.V) : read_by_vectors<float>(p.V))) return 0;   // (two-pass, for accuracy)
    // few row pairs shorter than one load per thread: the two-pass kernels, which need no marks to wait on (V = 1000,
    // 8 float32 row pairs: 19.0 us a call against 20.0; from 200 row pairs on, or with longer rows, this schedule is ahead)
    if (nv < 512 && pairs * 2 <= compute_units()) return 0;
    static_assert((kRowParts & (kRowParts - 1)) == 0, "a power of two");
    int P = 1;
    // Two tiles: one workgroup of 512 threads for a row of up to 4096 vectors (its overheads once per row: V = 32000
    // bfloat16, 128 drafts of 8: 78 us a call, 93 in two parts), but four workgroups of 256 per compute unit, with parts
    // of up to 2048 vectors, for longer rows, whose parts must not wait for one another in step (V = 128256: 187 in eight
    // parts, 213 in four; 8 x 4 drafts of 5, V = 32000 float32: 35.8 in four, 38.6 in two).  Parts of up to 1536 vectors take
    // a tile of their own, whose halves are the same for every lane (8 x 4 drafts of 8, V = 70001 float32: 84.1, 85.3 in the
    // tile of 2048).
    const int most = nv <= 4096 ? 4096 : 2048;
    while (P < kRowParts && (nv + P - 1) / P > most) P *= 2;
    if ((nv + P - 1) / P > 4096) return 0;
    const long long units = compute_units();
    while (P < kRowParts && pairs * P * 2 <= 2 * units && nv / (P * 2) >= 512) P *= 2;
    // With more than 512 workgroups of this schedule (two per unit) the two-pass kernels, which read most rows a second time
    // but have no workgroup wait for another, are ahead (measured at 880 shapes of 4 - 4800 row pairs, V = 1024 - 152064)
    //   - of rows in parts, unless the parts fill their tile: a workgroup takes the compute units for 6.9 + 0.6 ns per 256
    //     vectors in bfloat16, 6.6 + 0.2 in float32, the two passes for 3.6 and 3.0 ns per 1000 vectors and pass.  32 x 4
    //     drafts of 4, us a call in rows / two passes: bfloat16 V = 66000 (1032 vectors per part) 85 / 70, 100000 (1563)
    //     106 / 100, 131072 (2048) 106 / 112; float32 V = 66000 (1032) 128 / 109, 100000 (1563) 154 / 148; 128 x 1 of 5,
    //     65536 (2048) 102 / 126; with more than 2048 per part, two workgroups per unit, 140000 (2188) 260 / 187;
    //   - of whole rows in the tile of 4096 vectors, two workgroups per unit, in bfloat16 (32 x 8 drafts of 8, V = 24000
    //     98.6 / 92.3; float32 20 x 8 of 6, V = 9000 46.6 / 54.3); with less than two rounds of workgroups, of either type, of
    //     short drafts, whose rows 0 are a good part, unless the second round is nearly full (bfloat16 128 x 1 of 5,
    //     V = 24000 49.2 / 43.6, 20 x 8 of 6 55.6 / 63.3, 100 x 2 of 5 62.3 / 65.7; 12 x 5 of 12, V = 25365 65.2 / 81.7).
    const int per = (nv + P - 1) / P;
    const long long wgs = pairs * P;
    if (per > 1024 && wgs > 2 * units) {
        if (P > 1) {
            if (per > 2048 || per < (p.dtype == 1 ? 1750 : 1400)) return 0;
        } else if (per > 2048) {
            if (wgs > 4 * units ? p.dtype == 1 : p.L < 6 && wgs * 4 < 14 * units) return 0;
        }
    }
    return pairs * P < (1LL << 31) ? P : 0;
}

bool short_rows_schedule(const Problem &p) { return short_rows(p); }

hipError_t launch_rows_main(const Problem &p)
{
    return p.dtype == 1 ? launch_rows_typed<uint16_t>(p) : launch_rows_typed<float>(p);
}

}  // namespace specgbv
