// Schedule "split": two streaming passes over the logits.
//
//   k_row_stats : per row, log2 sum_x 2^(c z[x]) and the token's scaled logit
//                 (soft-max statistics of the distributions Algorithm 1 takes as input)
//   k_ot_sum    : per row pair i = 1..L-1, the vocabulary sum of Eq. (hik) divided by
//                 q(x^i):  s_i = sum_x q_i[x] max(1 - p_i[x] / (nu_i q_i[x]), 0)^K
//
// With a pending distribution modification (Algorithm 2 applied on the fly) a third kernel
// runs between the two:
//   k_pend_norm : per modified row, the block ratio mu Algorithm 2 uses there, the normaliser
//                 N = sum_x q[x] max(1 - p[x] / (mu q[x]), 0)^K of q_new, and the drafted
//                 token's factor,
// and k_ot_sum evaluates its sum against q_new = q t^K / N formed per entry (k_pend_norm takes the
// levels in turn; a level's rows are shared among workgroups when it has few of them left).
//
// Small batches, where a workgroup per row would leave most of the chip idle, use k_row_stats_parts and
// k_ot_sum_parts instead: every row is cut into
// parts, combined in part order by the consumers.
//
// Any V and any alignment is accepted (16-byte loads need no alignment on this hardware; short rows that are not a
// multiple of the vector go entry by entry, see read_by_vectors).  This schedule reads every row pair twice; it serves
// pending modifications, a few short rows, and callers who ask for it, the reference for the schedules that read once.
#include "specgbv_internal.hpp"

namespace specgbv {
namespace {

constexpr int kStatThreads = 512;
constexpr int kMaxRows = 64;         // rows of a draft (L <= 62)
static_assert(kRowParts <= kPendParts, "a row's partial Eq. (hik) sums have kPendParts places");

// What the level passes need before they start (pending modifications only): per level l and prefix b the
// number of rows the level modifies in the prefixes before b, K * sum_{b' < b} clamp(count[l][b'], 0, L), with the
// level's total at position batch.  One workgroup per level.
__device__ __forceinline__ void pend_offsets(const int32_t *count_l, int K, int L, int batch, int32_t *off_l)
{
    __shared__ double sh_scan[kStatThreads / kWave];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    const int chunk = (batch + kStatThreads - 1) / kStatThreads;
    const int b0 = tid * chunk, b1 = b0 + chunk < batch ? b0 + chunk : batch;
    double mine = 0.0;                                 // small integers: exact in float64
    for (int b = b0; b < b1; ++b) {
        const int cnt = count_l[b];
        mine += static_cast<double>(K) * static_cast<double>(cnt < 0 ? 0 : (cnt > L ? L : cnt));
    }
    const double incl = wave_inclusive_sum(mine);
    if (lane == kWave - 1) sh_scan[wid] = incl;
    __syncthreads();
    double before = incl - mine;
    for (int w = 0; w < wid; ++w) before += sh_scan[w];
    for (int b = b0; b < b1; ++b) {
        off_l[b] = static_cast<int32_t>(before);
        const int cnt = count_l[b];
        before += static_cast<double>(K) * static_cast<double>(cnt < 0 ? 0 : (cnt > L ? L : cnt));
    }
    if (tid == kStatThreads - 1) off_l[batch] = static_cast<int32_t>(before);     // the last thread's end is the total
}

constexpr int kAhead = 4;            // loads a thread of k_row_stats keeps in flight

// Vector v of a row into its running sum, without the drafted token and without entries the vector before holds.
template <typename T>
__device__ __forceinline__ void add_entries(RunningSum &acc, float (&z)[Elem<T>::kPerVec], int v, int tok, int V, float c)
{
    constexpr int PV = Elem<T>::kPerVec;
    mask_repeated<T>(z, v, V);
    leave_out(z, v == tok / PV, tok - vector_entry<T>(v, V));
    acc.add(z, c);
}
template <typename T>
__device__ __forceinline__ void add_vector(RunningSum &acc, const U4 &raw, int v, int tok, int V, float c)
{
    float z[Elem<T>::kPerVec];
    Elem<T>::unpack(raw, z);
    add_entries<T>(acc, z, v, tok, V, c);
}

// grid (row pairs + pending levels, 2): blocks (pair, 0 / 1) reduce the target / draft row of the pair; with
// pending modifications blocks (pairs + l, 0) compute level l's offsets (pend_offsets) and the row blocks write the levels'
// entries of their row: empty, or not there yet.
// ODD: V is odd and the type bfloat16, so that every other row starts at an odd entry (RowLoads; an instance of its own, which spares
// the others 0.2 - 0.5 % of a call).
template <typename T, bool VEC, bool ODD>
__global__ void __launch_bounds__(kStatThreads)
k_row_stats(const T *__restrict__ target, const T *__restrict__ draft,
            const int32_t *__restrict__ tokens, int K, int L, int V, float c,
            RowStat *__restrict__ stats, int32_t *__restrict__ final_counter, long long n_rows, int batch,
            const int32_t *__restrict__ pend_count, int32_t *__restrict__ pend_off,
            PendRow *__restrict__ pend, int nlev, double c_rel)
{
    __shared__ double sh_d[kStatThreads / kWave];
    __shared__ float sh_ref[kStatThreads / kWave];
    const long long pair = blockIdx.x;            // (b*K + k)*L + r
    const bool is_draft = blockIdx.y == 1;
    if (pair >= n_rows) {                         // uniform: one of the offset blocks
        const int level = static_cast<int>(pair - n_rows);
        if (!is_draft)
            pend_offsets(pend_count + static_cast<size_t>(level) * batch, K, L, batch,
                         pend_off + static_cast<size_t>(level) * (batch + 1));
        return;
    }
    const int r = static_cast<int>(pair % L);
    const long long bk = pair / L;
    if (threadIdx.x == 0 && !is_draft) {
        if (pair % (static_cast<long long>(K) * L) == 0)
            final_counter[pair / (static_cast<long long>(K) * L)] = 0;  // arrival counter of the final-token kernel
    }
    // the level's entries of this row: empty beyond its count, else not there yet (k_pend_norm)
    if (!is_draft && static_cast<int>(threadIdx.x) < nlev) {
        const bool modified = r < pend_count[static_cast<size_t>(threadIdx.x) * batch + bk / K];
        unsigned long long *const w = reinterpret_cast<unsigned long long *>(pend + threadIdx.x * n_rows + pair);
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = modified ? ~0ull : 0ull;
    }
    const T *row = is_draft ? draft + (bk * L + r) * static_cast<long long>(V)
                            : target + (bk * (L + 1) + r) * static_cast<long long>(V);
    const int tok_raw = token_index_queued(tokens, pair);
    uint32_t tok_bits = 0;                        // the token's logit, asked for behind the row's first loads
    RunningSum acc;                               // the drafted token is left out (leave_out)
    if (VEC) {
        const int nvec = row_vectors<T>(V);
        auto sweep = [&](const auto &from) {
            for (int i = threadIdx.x; i < nvec; i += kAhead * kStatThreads) {
                decltype(from.load(0)) v[kAhead];
#pragma unroll
                for (int a = 0; a < kAhead; ++a) {        // (no branch around a load: past the end the last vector again)
                    const int at = i + a * kStatThreads;
                    v[a] = from.load(at < nvec ? at : nvec - 1);
                }
                const int tok = token_index_used(tok_raw, V);
                if (i == static_cast<int>(threadIdx.x)) tok_bits = Elem<T>::bits(row + tok);
#pragma unroll
                for (int a = 0; a < kAhead; ++a) {
                    const int at = i + a * kStatThreads;
                    if (at < nvec) {
                        float z[Elem<T>::kPerVec];
                        from.entries(v[a], at, z);
                        add_entries<T>(acc, z, at, tok, V, c);
                    }
                }
            }
        };
        // (rows of an odd vocabulary that start at an even entry as all others: 97.4 / 96.6 us a call at 41 x 7 drafts of 6, V = 32003;
        // the others' entries straight from what was loaded, without putting the vectors together before: 99.2 / 98.3, 40 x 8 of 8,
        // V = 32001 130.2 / 129.2, 100 x 4 of 6, V = 20001 93.0 / 92.2)
        const RowLoads<T, ODD> from(row, V, nvec, pair == 0);
        if (from.turn != 0) sweep(from);
        else sweep(RowLoads<T, false>(row, V, nvec, false));
    } else {
        for (int x = threadIdx.x; x < V; x += kStatThreads) {
            float z[1] = {Elem<T>::scalar(row + x)};
            leave_out(z, x == token_index_used(tok_raw, V), 0);
            acc.add(z, c);
        }
    }
    // The waves' sums relative to integral references meet behind one barrier, and the first thread adds them up: a workgroup holds its
    // place on the compute unit through all of this, with nothing of its row to load any more.  Us a call, with a maximum and a sum
    // over the workgroup (four barriers), library exponentials and the token's logit fetched here / as here: one level on 100 x 8
    // drafts of 8, V = 3000 float32 165.3 / 150.8, two on 128 x 4 of 8, V = 8000 bfloat16 159.3 / 151.3, three iterations of 128 x 8 of
    // 8, V = 8000 782 / 734, 8 x 4 of 8, V = 128256 294.4 / 292.1; 32 x 8 of 8, V = 24000 without levels 88.5 / 86.1, 41 x 7 of 6,
    // V = 32003 96.5 / 95.9; 40 x 8 of 8, V = 32000 the same.  The logarithm stays the library's,
    // the more exact one (off by 0.6e-16 for sums between 1/2 and 2, log2_series by 5.7e-16; that takes another 0.2 - 0.6 % off calls with levels).
    constexpr int kWaves = kStatThreads / kWave;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    const float wave_ref = integral_reference(wave_max(acc.m2), 1.0f);
    const double wave_Z = wave_sum(acc.Z > 0.0f ? static_cast<double>(acc.Z) * exp2_small(static_cast<double>(acc.m2) - static_cast<double>(wave_ref)) : 0.0);
    if (lane == 0) { sh_ref[wid] = wave_ref; sh_d[wid] = wave_Z; }
    __syncthreads();
    if (tid == 0) {
        float M = -3.0e38f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) M = fmaxf(M, sh_d[w] > 0.0 ? sh_ref[w] : -3.0e38f);
        double total = 0.0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) total += ldexp(sh_d[w], reference_shift(sh_ref[w], M));
        const float ztok = VEC ? Elem<T>::from_bits(tok_bits) : Elem<T>::scalar(row + token_index_used(tok_raw, V));
        const double tok2_raw = static_cast<double>(ztok) * static_cast<double>(c);
        const RefSum all = with_token(static_cast<double>(M), total, tok2_raw);
        const double lse2 = all.ref + log2(all.Z);
        const double tok2 = token_scaled(tok2_raw, lse2, c_rel);
        if (is_draft) { stats[pair].lse2_p = lse2; stats[pair].tok2_p = tok2; }
        else { stats[pair].lse2_q = lse2; stats[pair].tok2_q = tok2; }
    }
}

// ---- small batches: rows shared among workgroups
//
// With few rows a workgroup per row leaves most of the chip idle and every workgroup pays the latency of
// streaming a whole row alone (16 - 21 us per kernel at one prefix, whatever the bandwidth).  Each row (pair) is
// then cut into P parts: k_row_stats_parts leaves partial statistics with integral reference exponents,
// k_ot_sum_parts combines the ones each of its workgroups needs (and stores the RowStat entries) and leaves P
// partial sums per row, which the final-token kernel adds up in part order.  No workgroup waits for another one.

// grid (row pairs * P, 2): block (pair * P + part, 0 / 1) reduces part `part` of the target / draft row of the pair
template <typename T, bool VEC, bool ODD>
__global__ void __launch_bounds__(kStatThreads)
k_row_stats_parts(const T *__restrict__ target, const T *__restrict__ draft, const int32_t *__restrict__ tokens, int L,
                  int V, float c, int P, Row0Part *__restrict__ parts)
{
    __shared__ double sh_d[kStatThreads / kWave];
    __shared__ float sh_f[kStatThreads / kWave];
    const long long pair = blockIdx.x / P;        // (b*K + k)*L + r
    const int part = static_cast<int>(blockIdx.x % P);
    const int r = static_cast<int>(pair % L);
    const long long bk = pair / L;
    const bool is_draft = blockIdx.y == 1;
    const T *row = is_draft ? draft + (bk * L + r) * static_cast<long long>(V)
                            : target + (bk * (L + 1) + r) * static_cast<long long>(V);
    constexpr int PV = Elem<T>::kPerVec;
    const int units = VEC ? row_vectors<T>(V) : V;
    const int per = (units + P - 1) / P;
    const int lo = part * per, hi = lo + per < units ? lo + per : units;
    const RowLoads<T, ODD> from(row, V, hi, pair == 0);
    const int tok_raw = token_index_queued(tokens, pair);
    RunningSum acc;                               // the drafted token is left out (leave_out)
    if (VEC) {
        // two loads in flight per thread (of the last step too: the second one's place beyond the part is the part's last vector)
        for (int i = lo + static_cast<int>(threadIdx.x); i < hi; i += 2 * kStatThreads) {
            const int i2 = i + kStatThreads;
            const Loaded<ODD> a = from.load(i), b2 = from.load(i2 < hi ? i2 : hi - 1);
            const int tk = token_index_used(tok_raw, V);
            add_vector<T>(acc, from.vector(a, i), i, tk, V, c);
            if (i2 < hi) add_vector<T>(acc, from.vector(b2, i2), i2, tk, V, c);
        }
    } else {
        for (int x = lo + static_cast<int>(threadIdx.x); x < hi; x += kStatThreads) {
            float z[1] = {Elem<T>::scalar(row + x)};
            leave_out(z, x == token_index_used(tok_raw, V), 0);
            acc.add(z, c);
        }
    }
    const int tok = token_index_used(tok_raw, V);
    const int tok_unit = VEC ? tok / PV : tok;
    const float M = block_max(acc.m2, sh_f);
    const double mine = static_cast<double>(acc.Z) * exp2(static_cast<double>(acc.m2) - static_cast<double>(M));
    const double total = block_sum(acc.Z > 0.0f ? mine : 0.0, sh_d);
    if (threadIdx.x == 0) {
        // the part that holds the drafted token adds its weight here, in float64
        const bool mine_tok = tok_unit >= lo && tok_unit < hi;
        const double tok2_raw = mine_tok ? static_cast<double>(Elem<T>::scalar(row + tok)) * static_cast<double>(c)
                                         : -static_cast<double>(__builtin_inff());
        const RefSum all = with_token(static_cast<double>(M), total, tok2_raw);
        Row0Part out;
        out.ref = floor(all.ref);
        out.Z = all.Z * exp2(all.ref - out.ref);
        parts[(pair * 2 + (is_draft ? 1 : 0)) * kRowParts + part] = out;
    }
}

// log2 sum_x 2^(c z[x]) of a row from its parts' sums (combined in part order: the same bits wherever it is done)
__device__ __forceinline__ double lse2_from_parts(const Row0Part *pp, int P)
{
    double ref = -1.0e300;
    for (int q = 0; q < P; ++q)
        if (pp[q].Z > 0.0 && pp[q].ref > ref) ref = pp[q].ref;
    double Z = 0.0;
    for (int q = 0; q < P; ++q) {
        const double d = pp[q].ref - ref;                     // an integer <= 0
        if (pp[q].Z > 0.0 && d > -2000.0) Z += ldexp(pp[q].Z, static_cast<int>(d));
    }
    return ref + log2(Z);
}

// grid rows * P, rows = batch * K * (L - 1): block row * P + part sums part `part` of the Eq. (hik) terms of row
// pair i = 1 .. L-1 of a draft (PEND: against the row as the pending levels leave it, exactly as k_ot_sum does).
// With stat_P > 1 the statistics of the draft's rows 0 .. i are still in parts
// (k_row_stats_parts): every workgroup combines the ones it needs, and part 0 stores the RowStat entry of its
// row (the workgroup of row 1 also that of row 0, and clears the arrival counter of the final-token kernel).
template <typename T, bool VEC, bool PEND, bool ODD>
__device__ __forceinline__ void
ot_sum_parts(const T *__restrict__ target, const T *__restrict__ draft, const int32_t *__restrict__ tokens, int K, int L,
             int V, float c, int P, const Row0Part *__restrict__ stat_parts, int stat_P, RowStat *stats,
             int32_t *__restrict__ final_counter, double *__restrict__ s_part, double *__restrict__ e_part,
             const PendRow *__restrict__ pend, long long n_rows, int nlev, double c_rel)
{
    __shared__ double sh_d[kStatThreads / kWave];
    __shared__ PendTable sh_tab;                  // PEND: the levels that modify this row
    __shared__ PendRow sh_pr[kMaxPend];
    __shared__ double sh_sumN;
    __shared__ double sh_lse[2 * kMaxRows], sh_tok[2 * kMaxRows];
    const long long idx = blockIdx.x / P;         // bk*(L-1) + (i-1)
    const int part = static_cast<int>(blockIdx.x % P);
    const int i = static_cast<int>(idx % (L - 1)) + 1;
    const long long bk = idx / (L - 1);
    const long long pair = bk * L + i;
    const T *rq = target + (bk * (L + 1) + i) * static_cast<long long>(V);
    const T *rp = draft + pair * static_cast<long long>(V);
    const int units = VEC ? row_vectors<T>(V) : V;
    const int per = (units + P - 1) / P;
    const int lo = part * per, hi = lo + per < units ? lo + per : units;
    constexpr bool kAhead = VEC && (PEND || Elem<T>::kPerVec == 4);      // (see first_pairs)
    const RowLoads<T, ODD> from_q(rq, V, hi, false), from_p(rp, V, hi, false);         // (i >= 1: not a tensor's first row)
    const FirstPairs<ODD> first = first_pairs<T, kAhead, kStatThreads>(from_q, from_p, lo, hi);
    RowStat st;
    double log2nu = 0.0;
    if (stat_P > 1) {
        for (int t = threadIdx.x; t < 2 * (i + 1); t += kStatThreads) {
            const int j = t >> 1, m = t & 1;
            const long long pj = bk * L + j;
            sh_lse[t] = lse2_from_parts(stat_parts + (pj * 2 + m) * kRowParts, stat_P);
            int tok = tokens[pj];
            tok = tok < 0 ? 0 : (tok >= V ? V - 1 : tok);
            const T *row = m ? draft + pj * static_cast<long long>(V) : target + (bk * (L + 1) + j) * static_cast<long long>(V);
            sh_tok[t] = token_scaled(static_cast<double>(Elem<T>::scalar(row + tok)) * static_cast<double>(c), sh_lse[t], c_rel);
        }
        __syncthreads();
        st.lse2_q = sh_lse[2 * i]; st.lse2_p = sh_lse[2 * i + 1];
        st.tok2_q = sh_tok[2 * i]; st.tok2_p = sh_tok[2 * i + 1];
        for (int j = 0; j < i; ++j) log2nu += (sh_tok[2 * j] - sh_lse[2 * j]) - (sh_tok[2 * j + 1] - sh_lse[2 * j + 1]);
        if (part == 0 && threadIdx.x == 0) {
            stats[pair] = st;
            if (i == 1) {
                RowStat s0;
                s0.lse2_q = sh_lse[0]; s0.lse2_p = sh_lse[1]; s0.tok2_q = sh_tok[0]; s0.tok2_p = sh_tok[1];
                stats[bk * L] = s0;
                if (bk % K == 0) final_counter[bk / K] = 0;
            }
        }
    } else {
        st = stats[pair];
        if (!PEND)
            for (int j = 0; j < i; ++j) {
                const RowStat a = stats[bk * L + j];
                log2nu += (a.tok2_q - a.lse2_q) - (a.tok2_p - a.lse2_p);
            }
    }
    double sumN = 0.0;
    if (PEND) {                                   // as in k_ot_sum: the row as the pending levels leave it
        log2nu = pend_block_ratio(stats, pend, n_rows, nlev, bk * L, i, sh_d);
        if (static_cast<int>(threadIdx.x) < nlev) sh_pr[threadIdx.x] = pend[static_cast<long long>(threadIdx.x) * n_rows + pair];
        __syncthreads();
        if (threadIdx.x == 0) sh_sumN = pend_build_table(sh_pr, 1, nlev, 0, st.lse2_p - st.lse2_q, sh_tab);
        __syncthreads();
        sumN = sh_sumN;
    }
    const float shift_q = static_cast<float>(st.lse2_q);
    constexpr int N = VEC ? Elem<T>::kPerVec : 1;
    const RatioConst rc(ratio_const(st.lse2_p, st.lse2_q, log2nu, c_rel) - sumN);
    float acc = 0.0f;
    if (PEND && sh_tab.n > 0) {                   // uniform over the workgroup
        for_each_pair_from<T, VEC, kAhead, kStatThreads>(first, from_q, from_p, V, lo, hi, [&](int, const float (&zq)[N], const float (&zp)[N]) {
            float wq[N], w[N];
            pending_weights(zq, zp, c, shift_q, sh_tab, rc, K, wq, w);
#pragma unroll
            for (int j = 0; j < N; ++j) acc += w[j];
        });
    } else {
        for_each_pair_from<T, VEC, kAhead, kStatThreads>(first, from_q, from_p, V, lo, hi, [&](int, const float (&zq)[N], const float (&zp)[N]) {
            float wq[N], w[N];
            ot_weights(zq, zp, c, shift_q, rc, K, wq, w);
#pragma unroll
            for (int j = 0; j < N; ++j) acc += w[j];
        });
    }
    double total = block_sum(static_cast<double>(acc), sh_d);
    if (threadIdx.x == 0 && !(PEND && sh_tab.n > 0))
        total = with_token_term<T>(total, st, log2nu, rq, rp, tokens + pair, V, lo * N, hi * N < V ? hi * N : V, c, shift_q, rc, K);
    // (whether the row's s and g nearly cancel, so that Eq. (hik) needs nu^2 (s - g) summed term by term, only the sum
    // over all parts can tell: the final-token kernel looks at it)
    if (threadIdx.x == 0) s_part[pair * kPendParts + part] = total * exp2(static_cast<double>(shift_q) - st.lse2_q - sumN);
    // (the final-token kernel looks at the complete sums itself and takes E where a row needs it: its parts start as
    // "not there yet")
    if (part == 0 && threadIdx.x < kPendParts) e_part[pair * kPendParts + threadIdx.x] = -1.0;
}

template <typename T, bool VEC, bool PEND>
__global__ void __launch_bounds__(kStatThreads)
k_ot_sum_parts(const T *__restrict__ target, const T *__restrict__ draft, const int32_t *__restrict__ tokens, int K, int L,
               int V, float c, int P, const Row0Part *__restrict__ stat_parts, int stat_P, RowStat *stats,
               int32_t *__restrict__ final_counter, double *__restrict__ s_part, double *__restrict__ e_part,
               const PendRow *__restrict__ pend, long long n_rows, int nlev, double c_rel)
{
    ot_sum_parts<T, VEC, PEND, false>(target, draft, tokens, K, L, V, c, P, stat_parts, stat_P, stats, final_counter, s_part, e_part, pend, n_rows, nlev, c_rel);
}
// bfloat16 rows of an odd vocabulary, by vectors
template <bool PEND>
__global__ void __launch_bounds__(kStatThreads)
k_ot_sum_parts_odd(const uint16_t *__restrict__ target, const uint16_t *__restrict__ draft, const int32_t *__restrict__ tokens, int K, int L,
                   int V, float c, int P, const Row0Part *__restrict__ stat_parts, int stat_P, RowStat *stats,
                   int32_t *__restrict__ final_counter, double *__restrict__ s_part, double *__restrict__ e_part,
                   const PendRow *__restrict__ pend, long long n_rows, int nlev, double c_rel)
{
    ot_sum_parts<uint16_t, true, PEND, true>(target, draft, tokens, K, L, V, c, P, stat_parts, stat_P, stats, final_counter, s_part, e_part, pend, n_rows, nlev, c_rel);
}

// The sum of a vector's terms, in pairs.  A thread adds it to what it has: term after term, a part of half as many workgroups would
// carry up to twice the error (rms over rows of 131072 bfloat16 entries of deviation 3, four workgroups per row 1.0e-8, eight
// 4.2e-9; four with the vector's terms added up first 2.1e-9).
template <int N>
__device__ __forceinline__ float vector_sum(const float (&w)[N])
{
    static_assert(N == 1 || N == 4 || N == 8, "entries of a vector");
    if constexpr (N == 1) return w[0];
    else {
        float a = (w[0] + w[2]) + (w[1] + w[3]);
        if constexpr (N == 8) a += (w[4] + w[6]) + (w[5] + w[7]);
        return a;
    }
}

// The levels [from, to) of pending modification (those before them are done).  A level's T rows are enumerated prefix by prefix (off[b]
// rows before prefix b; within a prefix row index slowest) and each is shared among P workgroups (level_parts), so that a level with
// few rows left still occupies the chip (one workgroup streaming a whole row pair with several levels of arithmetic per entry takes
// 100 - 200 us).  The levels' T P units stand in one line, level after level; a workgroup does the unit of its own number,
// and those behind the last unit leave at once.  A row's parts meet in the workspace (device-scope relaxed atomic accesses): the
// workgroup that arrives last at the entry's counter leaves the entry.  Sums and counters are a level's own, so that it does
// not matter in which order units of different levels come to them.
//
// A unit needs the entries of the levels below its own for its row and for the rows of its draft in front of it.  k_row_stats has marked
// the entries of modified rows as not there yet (all four words), so a unit looks for them until they are there.  They come from units of
// lower numbers, that is of workgroups of lower index, and workgroups are dispatched in index order, so
// what is waited for is running or has run.  Nothing relies on it: after `looks` looks a workgroup makes the entries that are still
// not there itself, one after the other (it looks again in front of each part), with the parts and in the order that their units
// have (the same bits).  That is many times their units' work, so the looks have to outlast whatever they can be waiting for
// (level_looks); 1024 of them did not: sixteen levels on all rows of 1 x 4 drafts of 17, V = 1000000 bfloat16 took 338 ms a call and
// take 2.7 now, 4 x 4 drafts of 17 651 and 21, seven levels on 8 x 8 of 8, V = 256000 float32 9.6 and 2.5.
//
// What bounds a level: where its rows fill the chip, arithmetic; else latencies (load, sum, hand-over: 8 - 15 us) and, before, launches: a
// kernel for every level, 3 us each, of which a call that updates its state in place makes L - 1, most of them of levels in which nothing is
// alive, and each of those had a workgroup per row to find that out.  Us a call, a launch per level / as here: three iterations of
// Algorithm 3, 8 x 4 drafts of 8, V = 128256 bfloat16 344 / 313; one prompt of 3 drafts 195 / 158; 3 x 3 of 8, V = 50257 float32 203 / 167;
// one iteration once two to six levels are alive on average, 24 x 8 of 8, V = 128256 584 / 531, the same drafts over and over 760 / 673;
// 8 x 4 of 16, V = 32000 372 / 330; 10 x 8 of 12, V = 3000 float32 209 / 157; three given levels on 16 x 4 of 8, V = 32000 110.7 / 101.8.
// The float64 constants are made by one wave, a level per lane, with the exponential's coefficients in LDS: as library calls of every
// thread they took 142 registers, or 224 bytes of scratch at 80 (three workgroups per compute unit), which cost more than
// the launches.
constexpr unsigned long long kNotThere = ~0ull;        // (a NaN that no sum produces; see entry_store)
constexpr unsigned long long kNoLevel = 0x8000000000000000ull;     // log2 N = -0.0: the level leaves the row as it is

__device__ __forceinline__ void entry_store(PendRow *pr, double log2mu, double log2N, double tokadj, bool some)
{
    unsigned long long *const w = reinterpret_cast<unsigned long long *>(pr);
    static_assert(sizeof(PendRow) == 32, "four words");
    if (log2mu != log2mu) log2mu = __builtin_nan("");    // (a carried ratio may be any NaN, also the one that says not there)
    __hip_atomic_store(w, static_cast<unsigned long long>(__double_as_longlong(log2mu)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(w + 1, static_cast<unsigned long long>(__double_as_longlong(log2N)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(w + 2, static_cast<unsigned long long>(__double_as_longlong(tokadj)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(w + 3, some ? 1ull : 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long entry_load(const PendRow *pr, int word)
{
    return __hip_atomic_load(reinterpret_cast<const unsigned long long *>(pr) + word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct LevelArgs {
    const double *carry;           // [nlev][batch]
    const int32_t *count;          // [nlev][batch]
    const int32_t *off;            // [nlev][batch + 1] rows a level modifies in the prefixes before
    const RowStat *stats;
    PendRow *pend;                 // [nlev][n_rows]
    double *sums;                  // [slots]: a unit's, by its place in the line
    long long n_rows;
    int K, L, V, batch;
    int looks;                     // at an entry that is not there yet, before a workgroup makes it itself
    int slots;                     // >= kPendParts * n_rows
    int from, to, most;            // the levels of this launch; parts of a row at most
    int first_grid, grid;          // workgroups that share a level's rows: the first level's, any other's
    int resident;                  // of a grid that is larger than the number of row pairs
    float c;
};

// Workgroups that share a row of a level of T rows (three or more of them only as far as all are resident at once: a second
// round costs more than larger parts; the first level's grid is no larger than that).
__device__ __forceinline__ int level_parts(const LevelArgs &ar, int level, int T)
{
    if (T <= 0) return 0;
    int P = (level == 0 ? ar.first_grid : ar.grid) / T;          // >= 1: the modified rows are among the grid's rows
    if (level > 0 && T * P > ar.resident && T * 3 <= ar.resident) P = ar.resident / T;
    return P > ar.most ? ar.most : P;
}

// What the levels do to the rows of a draft, and the constants of one sweep (LDS).
struct Levels {
    PendTable tab;                         // the levels in front that modify the row at hand
    double N[kMaxPend * kMaxRows], adj[kMaxPend * kMaxRows], mu[kMaxPend * kMaxRows];       // [level][row]
    double run;                            // log2 q^(l)[token] - log2 p[token] of the row at hand
    double scale;                          // log2 of what the sum is relative to, under the levels in front
    double sums[kPendParts];
    float shift_q, C2_hi, neg_kappa;
    int cnt[kMaxPend];                     // rows the levels modify
    // (what only a unit that makes entries needs: kept here for want of scalar registers)
    const PendRow *entries;                // of the draft
    long long n_rows;
    int looks;
    double exp2_coef[11];                  // (see exp2_from)
};

// exp2_small with its polynomial's coefficients in LDS: hoisted out of a loop, they would take registers that the sweeps need.
__device__ __forceinline__ double exp2_from(const double *coef, double x)
{
    const double n = rint(x), f = (x - n) * 0.693147180559945309417;
    double p = coef[0];
#pragma unroll
    for (int i = 1; i < 11; ++i) p = fma(p, f, coef[i]);
    p = fma(p, f, 1.0);
    p = fma(p, f, 1.0);
    return x > 1000.0 ? INFINITY : (x > -1000.0 ? ldexp(p, static_cast<int>(fmin(fmax(n, -1001.0), 1001.0))) : 0.0);
}
__device__ const double g_exp2_coef[11] = {1.0 / 479001600.0, 1.0 / 39916800.0, 1.0 / 3628800.0, 1.0 / 362880.0, 1.0 / 40320.0, 1.0 / 5040.0,
                                           1.0 / 720.0, 1.0 / 120.0, 1.0 / 24.0, 1.0 / 6.0, 0.5};
// log2_series with it.
__device__ __forceinline__ double log2_from(const double *coef, double z)
{
    int e;
    const double m = frexp(z, &e);
    const double y0 = static_cast<double>(__log2f(static_cast<float>(m)));
    const double d = m * exp2_from(coef, -y0) - 1.0;
    return static_cast<double>(e) + fma(d * 1.44269504088896340736, fma(d, -0.5, 1.0), y0);
}

// ONE: level 0 alone, which has none below it.
template <typename T, bool VEC, bool ONE>
__global__ void __launch_bounds__(kStatThreads, VEC ? 6 : 8)
k_pend_norm(const T *__restrict__ target, const T *__restrict__ draft, LevelArgs ar)
{
    __shared__ double sh_d[kStatThreads / kWave];
    __shared__ Levels sh;
    __shared__ int sh_b, sh_last;
    const int K = ar.K, L = ar.L, V = ar.V, batch = ar.batch;
    const float c = ar.c;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    int level = 0, P, at = static_cast<int>(blockIdx.x), P_l = 0;
    if constexpr (ONE) {
        const int T_0 = ar.off[batch];
        P = level_parts(ar, 0, T_0);
        if (at >= T_0 * P) return;                // uniform over the workgroup
    } else {
        // where each level's units end: a lane looks after a level, in every wave
        const int T_l = lane >= ar.from && lane < ar.to ? ar.off[lane * (batch + 1) + batch] : 0;
        if (!__ballot(T_l > 0)) return;           // uniform over the workgroup
        P_l = level_parts(ar, lane, T_l);
        int end = static_cast<int>(wave_inclusive_sum(static_cast<double>(T_l) * static_cast<double>(P_l)));
        if (__builtin_amdgcn_readlane(end, kWave - 1) > ar.slots) {       // uniform (many given levels on a few short drafts)
            const int most = ar.slots / static_cast<int>(wave_sum(static_cast<double>(T_l)));
            P_l = P_l < most ? P_l : most;
            end = static_cast<int>(wave_inclusive_sum(static_cast<double>(T_l) * static_cast<double>(P_l)));
        }
        const unsigned long long behind = __ballot(at < end);
        if (!behind) return;                      // uniform
        level = __ffsll(static_cast<long long>(behind)) - 1;
        P = __builtin_amdgcn_readlane(P_l, level);
        at -= __builtin_amdgcn_readlane(end, level) - __builtin_amdgcn_readlane(T_l, level) * P;
    }
    auto parts_of = [&](int l_) { return __builtin_amdgcn_readlane(P_l, l_); };
    if (tid < 11) sh.exp2_coef[tid] = g_exp2_coef[tid];
    const int item = at / P, part = at - item * P;
    const int32_t *const off = ar.off + level * (batch + 1);
    for (int base = 0; base < batch; base += kStatThreads) {
        const int bb = base + tid;
        if (bb < batch && off[bb] <= item && item < off[bb + 1]) sh_b = bb;          // exactly one thread
    }
    __syncthreads();
    const int b = __builtin_amdgcn_readfirstlane(sh_b);
    const int j = item - off[b], r = j / K;
    const long long bk = static_cast<long long>(b) * K + (j - r * K), pair = bk * L + r;
    const int n_units = VEC ? row_vectors<T>(V) : V;
    struct In { RowStat st; double carry; };
    auto loads = [&](int l_, int row_) {
        In in;
        in.st = ar.stats[bk * L + (lane < row_ ? lane : row_)];
        in.carry = ar.carry[static_cast<size_t>(l_) * batch + b];
        return in;
    };
    // one look at a level's entry of row tr: whether it is there, and if so what it says
    auto look = [&](const PendRow *pr, int tl, int tr) {
        const unsigned long long mu = entry_load(pr, 0), n = entry_load(pr, 1), a = entry_load(pr, 2), f = entry_load(pr, 3);
        if (mu == kNotThere || n == kNotThere || a == kNotThere || static_cast<unsigned>(f) == ~0u) return false;     // (f: flag and counter)
        const int to = tl * kMaxRows + tr;
        sh.mu[to] = __longlong_as_double(static_cast<long long>(mu));
        sh.N[to] = __longlong_as_double(static_cast<long long>(f != 0ull ? n : kNoLevel));
        sh.adj[to] = __longlong_as_double(static_cast<long long>(a));
        return true;
    };
    In in{};
    if constexpr (VEC) in = loads(level, r);      // (beside the entries; rows read entry by entry have no registers to spare)
    // What is summed: this unit's part, once; if an entry that it builds on does not appear, all parts of those entries first.
    int l = level, row = r, q = part, parts = P;
    bool alone = false;
    if constexpr (!ONE) {
        bool none = false;
        for (int t = tid; t < level * (r + 1); t += kStatThreads) {
            const int tl = t / (r + 1), tr = t - tl * (r + 1);
            bool there = tl < ar.from;            // (a level of an earlier launch)
            if (there) {
                const PendRow e = ar.pend[tl * ar.n_rows + bk * L + tr];
                sh.mu[tl * kMaxRows + tr] = e.log2mu; sh.adj[tl * kMaxRows + tr] = e.tokadj;
                sh.N[tl * kMaxRows + tr] = e.flag != 0 ? e.log2N : -0.0;
            }
            for (int n = 0; n < ar.looks && !there; ++n) {
                there = look(ar.pend + tl * ar.n_rows + bk * L + tr, tl, tr);
                if (!there) __builtin_amdgcn_s_sleep(2);
            }
            none = none || !there;
        }
        alone = __syncthreads_or(none) != 0;
        if (alone) {                              // (normally none is missing)
            if (tid == 0) { sh.entries = ar.pend + bk * L; sh.n_rows = ar.n_rows; sh.looks = ar.looks; }
            if (tid < level) {
                const int cnt = ar.count[static_cast<size_t>(tid) * batch + b];
                sh.cnt[tid] = cnt < 0 ? 0 : (cnt > L ? L : cnt);
            }
            __syncthreads();
            l = ar.from; row = 0; q = 0;          // (an earlier launch's are there)
            parts = parts_of(l);
        }
    }
    for (;;) {                                    // (uniform, as everything here; normally one pass)
        const bool own = ONE || (l == level && row == r);
        bool there = false;
        if constexpr (!ONE) {
            if (!own) {                           // it may have come meanwhile
                if (tid == 0) sh_last = sh.looks > 0 && look(sh.entries + l * sh.n_rows + row, l, row);
                __syncthreads();
                there = sh_last != 0;
            }
        }
        if (there) {
            // (sh has it)
        } else if (own || row < sh.cnt[l]) {
            if (tid < kWave) {
                // block ratio in front of the row: the carried one continued along the drafted tokens with the distribution this level
                // modifies (the target rows as modified by the levels below)
                if (alone || !VEC) in = loads(l, row);
                double run = (in.st.tok2_q - in.st.lse2_q) - (in.st.tok2_p - in.st.lse2_p);
                if constexpr (!ONE)
                    if (lane <= row)
                        for (int m = 0; m < l; ++m) run += sh.adj[m * kMaxRows + lane] - sh.N[m * kMaxRows + lane];
                RowStat st;
                st.lse2_q = lane_value(in.st.lse2_q, row); st.lse2_p = lane_value(in.st.lse2_p, row);
                const double log2mu = in.carry * 1.44269504088896340736 + wave_sum(lane < row ? run : 0.0);
                if (lane == row) sh.run = run;
                // the levels in front, a lane each; lane l: this level's ratio
                const double base = st.lse2_p - st.lse2_q;
                bool on = false;
                double upto = 0.0, n_l = 0.0;
                if constexpr (!ONE) {
                    on = lane < l && static_cast<unsigned long long>(__double_as_longlong(sh.N[(lane < l ? lane : 0) * kMaxRows + row])) != kNoLevel;
                    n_l = on ? sh.N[lane * kMaxRows + row] : 0.0;
                    upto = wave_inclusive_sum(n_l);
                }
                const unsigned long long ons = __ballot(on);
                const double sumN = ONE ? 0.0 : lane_value(upto, kWave - 1);
                const double C = on ? base + sh.mu[lane * kMaxRows + row] - (upto - n_l) : base + log2mu - sumN;
                const float C_hi = static_cast<float>(C);                 // (as RatioConst)
                const double kappa = exp2_from(sh.exp2_coef, static_cast<double>(C_hi) - C);
                const float nk = (kappa > 0.5 && kappa < 2.0) ? -static_cast<float>(kappa) : -1.0f;
                if (on) {
                    const int to = __popcll(ons & ((1ull << lane) - 1ull));
                    sh.tab.C_hi[to] = C_hi;
                    sh.tab.neg_kappa[to] = nk;
                }
                if (lane == l) {
                    sh.mu[l * kMaxRows + row] = log2mu;
                    sh.tab.n = __popcll(ons);
                    sh.shift_q = static_cast<float>(st.lse2_q); sh.C2_hi = C_hi; sh.neg_kappa = nk;
                    sh.scale = static_cast<double>(static_cast<float>(st.lse2_q)) - st.lse2_q - sumN;
                }
            }
            __syncthreads();
            const T *rq = target + (bk * (L + 1) + row) * static_cast<long long>(V);
            const T *rp = draft + (bk * L + row) * static_cast<long long>(V);
            const int per = (n_units + parts - 1) / parts, lo = q * per, hi = lo + per < n_units ? lo + per : n_units;
            const RowLoads<T, false> from_q(rq, V, hi, false), from_p(rp, V, hi, false);
            const float shift_q = sh.shift_q;
            const RatioConst rc(sh.C2_hi, sh.neg_kappa);
            constexpr int N = VEC ? Elem<T>::kPerVec : 1;
            float acc = 0.0f;
            if (ONE || sh.tab.n == 0) {
                for_each_pair_from<T, VEC, false, kStatThreads>(FirstPairs<false>(), from_q, from_p, V, lo, hi, [&](int, const float (&zq)[N], const float (&zp)[N]) {
                    float wq[N], w[N];
                    ot_weights(zq, zp, c, shift_q, rc, K, wq, w);
                    acc += vector_sum(w);
                });
            } else {
                for_each_pair_from<T, VEC, false, kStatThreads>(FirstPairs<false>(), from_q, from_p, V, lo, hi, [&](int, const float (&zq)[N], const float (&zp)[N]) {
                    float wq[N], w[N];
                    pending_weights(zq, zp, c, shift_q, sh.tab, rc, K, wq, w);
                    acc += vector_sum(w);
                });
            }
            double S = block_sum(static_cast<double>(acc), sh_d);         // relative to 2^shift_q
            if (own && parts > 1) {
                // the store is a device-scope access; the wait lasts until it has been performed, so the counter update that
                // follows (same thread) cannot be seen before it
                unsigned long long *const sums = reinterpret_cast<unsigned long long *>(ar.sums + (blockIdx.x - part));
                if (tid == 0) {
                    __hip_atomic_store(sums + part, static_cast<unsigned long long>(__double_as_longlong(S)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    wait_for_stores();
                    // (the counter lies beside the entry's flag, which is not there yet, and starts from -1 as that does)
                    const int arrived = __hip_atomic_fetch_add(&ar.pend[level * ar.n_rows + pair].pad, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    sh_last = arrived == parts - 2;
                }
                __syncthreads();
                if (!sh_last) break;
                if (tid < parts)
                    sh.sums[tid] = __longlong_as_double(static_cast<long long>(__hip_atomic_load(sums + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)));
            } else if (tid == 0) {
                sh.sums[q] = S;
            }
            __syncthreads();
            if (tid == 0 && (own || q == parts - 1)) {
                S = 0.0;
                for (int x = 0; x < parts; ++x) S += sh.sums[x];          // in part order: the same bits whoever does it
                const double W = S * exp2_from(sh.exp2_coef, sh.scale), log2mu = sh.mu[l * kMaxRows + row];     // mass of q^(l) t^K
                const bool some = W > 0.0;        // otherwise every weight is zero and the row stays q^(l)
                double log2N = 0.0, tokadj = 0.0;
                if (some) {
                    log2N = log2_from(sh.exp2_coef, W);
                    const double x = -sh.run - log2mu, t = 1.0 - exp2_from(sh.exp2_coef, x);     // 1 - p[token] / (mu q^(l)[token])
                    tokadj = x == x && t > 0.0 ? static_cast<double>(K) * log2_from(sh.exp2_coef, t) : -INFINITY;
                }
                if (own) {
                    entry_store(ar.pend + l * ar.n_rows + pair, log2mu, log2N, tokadj, some);
                    wait_for_stores();
                }
                sh.N[l * kMaxRows + row] = some ? log2N : -0.0;
                sh.adj[l * kMaxRows + row] = tokadj;
            }
        } else if (tid == 0) {
            sh.N[l * kMaxRows + row] = -0.0; sh.adj[l * kMaxRows + row] = 0.0;
        }
        if (own) break;
        __syncthreads();
        if (!there && row < sh.cnt[l] && q + 1 < parts) ++q;
        else {
            q = 0;
            if (++row > r) {
                row = 0; ++l;
                if (l == level) { row = r; q = part; }
                parts = parts_of(l);
            }
        }
    }
}

template <typename T, bool VEC, bool PEND, bool ODD>
__global__ void __launch_bounds__(kStatThreads)
k_ot_sum(const T *__restrict__ target, const T *__restrict__ draft, const int32_t *__restrict__ tokens, int K, int L, int V,
         float c, const RowStat *__restrict__ stats, const PendRow *__restrict__ pend, long long n_rows, int nlev,
         double *__restrict__ s_out, double *__restrict__ e_out, double *__restrict__ e_part, double c_rel)
{
    __shared__ double sh_d[kStatThreads / kWave];
    __shared__ PendTable sh_tab;
    __shared__ PendRow sh_pr[kMaxPend];           // the levels, at this row
    __shared__ double sh_sumN;
    const long long idx = blockIdx.x;             // bk*(L-1) + (i-1)
    const int i = static_cast<int>(idx % (L - 1)) + 1;
    const long long bk = idx / (L - 1);
    const T *rq = target + (bk * (L + 1) + i) * static_cast<long long>(V);
    const T *rp = draft + (bk * L + i) * static_cast<long long>(V);
    const int units = VEC ? row_vectors<T>(V) : V;
    constexpr bool kAhead = VEC && !PEND;         // (see first_pairs)
    const RowLoads<T, ODD> from_q(rq, V, units, false), from_p(rp, V, units, false);   // (i >= 1: not a tensor's first row)
    const FirstPairs<ODD> first = first_pairs<T, kAhead, kStatThreads>(from_q, from_p, 0, units);
    const RowStat st = stats[bk * L + i];
    // block likelihood ratio of the length-i block, from the rows before row i (their token
    // probabilities under the modified rows where levels are pending)
    double log2nu = 0.0, sumN = 0.0;
    if (PEND) {
        log2nu = pend_block_ratio(stats, pend, n_rows, nlev, bk * L, i, sh_d);
        if (static_cast<int>(threadIdx.x) < nlev) sh_pr[threadIdx.x] = pend[static_cast<long long>(threadIdx.x) * n_rows + bk * L + i];
        __syncthreads();
        if (threadIdx.x == 0) sh_sumN = pend_build_table(sh_pr, 1, nlev, 0, st.lse2_p - st.lse2_q, sh_tab);
        __syncthreads();
        sumN = sh_sumN;
    } else {
        for (int j = 0; j < i; ++j) {
            const RowStat a = stats[bk * L + j];
            log2nu += (a.tok2_q - a.lse2_q) - (a.tok2_p - a.lse2_p);
        }
    }
    const float shift_q = static_cast<float>(st.lse2_q);
    constexpr int N = VEC ? Elem<T>::kPerVec : 1;
    const RatioConst rc(ratio_const(st.lse2_p, st.lse2_q, log2nu, c_rel) - sumN);
    float acc = 0.0f;
    if (PEND && sh_tab.n > 0) {                   // uniform over the workgroup
        for_each_pair_from<T, VEC, kAhead, kStatThreads>(first, from_q, from_p, V, 0, units, [&](int, const float (&zq)[N], const float (&zp)[N]) {
            float wq[N], w[N];
            pending_weights(zq, zp, c, shift_q, sh_tab, rc, K, wq, w);
#pragma unroll
            for (int j = 0; j < N; ++j) acc += w[j];
        });
    } else {
        for_each_pair_from<T, VEC, kAhead, kStatThreads>(first, from_q, from_p, V, 0, units, [&](int, const float (&zq)[N], const float (&zp)[N]) {
            float wq[N], w[N];
            ot_weights(zq, zp, c, shift_q, rc, K, wq, w);
#pragma unroll
            for (int j = 0; j < N; ++j) acc += w[j];
        });
    }
    double total = block_sum(static_cast<double>(acc), sh_d);
    if (threadIdx.x == 0 && !(PEND && sh_tab.n > 0))
        total = with_token_term<T>(total, st, log2nu, rq, rp, tokens + (bk * L + i), V, 0, V, c, shift_q, rc, K);
    const double s_val = total * exp2(static_cast<double>(shift_q) - st.lse2_q - sumN);
    // where s and g = (1 - 1/nu)^K nearly cancel, Eq. (hik) needs nu^2 (s - g) summed term by term (rare: peaked
    // rows, large block ratios): the final-token kernel finds those rows and its workgroups sum E together (the
    // parts start as "not there yet")
    const double e_val = -1.0;
    if (threadIdx.x < kPendParts) e_part[(bk * L + i) * kPendParts + threadIdx.x] = -1.0;
    if (threadIdx.x == 0) { s_out[bk * L + i] = s_val; e_out[bk * L + i] = e_val; }
}

// Parts a row is cut into so that about four workgroups per compute unit are launched (1: one workgroup per row).
int row_parts(long long workgroups_per_row_unit, int V)
{
    if (V < 8192 || workgroups_per_row_unit < 1) return 1;         // short rows: nothing to share
    const long long want = 4LL * compute_units() / workgroups_per_row_unit;
    // below four parts the partial sums' extra steps cost what the sharing gains (measured)
    return static_cast<int>(want < 4 ? 1 : (want > kRowParts ? kRowParts : want));
}

// Looks that a unit of the levels takes at an entry, about a microsecond each: as many as elsewhere, and as many again for every
// sixteen steps (of a workgroup over a row's `units`) of all levels.  A unit waits for the units of the levels below it, one
// after the other, each at most a whole row long; a step under sixteen levels takes 8 us at most with three workgroups on a compute
// unit, and here has 64.
int level_looks(int units, int levels)
{
    const long long n = static_cast<long long>(wait_polls()) * (1 + static_cast<long long>(levels) * (units / kStatThreads) / 16);
    return static_cast<int>(n < 1 << 30 ? n : 1 << 30);
}

template <typename T>
hipError_t launch_typed(const Problem &p)
{
    const T *target = static_cast<const T *>(p.target);
    const T *draft = static_cast<const T *>(p.draft);
    RowStat *stats = reinterpret_cast<RowStat *>(p.ws + p.lay.stats);
    double *s = reinterpret_cast<double *>(p.ws + p.lay.s);
    int32_t *counter = reinterpret_cast<int32_t *>(p.ws + p.lay.counter);
    const long long pairs = static_cast<long long>(p.batch) * p.K * p.L;
    const bool vec = read_by_vectors<T>(p.V);
    constexpr bool kMayBeOdd = sizeof(T) == 2;
    const bool odd = kMayBeOdd && vec && p.V % 2 != 0;
    int32_t *pend_off = reinterpret_cast<int32_t *>(p.ws + p.lay.pend_off);
    double *pend_part = reinterpret_cast<double *>(p.ws + p.lay.pend_part);
    PendRow *pend = reinterpret_cast<PendRow *>(p.ws + p.lay.pend);
    // rows shared among workgroups (small batches); the sums' kernel then finishes the statistics, so L >= 2
    const int stat_parts = (p.pend_levels > 0 || p.s_parts < 2) ? 1 : row_parts(2 * pairs, p.V);
    Row0Part *stat_part = reinterpret_cast<Row0Part *>(p.ws + p.lay.stat_part);
    if (stat_parts > 1) {
        const dim3 gs(static_cast<unsigned>(pairs * stat_parts), 2);
#define SPECGBV_STATP_LAUNCH(VEC, ODD)                                                                              \
    hipLaunchKernelGGL((k_row_stats_parts<T, VEC, ODD>), gs, dim3(kStatThreads), 0, p.stream, target, draft, p.tokens, p.L, p.V, \
                       p.c, stat_parts, stat_part)
        if (odd) SPECGBV_STATP_LAUNCH(true, kMayBeOdd);
        else if (vec) SPECGBV_STATP_LAUNCH(true, false);
        else SPECGBV_STATP_LAUNCH(false, false);
#undef SPECGBV_STATP_LAUNCH
    } else {
        const dim3 g1(static_cast<unsigned>(pairs + p.pend_levels), 2);
#define SPECGBV_STATS_LAUNCH(VEC, ODD)                                                                              \
    hipLaunchKernelGGL((k_row_stats<T, VEC, ODD>), g1, dim3(kStatThreads), 0, p.stream, target, draft, p.tokens, p.K, p.L, p.V, \
                       p.c, stats, counter, pairs, p.batch, p.pend_count, pend_off, pend, p.pend_levels, p.c_rel)
        if (odd) SPECGBV_STATS_LAUNCH(true, kMayBeOdd);
        else if (vec) SPECGBV_STATS_LAUNCH(true, false);
        else SPECGBV_STATS_LAUNCH(false, false);
#undef SPECGBV_STATS_LAUNCH
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (p.pend_levels > 0) {
        // One workgroup per row pair, but at least two per compute unit, so that a small batch's rows can be shared (one, two, four per
        // unit, us a call: three iterations of Algorithm 3 with 8 x 4 drafts of 8, V = 128256 352, 339, 356, of which a launch whose
        // level is empty took 2.4 at four; 16 x 4 of 8, V = 32000 84.9, 85.0, 89.8; one prompt of 3 drafts 63.8, 64.1, 64.1).
        // With two per unit a level of more than half as many rows has a workgroup for each row alone, on half the places of the chip;
        // where that takes long (long rows, and the levels below them to be applied to every entry) the grid is large enough for
        // two, and has three per unit: 16 x 4 of 8, V = 128256 bfloat16 under three levels two / three / four per unit / as here
        // 271 / 259 / 254 / 246, 9 x 8 of 8, V = 129472 304 / 277 / 282 / 276, 14 x 5 of 8, V = 100000 245 / 233 / 229 / 222, 30 x 2 of
        // 8, V = 128256 under two 207 / 194 / 199 / 193.  Not the first level, although four workgroups of its instance are resident on a
        // unit (16 x 4 of 8 148.4 / 149.3 / 149.6, 16 x 4 of 6, V = 70000 float32 120.7 / 122.9 / 121.5), not where the levels are
        // the library's own, most of which are empty (two iterations, 16 x 4 of 8, V = 64000 204 / 205 / 212), not of shorter rows (20 x 4
        // of 8, V = 8000 float32 under two levels 61.7 / 62.0 / 67.2), and in float32, whose sweeps are shorter, only where two per
        // unit are not enough for two workgroups a row (10 x 8 of 4, V = 70000 127 / 130 / 135, 9 x 8 of 8, V = 64000 234 / 223 / 230).
        const long long cu = compute_units();
        LevelArgs la;
        la.carry = p.pend_carry; la.count = p.pend_count; la.off = pend_off;
        la.stats = stats; la.pend = pend;
        la.n_rows = pairs; la.K = p.K; la.L = p.L; la.V = p.V; la.batch = p.batch; la.c = p.c;
        la.looks = level_looks(vec ? row_vectors<T>(p.V) : p.V, p.pend_levels);
        const long long least = pairs > 2 * cu ? pairs : 2 * cu;
        long long grid = least;
        if (!p.state_count && row_vectors<T>(p.V) >= 6000 && 2 * pairs > (Elem<T>::kPerVec == 8 ? cu : 3 * cu) && 2 * pairs < 7 * cu)
            grid = 2 * pairs <= 3 * cu ? 3 * cu : 7 * cu / 2;
        // (three per unit are resident at once; not with every grid that a row pair each asks for)
        la.first_grid = static_cast<int>(least); la.grid = static_cast<int>(grid);
        la.resident = grid > pairs ? static_cast<int>(3 * cu) : 0x7fffffff;
        // The parts' sums stand where this call keeps nothing else: 64 a row pair, or, where that is not enough for sixteen parts at every
        // level of a few drafts, in the chain schedule's lists.
        const size_t here = p.lay.row0 - p.lay.stat_part, there = p.lay.kseq_pos - p.lay.later, room = here > there ? here : there;
        la.sums = here > there ? reinterpret_cast<double *>(stat_part) : reinterpret_cast<double *>(p.ws + p.lay.later);
        la.slots = static_cast<int>(room / sizeof(double) < 0x7fffffff ? room / sizeof(double) : 0x7fffffff);
        // Levels per launch.  Up to six rows per compute unit: all of the library's own (L - 1, most of them empty; an iteration once the
        // state has settled, each level its own launch / together: 30 x 6 drafts of 8, V = 16000 240 / 215 us, 48 x 4 of 8, V = 8000 177 / 155,
        // 24 x 8 of 8, V = 32000 float32 298 / 271, 1 x 4 of 8, V = 128256 62 / 56), and all that are given unless rows are long (two levels
        // on 16 x 4 drafts of 8, V = 8000 bfloat16 50.5 / 49.6, 32 x 4 of 8, V = 32000 118.1 / 117.0; but 32 x 3 of 8, V = 128256 265 / 273,
        // 16 x 4 of 6, V = 70000 float32 153.5 / 156.2: workgroups that wait hold places that a level's later parts could use).  With more
        // rows each level's fill the chip, and levels are launched one by one (two given levels on 64 x 4 of 8, V = 8000 100.3 / 102.4,
        // 128 x 16 542 / 596; three iterations with 128 x 8 of 8, V = 8000 875 / 916.  All but the first in one grid whose workgroups take
        // as many units as there are: 789 there, but 269 against 207 for a settled state of 64 x 4 of 8, V = 8000 and 2667 against
        // 952 for 32 x 8 of 8, V = 128256: the units of a level stand in a few workgroups, for which all the others wait).
        // Parts of a row: sixteen at most, and of levels that are launched together more than eight only where every thread of each part
        // has two vectors of it, and more than four only where a row has two for every thread of one workgroup: each unit holds a place
        // while it waits, and short ones take no less time than these.  A settled state
        // in sixteen parts / as here: 24 x 8 of 8, V = 32000 float32 274.1 / 267.1, 1 x 4 of 17, V = 32000 bfloat16 100.7 / 94.4, 4 x 4 of 12,
        // V = 32000 float32 169.1 / 162.6, 8 x 4 of 8, V = 128256 bfloat16 178.6 / 179.1.  (In 64 parts for all levels of the launch,
        // whether they modify a row or not: 268.5, 92.8, 174.8, 180.7; with all levels alive 1 x 4 of 16, V = 128256 619 against 388,
        // 2 x 3 of 12, V = 256000 618 against 441.)  Short rows in eight, five, four parts: 10 x 8 of 12, V = 3000 float32 125.2, 123.0, 121.5,
        // 40 x 4 of 8, V = 8000 bfloat16 129.2, 125.3, 123.0, 2 x 4 of 8 78.2, 76.8, 73.9, 2 x 2 of 16, V = 6000 168.5 and 149.5 in four.
        const bool small = pairs <= 6 * cu;
        for (la.from = 0; la.from < p.pend_levels; la.from = la.to) {
            la.to = small && (p.state_count || row_vectors<T>(p.V) < 6000) ? p.pend_levels : la.from + 1;
            const int steps = (vec ? row_vectors<T>(p.V) : p.V) / (2 * kStatThreads);
            la.most = la.to - la.from < 2 || steps > kPendParts ? kPendParts : (steps > 8 ? steps : (steps > 0 ? 8 : 4));
            const dim3 gp(static_cast<unsigned>((la.from == 0 ? least : grid) + (la.to - la.from - 1) * grid));
#define SPECGBV_PEND_LAUNCH(VEC, ONE) hipLaunchKernelGGL((k_pend_norm<T, VEC, ONE>), gp, dim3(kStatThreads), 0, p.stream, target, draft, la)
            if (la.to == 1) { if (vec) SPECGBV_PEND_LAUNCH(true, true); else SPECGBV_PEND_LAUNCH(false, true); }
            else { if (vec) SPECGBV_PEND_LAUNCH(true, false); else SPECGBV_PEND_LAUNCH(false, false); }
            e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
#undef SPECGBV_PEND_LAUNCH
    }
    if (p.L < 2) return hipSuccess;
    const long long rows = static_cast<long long>(p.batch) * p.K * (p.L - 1);
    if (p.s_parts > 1) {                            // small batch: partial sums, added up by the final-token kernel
        const dim3 gq(static_cast<unsigned>(rows * p.s_parts));
#define SPECGBV_OTP_LAUNCH(KERNEL)                                                                                  \
    hipLaunchKernelGGL(KERNEL, gq, dim3(kStatThreads), 0, p.stream, target, draft, p.tokens, p.K, p.L, p.V, p.c, p.s_parts, \
                       stat_part, stat_parts, stats, counter, pend_part, reinterpret_cast<double *>(p.ws + p.lay.excess_part), \
                       pend, pairs, p.pend_levels, p.c_rel)
        if constexpr (kMayBeOdd) {
            if (odd) {
                if (p.pend_levels > 0) SPECGBV_OTP_LAUNCH((k_ot_sum_parts_odd<true>));
                else SPECGBV_OTP_LAUNCH((k_ot_sum_parts_odd<false>));
                return hipGetLastError();
            }
        }
        if (p.pend_levels > 0) { if (vec) SPECGBV_OTP_LAUNCH((k_ot_sum_parts<T, true, true>)); else SPECGBV_OTP_LAUNCH((k_ot_sum_parts<T, false, true>)); }
        else { if (vec) SPECGBV_OTP_LAUNCH((k_ot_sum_parts<T, true, false>)); else SPECGBV_OTP_LAUNCH((k_ot_sum_parts<T, false, false>)); }
#undef SPECGBV_OTP_LAUNCH
        return hipGetLastError();
    }
    const dim3 g2(static_cast<unsigned>(rows));
#define SPECGBV_OT_LAUNCH(VEC, PEND, ODD)                                                                       \
    hipLaunchKernelGGL((k_ot_sum<T, VEC, PEND, ODD>), g2, dim3(kStatThreads), 0, p.stream, target, draft, p.tokens, p.K, p.L, \
                       p.V, p.c, stats, pend, pairs, p.pend_levels, s, reinterpret_cast<double *>(p.ws + p.lay.excess),        \
                       reinterpret_cast<double *>(p.ws + p.lay.excess_part), p.c_rel)
    if (p.pend_levels > 0) {
        if (odd) SPECGBV_OT_LAUNCH(true, true, kMayBeOdd);
        else if (vec) SPECGBV_OT_LAUNCH(true, true, false);
        else SPECGBV_OT_LAUNCH(false, true, false);
    } else {
        if (odd) SPECGBV_OT_LAUNCH(true, false, kMayBeOdd);
        else if (vec) SPECGBV_OT_LAUNCH(true, false, false);
        else SPECGBV_OT_LAUNCH(false, false, false);
    }
#undef SPECGBV_OT_LAUNCH
    return hipGetLastError();
}

}  // namespace

int split_sum_parts(const Problem &p)
{
    if (p.L < 2) return 1;
    return row_parts(static_cast<long long>(p.batch) * p.K * (p.L - 1), p.V);
}

hipError_t launch_split_main(const Problem &p)
{
    return p.dtype == 1 ? launch_typed<uint16_t>(p) : launch_typed<float>(p);
}

}  // namespace specgbv
