// Comparison verifier: SpecTr's K-SEQ rule (paper Section 3.2), and with one draft token-level speculative
// decoding (Section 3.1), on the inputs of the main verification.
//
// At a position the candidates are the tokens of the drafts still retained (those that agree with everything
// accepted so far), taken in draft order; candidate x is accepted with probability min{1, q(x) / (rho p(x))}, and
// if none is accepted the replacement is drawn from (q - rho min{p, q/rho}) / (1 - rho beta(rho)) = norm(max{q - rho p, 0}).
// rho in [1, k] solves 1 - (1 - beta(rho))^k = rho beta(rho), beta(rho) = sum_x min{p(x), q(x)/rho}, with k the
// number of drafts retained at that position.
//
// Which drafts are retained when a position is reached depends only on the tokens: they are the drafts that share
// the accepted block, and the accepted block is always some draft's prefix.  So the root can be found up front
// for every (draft, row), with k = the number of drafts sharing that draft's first r tokens -- all row pairs in
// parallel, no dependence on the random decisions.  That is what k_kseq_rows does:
//     rho beta(rho) = 1 - S(rho),   S(rho) = sum_x max{q - rho p, 0} = sum_x q max(1 - rho p/q, 0)
// is the K = 1 vocabulary sum of the main verifier at block ratio 1/rho, so one sweep over the row pair gives S and
// its slope (-sum_{rho p < q} p), and a safeguarded Newton iteration on f(rho) = (1 - beta)^k - S finds the root in
// a handful of sweeps.  The sequential part (which candidate wins at each position) is then a scalar scan per
// prefix inside the final-token kernel, and the replacement token is that kernel's K = 1 residual draw.
#include "specgbv_internal.hpp"

namespace specgbv {
namespace {

constexpr int kKseqThreads = 512;
// the sweeps of a workgroup read the same row pair again and again: ordinary loads, not the streaming ones
// (2 - 7 % faster: part of a sweep is then served by the cache levels in front of HBM)
constexpr bool kKseqKeep = true;

// G(rho) = sum_x min{rho p, q} = rho beta(rho), S(rho) = sum_x max{q - rho p, 0} = 1 - G, and rho * sum_{rho p < q} p.
// G and S are summed separately and normalised by their own total, so that each keeps its leading digits where it is
// small (G where the models hardly overlap, S where they nearly coincide) whatever the accuracy of the row's normaliser.
struct KseqSums { double G, S, Dr; };

// Three workgroup-wide sums with one barrier: sh holds 2 * 3 * (waves) doubles, `turn` alternates between its halves.
__device__ __forceinline__ KseqSums kseq_block_sums(double G, double S, double Dr, double *sh, int turn)
{
    constexpr int kWaves = kKseqThreads / kWave;
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    double *at = sh + turn * 3 * kWaves;
    G = wave_sum(G); S = wave_sum(S); Dr = wave_sum(Dr);
    if (lane == 0) { at[wid] = G; at[kWaves + wid] = S; at[2 * kWaves + wid] = Dr; }
    __syncthreads();
    KseqSums out{0.0, 0.0, 0.0};
#pragma unroll
    for (int w = 0; w < kWaves; ++w) { out.G += at[w]; out.S += at[kWaves + w]; out.Dr += at[2 * kWaves + w]; }
    const double tot = out.G + out.S;                      // = sum_x q in the sums' own units
    if (tot > 0.0) { out.G /= tot; out.S /= tot; out.Dr /= tot; }
    return out;
}

// The root: f(rho) = G(rho) - 1 + (1 - beta)^n, beta = G / rho, is non-positive at 1, non-negative at n, increasing.  It is
// evaluated as G - beta sum_{j<n} (1 - beta)^j, which keeps its leading digits when G is tiny, or as (1 - beta)^n - S, which
// keeps them where S is.  Newton from the left end, kept inside the bracket by bisection; every quantity is workgroup-uniform.
// It ends where f is below the noise of the float32 sums, or where the bracket or a step is within 2e-7 rho.  A short step
// alone proves nothing: G is piecewise linear, and where one entry holds nearly all mass (low temperatures) its slope falls by
// orders of magnitude as rho p[x] passes q[x], so that a root 2e-7 ahead by the slope in front of that point may be 1e-2 away.
// So the step counts only if f could not move the root further with any slope that f may have on that side; else the next
// sweep is made 2e-7 rho further on, where it either closes the bracket or finds the slope beyond the point.  (0.2 - 1 % more
// sweeps, 8 % where 64 drafts nearly coincide with the target; by the step alone, and with rho kept in float32, rho was off by
// up to 1e-2 at K = 4, V = 100, T = 0.3, drafts close to the target, where it is good to 1e-6.)
// (rho, beta) is the pair of the last sweep, or its continuation along the tangent of G by at most 2e-7 rho.
// sweep(rho, it): KseqSums of step it, the first at rho = 1.  (It is called at one place: a second copy of a sweep over memory took
// k_kseq_rows from three resident workgroups per compute unit to two.)
struct KseqRoot { double rho, beta; };
template <typename Sweep>
__device__ __forceinline__ KseqRoot kseq_root(int n, Sweep sweep)
{
    constexpr double kStep = 2.0e-7;
    double rho = 1.0, lo = 1.0, hi = static_cast<double>(n), beta = 0.0;
    for (int it = 0;; ++it) {
        const KseqSums sm = sweep(rho, it);
        beta = sm.G / rho;
        if (n <= 1) break;                                 // one candidate: rho = 1 (Section 3.1)
        const double b1 = beta < 1.0 ? beta : 1.0, A = 1.0 - b1;
        double geo = 1.0, pw1 = 1.0;                       // sum_{j<n} A^j and A^(n-1)
        for (int j = 1; j < n; ++j) { pw1 *= A; geo += pw1; }
        const double f = b1 > 0.5 ? pw1 * A - sm.S : sm.G - b1 * geo;
        if (f >= 0.0) hi = rho; else lo = rho;
        const double D = sm.Dr / rho;                      // d(rho beta)/d rho = mass of p where rho p < q: falls as rho grows
        const double cc = static_cast<double>(n) * pw1 / rho;
        const double fp = D + cc * (beta - D);
        double nxt = fp > 0.0 ? rho - f / fp : 0.5 * (lo + hi);
        const bool inside = nxt > lo && nxt < hi;
        if (!inside) nxt = 0.5 * (lo + hi);
        const double step = nxt - rho;
        const bool is_short = fabs(step) <= kStep * rho;
        const double D_far = f >= 0.0 ? 1.0 : 0.0;         // D at the far end of the side the root is on: D is between the two
        const double flattest = fmin(fp, D_far + cc * (beta - D_far));
        if (fabs(f) <= 1.0e-7 * fmin(sm.G, sm.S) || hi - lo <= kStep * rho || it >= 40 ||
            (is_short && it > 0 && fabs(f) <= kStep * rho * flattest)) {
            if (inside && is_short) { beta = (sm.G + D * step) / nxt; rho = nxt; }
            break;
        }
        if (is_short) {
            nxt = f >= 0.0 ? rho * (1.0 - kStep) : rho * (1.0 + kStep);
            if (!(nxt > lo && nxt < hi)) nxt = 0.5 * (lo + hi);
        }
        if (nxt == rho) break;
        rho = nxt;
    }
    return KseqRoot{rho, beta};
}

// What a workgroup of either kernel works on: grid batch * ndrafts * L, the row index slowest (rows 0, which all drafts
// share and which take the most steps, come first and the others fill in behind them): row pair r of draft k of prefix b,
// and the number n of drafts (among the first ndrafts) that share the draft's first r tokens.
struct KseqPair { long long bk, pair; int r, k; long long b; };
__device__ __forceinline__ KseqPair kseq_pair(int K, int L, int ndrafts)
{
    KseqPair w;
    const unsigned chains = gridDim.x / static_cast<unsigned>(L), at = blockIdx.x % chains;
    w.r = static_cast<int>(blockIdx.x / chains);
    w.k = static_cast<int>(at % static_cast<unsigned>(ndrafts));
    w.b = at / static_cast<unsigned>(ndrafts);
    w.bk = w.b * K + w.k;
    w.pair = w.bk * L + w.r;
    return w;
}
__device__ __forceinline__ void kseq_begin(const KseqPair &w, const int32_t *tokens, int K, int L, int ndrafts, int32_t *final_counter, int *sh_n)
{
    const int tid = threadIdx.x;
    if (tid == 0) {
        *sh_n = 0;
        if (w.k == 0 && w.r == 0) final_counter[w.b] = 0;  // arrival counter of the final-token kernel
    }
    __syncthreads();
    if (tid < ndrafts) {
        bool same = true;
        for (int j = 0; j < w.r; ++j) same = same && tokens[(w.b * K + tid) * L + j] == tokens[w.bk * L + j];
        if (same) atomicAdd(sh_n, 1);
    }
}
// (zq, zp: the drafted token's two logits)
__device__ __forceinline__ void kseq_store_stats(const KseqPair &w, float zq, float zp, double lse2_q, double lse2_p, float c, double c_rel, RowStat *stats)
{
    RowStat st;
    st.lse2_q = lse2_q; st.lse2_p = lse2_p;
    st.tok2_q = token_scaled(static_cast<double>(zq) * static_cast<double>(c), lse2_q, c_rel);
    st.tok2_p = token_scaled(static_cast<double>(zp) * static_cast<double>(c), lse2_p, c_rel);
    stats[w.pair] = st;
}

// Rows from memory, one sweep per step (any length and address): those that do not fit a workgroup's registers.  With the
// row index slowest and one barrier per step, 32 x 8 drafts of 8 at V = 128256 take 452 us a call, 920 before.
template <typename T, bool VEC>
__global__ void __launch_bounds__(kKseqThreads)
k_kseq_rows(const T *__restrict__ target, const T *__restrict__ draft, const int32_t *__restrict__ tokens, int K, int L,
            int V, int ndrafts, float c, double c_rel, RowStat *__restrict__ stats, double *__restrict__ rho_out,
            double *__restrict__ beta_out, int32_t *__restrict__ final_counter)
{
    __shared__ double sh_d[2 * 3 * (kKseqThreads / kWave)];
    __shared__ float sh_f[kKseqThreads / kWave];
    __shared__ int sh_n;
    const int tid = threadIdx.x;
    const KseqPair w = kseq_pair(K, L, ndrafts);
    kseq_begin(w, tokens, K, L, ndrafts, final_counter, &sh_n);
    const T *rq = target + (w.bk * (L + 1) + w.r) * static_cast<long long>(V);
    const T *rp = draft + w.pair * static_cast<long long>(V);
    constexpr int N = VEC ? Elem<T>::kPerVec : 1;
    RunningSum aq, ap;
    for_each_pair<T, VEC, kKseqThreads, kKseqKeep>(rq, rp, V, [&](int, const float (&zq)[N], const float (&zp)[N]) {
        aq.add(zq, c);
        ap.add(zp, c);
    });
    const float Mq = block_max(aq.m2, sh_f);
    const double Zq = block_sum(aq.Z > 0.0f ? static_cast<double>(aq.Z) * exp2(static_cast<double>(aq.m2) - static_cast<double>(Mq)) : 0.0, sh_d);
    const float Mp = block_max(ap.m2, sh_f);
    const double Zp = block_sum(ap.Z > 0.0f ? static_cast<double>(ap.Z) * exp2(static_cast<double>(ap.m2) - static_cast<double>(Mp)) : 0.0, sh_d);
    const double lse2_q = static_cast<double>(Mq) + log2(Zq), lse2_p = static_cast<double>(Mp) + log2(Zp);
    if (tid == 0) {
        int tok = tokens[w.pair];
        tok = tok < 0 ? 0 : (tok >= V ? V - 1 : tok);
        kseq_store_stats(w, Elem<T>::scalar(rq + tok), Elem<T>::scalar(rp + tok), lse2_q, lse2_p, c, c_rel, stats);
    }
    const int n = sh_n;                                    // (the block sums above contain the barriers that publish it)
    const float shift_q = rintf(static_cast<float>(lse2_q));
    const double C1 = lse2_p - lse2_q;
    __syncthreads();                                       // (the last block sum has been read)
    const KseqRoot root = kseq_root(n, [&](double rho, int it) {
        const RatioConst rc(C1 - log2(rho));               // rho p / q = 2^(c (z_p - z_q) - C2)
        const float kappa = -rc.neg_kappa;
        // summed as min{rho p, q} (not as max{q - rho p, 0} = q - min): where the two models hardly overlap the sum is
        // tiny and the equation for rho is decided by its leading digits
        float G = 0.0f, S = 0.0f, Dr = 0.0f;
        for_each_pair<T, VEC, kKseqThreads, kKseqKeep>(rq, rp, V, [&](int, const float (&zq)[N], const float (&zp)[N]) {
#pragma unroll
            for (int j = 0; j < N; ++j) {
                const float r = exp2_fast(fmaf(zp[j] - zq[j], c, -rc.C2_hi)) * kappa;        // rho p / q
                const float e = exp2_fast(fmaf(zq[j], c, -shift_q));
                const bool open = r < 1.0f;                                                   // rho p < q
                G = fmaf(e, open ? r : 1.0f, G);
                S = fmaf(e, open ? 1.0f - r : 0.0f, S);
                Dr += open ? e * r : 0.0f;
            }
        });
        return kseq_block_sums(static_cast<double>(G), static_cast<double>(S), static_cast<double>(Dr), sh_d, it & 1);
    });
    if (tid == 0) { rho_out[w.pair] = root.rho; beta_out[w.pair] = root.beta; }
}

// Rows of at most NS * kKseqThreads vectors, read once: after the statistics a thread keeps of its entries the weights
// e = q[x] and the ratios p[x] / q[x], and a step is ten instructions per entry, without an exponential and without
// memory.  At 64 entries per thread a workgroup has the compute unit's registers to itself; what bounds it is a row's
// own chain: load, statistics, and a step's sweep and barrier for each of five steps in the rows 0 (most others have a
// single candidate and one step).  Before, a workgroup streamed its row pair alone for every step, 27 us each at
// V = 32000 float32: 32 x 4 drafts of 8 took 206 us a call, 99 now; 64 x 8 in bfloat16 634, 280 now.  A row of one candidate
// takes 18 us there, 7 of them its load and the rest arithmetic (two waves per SIMD, one behind the other), so the first
// step's sums are taken while the weights are formed: 102.7 / 100.3 us a call, 64 x 8 in bfloat16 269.7 / 258.1, 16 x 4 of 5,
// V = 20000 float32 45.2 / 44.7.  (1024 threads with half the entries each: 118 and 317.  One candidate's sums apart, nothing
// kept: the compiler then holds a row twice, 108.)
template <typename T, int NS>
__global__ void __launch_bounds__(kKseqThreads, 2)
k_kseq_onchip(const T *__restrict__ target, const T *__restrict__ draft, const int32_t *__restrict__ tokens, int K, int L,
              int V, int ndrafts, float c, double c_rel, RowStat *__restrict__ stats, double *__restrict__ rho_out,
              double *__restrict__ beta_out, int32_t *__restrict__ final_counter)
{
    constexpr int PV = Elem<T>::kPerVec, NE = NS * PV;
    __shared__ double sh_d[2 * 3 * (kKseqThreads / kWave)];
    __shared__ double sh_Z[2 * (kKseqThreads / kWave)];
    __shared__ float sh_ref[2 * (kKseqThreads / kWave)];
    __shared__ int sh_n;
    const int tid = threadIdx.x;
    const KseqPair w = kseq_pair(K, L, ndrafts);
    const T *rq = target + (w.bk * (L + 1) + w.r) * static_cast<long long>(V);
    const T *rp = draft + w.pair * static_cast<long long>(V);
    const int nv = (V + PV - 1) / PV, before = (PV - V % PV) % PV;      // entries of the last vector that the one before it holds
    const int tok_raw = token_index_queued(tokens, w.pair);
    U4 q[NS], p[NS];
#pragma unroll
    for (int j = 0; j < NS; ++j) {                         // (no branch: a load under one is waited for where the branch ends)
        const int v = j * kKseqThreads + tid;
        int e = (v < nv ? v : nv - 1) * PV;
        e = e < V - PV ? e : V - PV;
        q[j] = load16_stream_any(rq + e);
        p[j] = load16_stream_any(rp + e);
    }
    // (the token's logits are asked for behind the row's loads: fetched where the statistics are stored, their latency held up
    // the whole workgroup at the next barrier)
    const int tok = token_index_used(tok_raw, V);
    const uint32_t tok_q = Elem<T>::bits(rq + tok), tok_p = Elem<T>::bits(rp + tok);
    kseq_begin(w, tokens, K, L, ndrafts, final_counter, &sh_n);
    // entries of slot j: those beyond the row, or held by the vector before, become -inf
    auto unpack = [&](int j, float (&zq)[PV], float (&zp)[PV]) {
        Elem<T>::unpack(q[j], zq);
        Elem<T>::unpack(p[j], zp);
        if ((j + 1) * kKseqThreads >= nv) {                // uniform
            const int v = j * kKseqThreads + tid, cut = v >= nv ? PV : (v == nv - 1 ? before : 0);
#pragma unroll
            for (int e = 0; e < PV; ++e)
                if (e < cut) { zq[e] = -__builtin_inff(); zp[e] = -__builtin_inff(); }
        }
    };
    // Statistics: a running reference per lane, as in k_kseq_rows.  A row that is not a multiple of the vector and gives no
    // lane more than one is summed in float64: entry by entry a lane would add up two of them at most, and eight terms
    // relative to one reference cost accuracy there (ln-normalisers at V = 100 bfloat16, T = 0.8: relative to one reference
    // for the whole row in float32 5.3e-8 rms and 2.6e-7 at most, entry by entry 2e-8 and 6e-8, in float64 4e-11 at most).
    float m2q = -3.0e38f, m2p = -3.0e38f;
    double zsum_q = 0.0, zsum_p = 0.0;
    if (read_by_vectors<T>(V)) {                           // uniform
        RunningSum aq, ap;
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            if (j * kKseqThreads < nv) {                   // uniform
                float zq[PV], zp[PV];
                unpack(j, zq, zp);
                aq.add(zq, c);
                ap.add(zp, c);
            }
            // (opaque touches: the unpacked floats are not kept for the sweeps)
            asm volatile("" : "+v"(q[j].x), "+v"(q[j].y), "+v"(q[j].z), "+v"(q[j].w), "+v"(aq.Z));
            asm volatile("" : "+v"(p[j].x), "+v"(p[j].y), "+v"(p[j].z), "+v"(p[j].w), "+v"(ap.Z));
        }
        m2q = aq.m2; m2p = ap.m2;
        zsum_q = static_cast<double>(aq.Z); zsum_p = static_cast<double>(ap.Z);
    } else {                                               // (nv <= kKseqThreads: slot 0 holds the row)
        RunningSum64 aq, ap;
        float zq[PV], zp[PV];
        unpack(0, zq, zp);
        aq.add(zq, c);
        ap.add(zp, c);
        m2q = aq.m2; m2p = ap.m2;
        zsum_q = aq.Z; zsum_p = ap.Z;
    }
    // The waves' sums relative to integral references meet behind one barrier; every thread adds them up.
    constexpr int kWaves = kKseqThreads / kWave;
    const int lane = tid & (kWave - 1), wid = tid / kWave;
    {
        const float ref_q = integral_reference(wave_max(m2q), 1.0f), ref_p = integral_reference(wave_max(m2p), 1.0f);
        const double a = wave_sum(zsum_q > 0.0 ? zsum_q * exp2_small(static_cast<double>(m2q) - static_cast<double>(ref_q)) : 0.0);
        const double b = wave_sum(zsum_p > 0.0 ? zsum_p * exp2_small(static_cast<double>(m2p) - static_cast<double>(ref_p)) : 0.0);
        if (lane == 0) { sh_ref[wid] = ref_q; sh_ref[kWaves + wid] = ref_p; sh_Z[wid] = a; sh_Z[kWaves + wid] = b; }
    }
    __syncthreads();
    double lse2_q, lse2_p;
    {                                                      // even lanes: the target's row, odd lanes: the draft's
        const int at = (lane & 1) * kWaves;
        float M = -3.0e38f;
#pragma unroll
        for (int x = 0; x < kWaves; ++x) M = fmaxf(M, sh_Z[at + x] > 0.0 ? sh_ref[at + x] : -3.0e38f);
        double Z = 0.0;
#pragma unroll
        for (int x = 0; x < kWaves; ++x) Z += ldexp(sh_Z[at + x], reference_shift(sh_ref[at + x], M));
        const double l = Z > 0.0 ? static_cast<double>(M) + log2_series(Z) : -static_cast<double>(__builtin_inff());
        lse2_q = lane_value(l, 0); lse2_p = lane_value(l, 1);
    }
    if (tid == 0) kseq_store_stats(w, Elem<T>::from_bits(tok_q), Elem<T>::from_bits(tok_p), lse2_q, lse2_p, c, c_rel, stats);
    const int n = __builtin_amdgcn_readfirstlane(sh_n);    // (written in front of the barrier above)
    const float shift_q = rintf(static_cast<float>(lse2_q));
    const RatioConst rc(lse2_p - lse2_q);
    const float kappa = -rc.neg_kappa;
    // The weights and ratios, and the first step's sums (rho = 1) as they are formed.
    float ew[NE], rw[NE];
    float C0 = 0.0f, S0 = 0.0f, D0 = 0.0f;
    auto add = [](float e, float r, float &C, float &S, float &Dr) {
        const float s = 1.0f - r;
        const bool open = s > 0.0f;                        // rho p < q, the same for all three sums
        Dr = fmaf(e, open ? r : 0.0f, Dr);
        S = fmaf(e, fmaxf(s, 0.0f), S);
        C += open ? 0.0f : e;                              // mass of q where rho p >= q
    };
#pragma unroll
    for (int j = 0; j < NS; ++j) {
        float zq[PV], zp[PV];
        unpack(j, zq, zp);
#pragma unroll
        for (int e = 0; e < PV; ++e) {
            const float x = exp2_fast(fmaf(zq[e], c, -shift_q));
            const float r = exp2_fast(fmaf(zp[e] - zq[e], c, -rc.C2_hi)) * kappa;     // (masked entries: weight 0, whatever the ratio)
            ew[j * PV + e] = x; rw[j * PV + e] = r;
            add(x, r, C0, S0, D0);
        }
    }
    const KseqSums at_one = kseq_block_sums(static_cast<double>(C0) + static_cast<double>(D0), static_cast<double>(S0), static_cast<double>(D0), sh_d, 0);
    const KseqRoot root = kseq_root(n, [&](double rho, int it) {
        if (it == 0) return at_one;                        // (uniform)
        const float rf = static_cast<float>(rho), rl = static_cast<float>(rho - static_cast<double>(rf));
        float C = 0.0f, S = 0.0f, Dr = 0.0f;
#pragma unroll
        for (int e = 0; e < NE; ++e) add(ew[e], fmaf(rf, rw[e], rl * rw[e]), C, S, Dr);     // (where p / q overflows r may be NaN: then not open)
        return kseq_block_sums(static_cast<double>(C) + static_cast<double>(Dr), static_cast<double>(S), static_cast<double>(Dr), sh_d, it & 1);
    });
    if (tid == 0) { rho_out[w.pair] = root.rho; beta_out[w.pair] = root.beta; }
}

template <typename T>
hipError_t launch_kseq_typed(const Problem &p, int ndrafts)
{
    const T *target = static_cast<const T *>(p.target);
    const T *draft = static_cast<const T *>(p.draft);
    const bool vec = read_by_vectors<T>(p.V);
    const dim3 grid(static_cast<unsigned>(static_cast<long long>(p.batch) * ndrafts * p.L));
    RowStat *stats = reinterpret_cast<RowStat *>(p.ws + p.lay.stats);
    double *rho = reinterpret_cast<double *>(p.ws + p.lay.s);
    double *beta = reinterpret_cast<double *>(p.ws + p.lay.excess);
    int32_t *counter = reinterpret_cast<int32_t *>(p.ws + p.lay.counter);
    constexpr int PV = Elem<T>::kPerVec;
    const int nv = (p.V + PV - 1) / PV;
#define SPECGBV_KSEQ_ONCHIP(NS)                                                                                       \
    hipLaunchKernelGGL((k_kseq_onchip<T, NS>), grid, dim3(kKseqThreads), 0, p.stream, target, draft, p.tokens, p.K, p.L, \
                       p.V, ndrafts, p.c, p.c_rel, stats, rho, beta, counter)
    // 16, 32 and 64 entries per thread; 64 leave room for one workgroup per compute unit, whose load, statistics and steps
    // then follow one another with nothing beside them.  That pays where rows 0 take five steps from registers instead of
    // memory, not for a single draft, whose rows all take one (128 drafts of 5, V = 20000 float32: 63 us from registers, 51
    // from memory), and not for rows that 32 hold (64 x 4 drafts of 5, V = 10000 float32: 112 us with 64, 73 with 32, 83
    // from memory; 128 drafts of 5: 54, 37, 36; at 16384: 60, 41, 44).
    if (p.V >= PV && nv <= 16 / PV * kKseqThreads) SPECGBV_KSEQ_ONCHIP(16 / PV);
    else if (p.V >= PV && nv <= 32 / PV * kKseqThreads) SPECGBV_KSEQ_ONCHIP(32 / PV);
    else if (p.V >= PV && ndrafts > 1 && nv <= 64 / PV * kKseqThreads) SPECGBV_KSEQ_ONCHIP(64 / PV);
    else if (vec)
        hipLaunchKernelGGL((k_kseq_rows<T, true>), grid, dim3(kKseqThreads), 0, p.stream, target, draft, p.tokens, p.K, p.L,
                           p.V, ndrafts, p.c, p.c_rel, stats, rho, beta, counter);
    else
        hipLaunchKernelGGL((k_kseq_rows<T, false>), grid, dim3(kKseqThreads), 0, p.stream, target, draft, p.tokens, p.K, p.L,
                           p.V, ndrafts, p.c, p.c_rel, stats, rho, beta, counter);
#undef SPECGBV_KSEQ_ONCHIP
    return hipGetLastError();
}

}  // namespace

hipError_t launch_kseq_rows(const Problem &p, int ndrafts)
{
    return p.dtype == 1 ? launch_kseq_typed<uint16_t>(p, ndrafts) : launch_kseq_typed<float>(p, ndrafts);
}

}  // namespace specgbv
