// Distribution modification (Algorithm 2): the target distribution of the first rows of the
// next iteration.
//
// After an iteration accepted t^tau and drew the final token y, the first count = L - tau - 1
// rows of every new draft use
//     q_new[x] = w[x] / sum_x w[x],   w[x] = q_r[x] max(1 - p_r[x] / (nu q_r[x]), 0)^K
// (Algorithm 2 divided through by the joint probability of the conditioning block: the same
// per-token form as Eq. (pres)), with nu = [q(t^tau, y) / p(t^tau, y)] continued along the new
// draft's own tokens with the original target probabilities.
//
// Three streaming kernels, each with one workgroup per row (pair), so that any batch size
// fills the chip:
//   k_mod_stats : per row, log2 sum_x 2^(c z[x]) and the drafted token's scaled logit
//   k_mod_norm  : per modified row pair, nu (a prefix sum over the statistics of the rows
//                 before it) and the normaliser sum_x w[x]
//   k_mod_write : per row pair, natural-log probabilities in float32 (-inf where the
//                 probability is 0): ln q_new for modified rows, ln q otherwise, and ln p.
// An optional extra target row (the bonus row of the verification) is converted to
// log-probabilities as well, so that the whole output can be verified at temperature 1.
//
// Rows of up to kRowSlots * 512 sixteen-byte vectors take a shorter route: k_mod_row keeps a row in the registers of
// its workgroup between the statistics sweep and the store of its log-probabilities, so every row that no
// modification touches (all draft rows, the target rows from the prefix's count on, the bonus row) is read once;
// k_mod_pair then makes normaliser and ln q_new of the modified target rows.
#include "specgbv_internal.hpp"

namespace specgbv {
namespace {

constexpr int kModThreads = 512;

struct ModStat { double lse2, tok2; };       // base-2 log-normaliser, scaled logit of the row's token

// Workspace of one call: statistics of the target rows, of the draft rows, normalisers, flags.
struct ModLayout {
    size_t tstat, dstat, norm, fb, total;
};
__host__ __device__ inline size_t mod_align(size_t v) { return (v + 255) & ~static_cast<size_t>(255); }
inline ModLayout mod_layout(int batch, int K, int M, int bonus)
{
    ModLayout l{};
    const size_t bk = static_cast<size_t>(batch) * K;
    size_t off = 0;
    l.tstat = off; off = mod_align(off + bk * (M + bonus) * sizeof(ModStat));
    l.dstat = off; off = mod_align(off + bk * M * sizeof(ModStat));
    l.norm = off; off = mod_align(off + bk * M * sizeof(double));
    l.fb = off; off = mod_align(off + bk * M * sizeof(int32_t));
    l.total = off;
    return l;
}

// grid.x = target rows followed by draft rows
template <typename T, bool VEC>
__global__ void __launch_bounds__(kModThreads)
k_mod_stats(const T *__restrict__ target, const T *__restrict__ draft, const int32_t *__restrict__ tokens,
            int M, int bonus, int V, float c, long long n_trows, ModStat *__restrict__ tstat,
            ModStat *__restrict__ dstat)
{
    __shared__ double sh_d[kModThreads / kWave];
    __shared__ float sh_f[kModThreads / kWave];
    const long long id = blockIdx.x;
    const bool is_draft = id >= n_trows;
    const long long row = is_draft ? id - n_trows : id;
    const T *z_row = (is_draft ? draft : target) + row * static_cast<long long>(V);
    const int rows_t = M + bonus;
    const int r = static_cast<int>(row % (is_draft ? M : rows_t));
    const long long bk = row / (is_draft ? M : rows_t);
    constexpr int PV = Elem<T>::kPerVec;
    RunningSum acc;
    if (VEC) {
        const int nvec = row_vectors<T>(V);
        auto add = [&](const U4 &raw, int v) {
            float z[PV];
            Elem<T>::unpack(raw, z);
            mask_repeated<T>(z, v, V);
            acc.add(z, c);
        };
        int v = threadIdx.x;
        for (; v + kModThreads < nvec; v += 2 * kModThreads) {          // two loads in flight per thread
            const U4 a = load16_stream_any(z_row + vector_entry<T>(v, V));
            const U4 b = load16_stream_any(z_row + vector_entry<T>(v + kModThreads, V));
            add(a, v);
            add(b, v + kModThreads);
        }
        if (v < nvec) add(load16_stream_any(z_row + vector_entry<T>(v, V)), v);
    } else {
        for (int x = threadIdx.x; x < V; x += kModThreads) {
            const float z[1] = {Elem<T>::scalar(z_row + x)};
            acc.add(z, c);
        }
    }
    const float Mx = block_max(acc.m2, sh_f);
    const double total = block_sum(static_cast<double>(acc.Z * exp2_fast(acc.m2 - Mx)), sh_d);
    if (threadIdx.x == 0) {
        ModStat st;
        st.lse2 = static_cast<double>(Mx) + log2(total);
        st.tok2 = 0.0;
        if (r < M) {                                   // the bonus row has no token
            int tok = tokens[bk * M + r];
            tok = tok < 0 ? 0 : (tok >= V ? V - 1 : tok);
            st.tok2 = static_cast<double>(Elem<T>::scalar(z_row + tok)) * static_cast<double>(c);
        }
        (is_draft ? dstat : tstat)[row] = st;
    }
}

// Vectors per thread that k_mod_row keeps.  40: rows up to 163840 bfloat16 / 81920 float32 entries, one workgroup per
// compute unit.  12: up to 49152 / 24576 entries, three workgroups per compute unit, which a row of few vectors needs, since
// its load, sum and stores follow one another; two of rows in halves (ModLane), whose second addresses take it to 82 registers.
// (Held to 80, with three: 64 x 16 drafts of 8, V = 10000 241 us a call / 237, 12288 271 / 267, but 32 x 8 of 8, V = 24000 140 /
// 148, 32000 188 / 197.)  32 x 8 drafts of 8, bfloat16, by 40, by 12 and by k_mod_stats (rows read
// twice), us a call: V = 8193 133, 81, 80; 16385 184, 129, 138; 40961 353, 321, 359.  (8 or 16 are each 3 - 10 % slower at
// one end of the range that they share with 12.)
constexpr int kRowSlots = 40, kShortRowSlots = 12;

// Four floats to an address that needs the alignment of one only.
__device__ __forceinline__ void store16_any(float *dst, float a, float b, float c, float d)
{
    typedef float F4 __attribute__((ext_vector_type(4)));
    typedef F4 F4any __attribute__((aligned(4)));
    *(__attribute__((address_space(1))) F4any *)dst = F4{a, b, c, d};
}
// ... which nothing reads again soon (for stores of a wave that lie side by side: with gaps between the lanes they are slower).
__device__ __forceinline__ void store16_stream_any(float *dst, float a, float b, float c, float d)
{
    typedef float F4 __attribute__((ext_vector_type(4)));
    typedef F4 F4any __attribute__((aligned(4)));
    __builtin_nontemporal_store(F4{a, b, c, d}, (__attribute__((address_space(1))) F4any *)dst);
}

// 8 (or 4) consecutive floats of an output row.  (k_mod_write: four are a wave's 1 KiB without gaps, 8 x 8 drafts of 8 at
// V = 128000 float32 403 / 394 us a call.)
template <int N>
__device__ __forceinline__ void store_vals(float *dst, const float (&v)[N])
{
    if (N % 4 == 0) {
#pragma unroll
        for (int j = 0; j < N; j += 4) {
            if constexpr (N == 4) store16_stream_any(dst, v[0], v[1], v[2], v[3]);
            else store16_any(dst + j, v[j], v[j + 1], v[j + 2], v[j + 3]);
        }
    } else {
#pragma unroll
        for (int j = 0; j < N; ++j) dst[j] = v[j];
    }
}

// How k_mod_row and k_mod_pair deal a row out: vector v of the row is lane v % 64's.  What bounds them is memory, two thirds of
// it the results' stores (5.2 TB/s at V = 128256 before).  Of whole bfloat16 rows (V a multiple of 8) a lane takes two half
// vectors, four entries each, 256 entries apart: the four floats that a half becomes then lie beside the neighbouring lane's,
// so that a wave's store is 1 KiB without gaps and can pass the caches by.  (With a lane's eight floats in two stores, every
// other 16 bytes each, stores that pass the caches by take 25 % longer than ordinary ones; halves with ordinary stores 109 us at
// V = 16384 below.)  Us a call before / after: 32 x 8 drafts of 8 bfloat16, V = 128256 837 / 809, 49152 311 / 299, 32000 208 /
// 187, 16384 111 / 99; float32, whose vectors always lay so, V = 64128 570 / 529, 32 x 4 of 8 at V = 12000 59 / 52.
enum ModForm { kRagged, kWhole, kHalved };                     // (the row is not a multiple of the vector, is one, and in halves)
template <typename T, ModForm FORM>
struct ModLane {
    static constexpr int PV = Elem<T>::kPerVec;
    static constexpr bool WHOLE = FORM != kRagged, kHalves = FORM == kHalved;
    static_assert(!kHalves || PV == 8, "halves of four entries");
    static constexpr int kHalfStep = kWave * 4;                // entries from a lane's first half to its second
    __device__ static __forceinline__ int first_entry(int v) { return (v & ~(kWave - 1)) * PV + (v & (kWave - 1)) * 4; }
    // Whether the lane has entries of vector v in a row of nvec, and whether any lane of the wave has.
    __device__ static __forceinline__ bool live(int v, int nvec) { return kHalves ? first_entry(v) < nvec * PV : v < nvec; }
    __device__ static __forceinline__ bool any_live(int v, int nvec) { return (kHalves ? v & ~(kWave - 1) : v) < nvec; }
    // (in the row for any v: what lies beyond it is not used)
    template <bool STREAM>
    __device__ static __forceinline__ U4 load(const T *row, int v, int nvec, int V)
    {
        if constexpr (kHalves) {
            typedef unsigned int V2 __attribute__((ext_vector_type(2)));
            typedef V2 V2any __attribute__((aligned(2)));
            const int e0 = first_entry(v), e1 = e0 + kHalfStep;
            const auto *a = (const __attribute__((address_space(1))) V2any *)(row + (e0 < V ? e0 : V - 4));
            const auto *b = (const __attribute__((address_space(1))) V2any *)(row + (e1 < V ? e1 : V - 4));
            const V2 x = STREAM ? __builtin_nontemporal_load(a) : *a, y = STREAM ? __builtin_nontemporal_load(b) : *b;
            return U4{x.x, x.y, y.x, y.y};
        } else {
            const T *at = row + (WHOLE ? (v < nvec ? v : nvec - 1) * PV : vector_entry<T>(v, V));
            return STREAM ? load16_stream_any(at) : load16_any(at);
        }
    }
    // A live vector's logits; entries that are not the lane's become -inf.
    __device__ static __forceinline__ void unpack(const U4 &raw, int v, int V, float (&z)[PV])
    {
        Elem<T>::unpack(raw, z);
        if constexpr (kHalves) {
            if (first_entry(v) + kHalfStep >= V) {
#pragma unroll
                for (int e = 4; e < PV; ++e) z[e] = -__builtin_inff();
            }
        } else if constexpr (!WHOLE) mask_repeated<T>(z, v, V);
    }
    // A live vector's results.  (Entries that the vector before holds too: the same values again.)
    __device__ static __forceinline__ void store(float *row, int v, int V, const float (&o)[PV])
    {
        if constexpr (kHalves) {
            float *dst = row + first_entry(v);
            store16_stream_any(dst, o[0], o[1], o[2], o[3]);
            if (first_entry(v) + kHalfStep < V) store16_stream_any(dst + kHalfStep, o[4], o[5], o[6], o[7]);
        } else if constexpr (PV == 4) {
            store16_stream_any(row + (WHOLE ? v * PV : vector_entry<T>(v, V)), o[0], o[1], o[2], o[3]);
        } else {
            store_vals(row + (WHOLE ? v * PV : vector_entry<T>(v, V)), o);
        }
    }
};

// k_mod_stats for rows of at most kRowSlots * kModThreads vectors, with the row kept in registers: the workgroup
// then also writes the row's natural-log probabilities unless a modification is pending for it (target rows below
// the prefix's count: k_mod_pair does those).  grid.x = target rows followed by draft rows; all of a
// thread's loads are issued before the first is used.  FORM: see ModLane (masking a repeated end in
// all slots instead costs 2 - 9 % in float32: 2 x 8 drafts of 4 at V = 64000 58 us, 62 with it).
template <typename T, ModForm FORM, int SLOTS>
__global__ void __launch_bounds__(kModThreads)
k_mod_row(const T *__restrict__ target, const T *__restrict__ draft, const int32_t *__restrict__ tokens, int K,
          int M, int bonus, int V, float c, long long n_trows, const int32_t *__restrict__ modify_count,
          ModStat *__restrict__ tstat, ModStat *__restrict__ dstat, float *__restrict__ out_logq,
          float *__restrict__ out_logp)
{
    constexpr float kLn2f = 0.693147180559945309417f;
    __shared__ double sh_d[kModThreads / kWave];
    __shared__ float sh_f[kModThreads / kWave];
    const long long id = blockIdx.x;
    const bool is_draft = id >= n_trows;
    const long long row = is_draft ? id - n_trows : id;
    const T *z_row = (is_draft ? draft : target) + row * static_cast<long long>(V);
    const int rows_t = M + bonus;
    const int r = static_cast<int>(row % (is_draft ? M : rows_t));
    const long long bk = row / (is_draft ? M : rows_t);
    constexpr int PV = Elem<T>::kPerVec;
    using Lane = ModLane<T, FORM>;
    const int nvec = row_vectors<T>(V);                    // host: nvec <= SLOTS * kModThreads
    const int tid = threadIdx.x;
    U4 v[SLOTS];
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) {
        const int idx = j * kModThreads + tid;
        if (j * kModThreads < nvec)                        // (uniform: slots the row does not reach issue nothing)
            v[j] = Lane::template load<true>(z_row, idx, nvec, V);
        else
            v[j] = U4{0, 0, 0, 0};
    }
    RunningSum acc;
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) {
        if (Lane::live(j * kModThreads + tid, nvec)) {
            float z[PV];
            Lane::unpack(v[j], j * kModThreads + tid, V, z);
            acc.add(z, c);
        }
    }
    const float Mx = block_max(acc.m2, sh_f);
    const double total = block_sum(static_cast<double>(acc.Z * exp2_fast(acc.m2 - Mx)), sh_d);
    const double lse2 = static_cast<double>(Mx) + log2(total);
    if (tid == 0) {
        ModStat st;
        st.lse2 = lse2;
        st.tok2 = 0.0;
        if (r < M) {                                       // the bonus row has no token
            int tok = tokens[bk * M + r];
            tok = tok < 0 ? 0 : (tok >= V ? V - 1 : tok);
            st.tok2 = static_cast<double>(Elem<T>::scalar(z_row + tok)) * static_cast<double>(c);
        }
        (is_draft ? dstat : tstat)[row] = st;
    }
    float *out = is_draft ? out_logp : out_logq;
    if (!is_draft && r < M && r < modify_count[bk / K]) out = nullptr;     // a modification is pending for this row
    if (!out) return;
    out += row * static_cast<long long>(V);
    // log2 prob[x] = fma(z, c, -h) - d with a float reference h and its float64 remainder d (as k_mod_write)
    const float h = static_cast<float>(lse2);
    const float dlt = static_cast<float>(lse2 - static_cast<double>(h));
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) {
        const int idx = j * kModThreads + tid;
        if (Lane::live(idx, nvec)) {
            float z[PV], a[PV];
            Elem<T>::unpack(v[j], z);
#pragma unroll
            for (int e = 0; e < PV; ++e) a[e] = (fmaf(z[e], c, -h) - dlt) * kLn2f;
            Lane::store(out, idx, V, a);
        }
    }
}

// log2 of the block ratio in front of row r of draft bk: the carried ratio times the token
// ratios of rows 0..r-1 (original target probabilities).
__device__ __forceinline__ double mod_log2nu(const ModStat *tstat, const ModStat *dstat, long long bk, int rows_t,
                                             int M, int r, double carry_ln)
{
    double l = carry_ln * 1.44269504088896340736;
    for (int j = 0; j < r; ++j) {
        const ModStat a = tstat[bk * rows_t + j], b = dstat[bk * M + j];
        l += (a.tok2 - a.lse2) - (b.tok2 - b.lse2);
    }
    return l;
}

// grid.x = batch * K * M, row index slowest (the live workgroups, rows below the prefix's count, are then
// consecutive and spread over all dies whatever M is); row pairs with r >= count leave at once
template <typename T, bool VEC>
__global__ void __launch_bounds__(kModThreads)
k_mod_norm(const T *__restrict__ target, const T *__restrict__ draft, int K, int M, int bonus, int V, float c,
           const double *__restrict__ carry_log_nu, const int32_t *__restrict__ modify_count,
           const ModStat *__restrict__ tstat, const ModStat *__restrict__ dstat, double *__restrict__ norm,
           int32_t *__restrict__ fb_out)
{
    __shared__ double sh_d[kModThreads / kWave];
    const long long nbk = gridDim.x / M;
    const int r = static_cast<int>(blockIdx.x / nbk);
    const long long bk = blockIdx.x % nbk;
    const long long drow = bk * M + r;
    const int b = static_cast<int>(bk / K);
    const int rows_t = M + bonus;
    if (r >= modify_count[b]) {                       // uniform over the workgroup
        if (threadIdx.x == 0) { norm[drow] = 1.0; fb_out[drow] = 0; }
        return;
    }
    const ModStat sq = tstat[bk * rows_t + r], sp = dstat[drow];
    const float shift_q = static_cast<float>(sq.lse2);
    const RatioConst rc(sp.lse2 - sq.lse2 + mod_log2nu(tstat, dstat, bk, rows_t, M, r, carry_log_nu[b]));
    const T *rq = target + (bk * rows_t + r) * static_cast<long long>(V);
    const T *rp = draft + drow * static_cast<long long>(V);
    constexpr int N = VEC ? Elem<T>::kPerVec : 1;
    float acc = 0.0f;
    for_each_pair<T, VEC, kModThreads>(rq, rp, V, [&](int, const float (&zq)[N], const float (&zp)[N]) {
        float wq[N], w[N];
        ot_weights(zq, zp, c, shift_q, rc, K, wq, w);
#pragma unroll
        for (int j = 0; j < N; ++j) acc += w[j];
    });
    const double S = block_sum(static_cast<double>(acc), sh_d);           // relative to 2^shift_q
    if (threadIdx.x == 0) {
        const double W = S * exp2(static_cast<double>(shift_q) - sq.lse2);
        const bool zero = !(W > 0.0);                // every weight is zero: the row stays q
        norm[drow] = zero ? 1.0 : W;
        fb_out[drow] = zero ? 1 : 0;
    }
}

// Modified row pairs of rows that k_mod_row takes: normaliser and ln q_new in one kernel.  grid.x = batch * K * M, row index
// slowest as in k_mod_norm; row pairs with r >= count leave at once.  What bounds it: HBM, the pair's reads and one write of the
// row.  A workgroup keeps the first SLOTS vector pairs per thread in registers between the sum and the stores; the rest of a longer
// row is read again by the workgroup that has just read it, last vectors first, with no non-temporal hint on its first read.  (At
// V = 128256 bfloat16 nine of 32 slots are kept and 71 % of the pair is read again; 1.61 times the pair passes the second-level
// caches, so that 0.1 of the 0.71 is met there, and how much the last-level cache holds no counter here tells.  The two
// kernels this one replaces read all of it twice.)  Two workgroups per compute
// unit: one loads while the other stores.  Microseconds a call with the two kernels / with this one: 32 x 8 drafts of 8,
// bfloat16, V = 128256 841 / 822 (the reads and writes together run at 5 TB/s, as a copy does), 32000 223 / 209, 8193 82.7 /
// 78.4; 16 x 8 of 8, V = 40961 192 / 161; 32 x 4 of 8, V = 12000 float32 71 / 59.6; 2 x 3 of 8, V = 128256 84 / 74.  Slots: 20
// (one workgroup per unit) 833 at V = 128256 and 225 at 32000, 6 831 and 206; rows of up to 6 slots in the tile of 9
// 63.9 instead of 59.6 (V = 12000), 49.8 instead of 48.6 (32 x 8 of 8, V = 4096).
constexpr int kPairSlots = 9, kShortPairSlots = 6;

template <typename T, ModForm FORM, int SLOTS>
__global__ void __launch_bounds__(kModThreads, 4)
k_mod_pair(const T *__restrict__ target, const T *__restrict__ draft, int K, int M, int bonus, int V, float c,
           const double *__restrict__ carry_log_nu, const int32_t *__restrict__ modify_count,
           const ModStat *__restrict__ tstat, const ModStat *__restrict__ dstat, double *__restrict__ norm,
           int32_t *__restrict__ fb_out, float *__restrict__ out_logq)
{
    constexpr float kLn2f = 0.693147180559945309417f;
    __shared__ double sh_d[kModThreads / kWave];
    const long long nbk = gridDim.x / M;
    const int r = static_cast<int>(blockIdx.x / nbk);
    const long long bk = blockIdx.x % nbk;
    const long long drow = bk * M + r;
    const int b = static_cast<int>(bk / K);
    const int rows_t = M + bonus, tid = threadIdx.x;
    if (r >= modify_count[b]) {                       // uniform over the workgroup
        if (tid == 0) { norm[drow] = 1.0; fb_out[drow] = 0; }
        return;
    }
    constexpr int PV = Elem<T>::kPerVec;
    using Lane = ModLane<T, FORM>;
    const T *rq = target + (bk * rows_t + r) * static_cast<long long>(V);
    const T *rp = draft + drow * static_cast<long long>(V);
    float *oq = out_logq + (bk * rows_t + r) * static_cast<long long>(V);
    const int nvec = row_vectors<T>(V);
    U4 q[SLOTS], p[SLOTS];
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) {
        q[j] = p[j] = U4{0, 0, 0, 0};
        if (j * kModThreads < nvec) {                 // (uniform)
            q[j] = Lane::template load<true>(rq, j * kModThreads + tid, nvec, V);
            p[j] = Lane::template load<true>(rp, j * kModThreads + tid, nvec, V);
        }
    }
    const ModStat sq = tstat[bk * rows_t + r], sp = dstat[drow];
    const float shift_q = static_cast<float>(sq.lse2);
    const RatioConst rc(sp.lse2 - sq.lse2 + mod_log2nu(tstat, dstat, bk, rows_t, M, r, carry_log_nu[b]));
    float acc = 0.0f;
    auto add = [&](const U4 &a, const U4 &d, int v) {
        float zq[PV], zp[PV], wq[PV], w[PV];
        Lane::unpack(a, v, V, zq);
        Lane::unpack(d, v, V, zp);
        ot_weights(zq, zp, c, shift_q, rc, K, wq, w);
#pragma unroll
        for (int e = 0; e < PV; ++e) acc += w[e];
    };
    // (a slot's registers pass through a point in program order: its unpacked values are neither formed ahead of time nor kept)
    auto touch = [](U4 &v) { asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w)); };
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) {
        if (Lane::live(j * kModThreads + tid, nvec)) {
            touch(q[j]); touch(p[j]);
            add(q[j], p[j], j * kModThreads + tid);
        }
    }
    auto again = [&](const T *row, int v) { return Lane::template load<false>(row, v, nvec, V); };
    for (int v = SLOTS * kModThreads + tid; Lane::any_live(v, nvec); v += 2 * kModThreads) {
        const int u = v + kModThreads;
        const U4 q0 = again(rq, v), p0 = again(rp, v), q1 = again(rq, u), p1 = again(rp, u);
        if (Lane::live(v, nvec)) add(q0, p0, v);
        if (Lane::live(u, nvec)) add(q1, p1, u);
    }
    const double S = block_sum(static_cast<double>(acc), sh_d);           // relative to 2^shift_q
    const double W = S * exp2(static_cast<double>(shift_q) - sq.lse2);
    const bool zero = !(W > 0.0);                     // every weight is zero: the row stays q
    if (tid == 0) { norm[drow] = zero ? 1.0 : W; fb_out[drow] = zero ? 1 : 0; }
    // ln q_new = ln q + K ln t - ln W; log2 q[x] = fma(z, c, -hq) - dq with a float reference hq and its float64 remainder dq
    const float hq = shift_q, Kf = zero ? 0.0f : static_cast<float>(K);
    const float dq = zero ? static_cast<float>(sq.lse2 - static_cast<double>(hq))
                          : static_cast<float>(log2(W) + sq.lse2 - static_cast<double>(hq));
    auto write = [&](const U4 &a, const U4 &d, int v) {
        float zq[PV], zp[PV], o[PV];
        Elem<T>::unpack(a, zq);
        Elem<T>::unpack(d, zp);
        if (zero) {                                   // uniform
#pragma unroll
            for (int e = 0; e < PV; ++e) o[e] = (fmaf(zq[e], c, -hq) - dq) * kLn2f;
        } else {
#pragma unroll
            for (int e = 0; e < PV; ++e)
                o[e] = (fmaf(Kf, __log2f(rc.one_minus_ratio(zp[e] - zq[e], c)), fmaf(zq[e], c, -hq)) - dq) * kLn2f;
        }
        Lane::store(oq, v, V, o);
    };
    // the vectors that are read again, last first
    for (int j = (nvec - 1) / kModThreads; j >= SLOTS; j -= 2) {          // uniform
        const int v = j * kModThreads + tid, u = j - 1 >= SLOTS ? v - kModThreads : v;
        const U4 q0 = again(rq, v), p0 = again(rp, v), q1 = again(rq, u), p1 = again(rp, u);
        if (Lane::live(v, nvec)) write(q0, p0, v);
        if (u != v) write(q1, p1, u);
    }
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) {
        if (Lane::live(j * kModThreads + tid, nvec)) {
            touch(q[j]); touch(p[j]);
            write(q[j], p[j], j * kModThreads + tid);
        }
    }
}

// grid.x = batch * K * (M + bonus) target rows
template <typename T, bool VEC>
__global__ void __launch_bounds__(kModThreads)
k_mod_write(const T *__restrict__ target, const T *__restrict__ draft, int K, int M, int bonus, int V, float c,
            const double *__restrict__ carry_log_nu, const int32_t *__restrict__ modify_count,
            const ModStat *__restrict__ tstat, const ModStat *__restrict__ dstat, const double *__restrict__ norm,
            const int32_t *__restrict__ fb_in, float *__restrict__ out_logq, float *__restrict__ out_logp)
{
    constexpr float kLn2f = 0.693147180559945309417f;
    const long long trow = blockIdx.x;
    const int rows_t = M + bonus;
    const int r = static_cast<int>(trow % rows_t);
    const long long bk = trow / rows_t;
    const int b = static_cast<int>(bk / K);
    const bool has_draft = r < M;
    const long long drow = bk * M + (has_draft ? r : M - 1);          // bonus row: any valid draft row, unused
    const ModStat sq = tstat[trow], sp = dstat[drow];
    // log2 q[x] = fma(z, c, -hq) - dq with a float reference hq and its float64 remainder dq
    const float hq = static_cast<float>(sq.lse2), hp = static_cast<float>(sp.lse2);
    const float dq = static_cast<float>(sq.lse2 - static_cast<double>(hq));
    const float dp = static_cast<float>(sp.lse2 - static_cast<double>(hp));
    const bool modified = has_draft && r < modify_count[b] && fb_in[drow] == 0;
    const T *rq = target + trow * static_cast<long long>(V);
    const T *rp = has_draft ? draft + drow * static_cast<long long>(V) : rq;   // bonus row: no second stream
    float *oq = out_logq + trow * static_cast<long long>(V);
    float *op = (out_logp && has_draft) ? out_logp + drow * static_cast<long long>(V) : nullptr;
    constexpr int N = VEC ? Elem<T>::kPerVec : 1;
    if (modified) {
        // ln q_new = ln q + K ln t - ln W
        const RatioConst rc(sp.lse2 - sq.lse2 + mod_log2nu(tstat, dstat, bk, rows_t, M, r, carry_log_nu[b]));
        const float log2W = static_cast<float>(log2(norm[drow]) + sq.lse2 - static_cast<double>(hq));   // relative to 2^hq
        const float Kf = static_cast<float>(K);
        for_each_pair<T, VEC, kModThreads, false, true>(rq, rp, V, [&](int x, const float (&zq)[N], const float (&zp)[N]) {
            float a[N], bb[N];
#pragma unroll
            for (int j = 0; j < N; ++j) {
                a[j] = (fmaf(Kf, __log2f(rc.one_minus_ratio(zp[j] - zq[j], c)), fmaf(zq[j], c, -hq)) - log2W) * kLn2f;
                bb[j] = (fmaf(zp[j], c, -hp) - dp) * kLn2f;
            }
            store_vals(oq + x, a);
            if (op) store_vals(op + x, bb);
        });
    } else {
        for_each_pair<T, VEC, kModThreads, false, true>(rq, rp, V, [&](int x, const float (&zq)[N], const float (&zp)[N]) {
            float a[N], bb[N];
#pragma unroll
            for (int j = 0; j < N; ++j) {
                a[j] = (fmaf(zq[j], c, -hq) - dq) * kLn2f;
                bb[j] = (fmaf(zp[j], c, -hp) - dp) * kLn2f;
            }
            store_vals(oq + x, a);
            if (op) store_vals(op + x, bb);
        });
    }
}

// Whether n floats at `out` share memory with m logits at `in`.
template <typename T>
bool overlap(const float *out, long long n, const T *in, long long m)
{
    const uintptr_t o = reinterpret_cast<uintptr_t>(out), i = reinterpret_cast<uintptr_t>(in);
    return out && o < i + static_cast<uintptr_t>(m) * sizeof(T) && i < o + static_cast<uintptr_t>(n) * sizeof(float);
}

template <typename T>
hipError_t launch_modify_typed(const void *target_v, const void *draft_v, const int32_t *tokens, int K, int M,
                               int bonus, int V, int batch, float c, const double *carry, const int32_t *count,
                               float *out_logq, float *out_logp, double *norm_out, int32_t *fallback_out,
                               char *ws, hipStream_t stream)
{
    const T *target = static_cast<const T *>(target_v), *draft = static_cast<const T *>(draft_v);
    const ModLayout lay = mod_layout(batch, K, M, bonus);
    ModStat *tstat = reinterpret_cast<ModStat *>(ws + lay.tstat), *dstat = reinterpret_cast<ModStat *>(ws + lay.dstat);
    double *norm = norm_out ? norm_out : reinterpret_cast<double *>(ws + lay.norm);
    int32_t *fb = fallback_out ? fallback_out : reinterpret_cast<int32_t *>(ws + lay.fb);
    const long long bk = static_cast<long long>(batch) * K;
    const long long n_t = bk * (M + bonus), n_d = bk * M;
    const dim3 blk(kModThreads);
    // Results that replace their inputs (a level applied on top of another one, in its buffers): no row is written before the
    // last kernel, which then has every entry read and written by one thread.  By vectors that holds unless the last one
    // repeats entries of the vector before it, which another thread may have written.
    const bool in_place = overlap(out_logq, n_t * V, target, n_t * V) || overlap(out_logq, n_t * V, draft, n_d * V) ||
                          overlap(out_logp, n_d * V, target, n_t * V) || overlap(out_logp, n_d * V, draft, n_d * V);
    const bool vec = read_by_vectors<T>(V) && !(in_place && V % Elem<T>::kPerVec != 0);
    // rows short enough to stay in a workgroup's registers are read once unless a modification is pending for them
    const bool rows_fit = vec && !in_place && row_vectors<T>(V) <= kRowSlots * kModThreads;
    const bool short_rows = row_vectors<T>(V) <= kShortRowSlots * kModThreads, whole = V % Elem<T>::kPerVec == 0;
    if (rows_fit) {
#define SPECGBV_MOD_ROWS(FORM, SLOTS, PAIR_SLOTS)                                                                    \
    do {                                                                                                             \
        hipLaunchKernelGGL((k_mod_row<T, FORM, SLOTS>), dim3(static_cast<unsigned>(n_t + n_d)), blk, 0, stream, target, \
                           draft, tokens, K, M, bonus, V, c, n_t, count, tstat, dstat, out_logq, out_logp);          \
        hipLaunchKernelGGL((k_mod_pair<T, FORM, PAIR_SLOTS>), dim3(static_cast<unsigned>(n_d)), blk, 0, stream, target, \
                           draft, K, M, bonus, V, c, carry, count, tstat, dstat, norm, fb, out_logq);                \
    } while (0)
        const bool short_pairs = row_vectors<T>(V) <= kShortPairSlots * kModThreads;
        // Rows in halves from two and a quarter vectors per thread on: what a short row takes is its workgroup's instructions, and
        // a half has its own address and bound.  Whole vectors / halves, us a call: 128 x 16 drafts of 8, V = 1024 242 / 279, 6000
        // 351 / 382; 64 x 16 of 8, V = 8200 222 / 223, 10000 254 / 242, 12288 291 / 270, 24000 574 / 513.
        constexpr ModForm kLong = Elem<T>::kPerVec == 8 ? kHalved : kWhole;
        if (whole && row_vectors<T>(V) <= 9 * kModThreads / 4) SPECGBV_MOD_ROWS(kWhole, kShortRowSlots, kShortPairSlots);
        else if (short_pairs && whole) SPECGBV_MOD_ROWS(kLong, kShortRowSlots, kShortPairSlots);
        else if (short_pairs) SPECGBV_MOD_ROWS(kRagged, kShortRowSlots, kShortPairSlots);
        else if (short_rows && whole) SPECGBV_MOD_ROWS(kLong, kShortRowSlots, kPairSlots);
        else if (short_rows) SPECGBV_MOD_ROWS(kRagged, kShortRowSlots, kPairSlots);
        else if (whole) SPECGBV_MOD_ROWS(kLong, kRowSlots, kPairSlots);
        else SPECGBV_MOD_ROWS(kRagged, kRowSlots, kPairSlots);
#undef SPECGBV_MOD_ROWS
        return hipGetLastError();
    }
#define SPECGBV_MOD_LAUNCH(VEC)                                                                                   \
    do {                                                                                                          \
        hipLaunchKernelGGL((k_mod_stats<T, VEC>), dim3(static_cast<unsigned>(n_t + n_d)), blk, 0, stream,          \
                           target, draft, tokens, M, bonus, V, c, n_t, tstat, dstat);                             \
        hipLaunchKernelGGL((k_mod_norm<T, VEC>), dim3(static_cast<unsigned>(n_d)), blk, 0, stream, target, draft,  \
                           K, M, bonus, V, c, carry, count, tstat, dstat, norm, fb);                              \
        hipLaunchKernelGGL((k_mod_write<T, VEC>), dim3(static_cast<unsigned>(n_t)), blk, 0, stream, target, draft, \
                           K, M, bonus, V, c, carry, count, tstat, dstat, norm, fb, out_logq, out_logp);          \
    } while (0)
    if (vec) SPECGBV_MOD_LAUNCH(true);
    else SPECGBV_MOD_LAUNCH(false);
#undef SPECGBV_MOD_LAUNCH
    return hipGetLastError();
}

// ---- advancing a pending modification's block ratio along the tokens an iteration emitted
//
// grid (M, batch).  Workgroup (j, b) handles emitted position j of prefix b: the token is draft
// f's j-th token for j < tau and the final token for j = tau; its log-ratio
// ln q_j[e] - ln p_j[e] under the rows the pending modification modifies goes to delta[b, j].
// Nothing is computed for prefixes whose modification expires with this iteration
// (count <= tau + 1) or that accepted a whole block.
template <typename T, bool VEC>
__global__ void __launch_bounds__(kModThreads)
k_carry_rows(const T *__restrict__ rows_q, const T *__restrict__ rows_p, const int32_t *__restrict__ tokens,
             const int32_t *__restrict__ accepted_len, const int32_t *__restrict__ accepted_idx,
             const int32_t *__restrict__ out_tokens, const int32_t *__restrict__ count, int K, int M, int rows_t,
             int V, float c, double *__restrict__ delta)
{
    __shared__ double sh_d[kModThreads / kWave];
    __shared__ float sh_f[kModThreads / kWave];
    const int j = blockIdx.x, b = blockIdx.y;
    const int tau = accepted_len[b];
    if (tau >= M || j > tau || count[b] <= tau + 1) return;          // uniform over the workgroup
    int f = accepted_idx[b];
    f = f < 0 ? 0 : (f >= K ? K - 1 : f);
    int e = j < tau ? tokens[(static_cast<long long>(b) * K + f) * M + j] : out_tokens[static_cast<long long>(b) * (M + 1) + tau];
    e = e < 0 ? 0 : (e >= V ? V - 1 : e);
    const T *rq = rows_q + ((static_cast<long long>(b) * K + f) * rows_t + j) * static_cast<long long>(V);
    const T *rp = rows_p + ((static_cast<long long>(b) * K + f) * M + j) * static_cast<long long>(V);
    constexpr int PV = Elem<T>::kPerVec;
    RunningSum aq, ap;
    if constexpr (VEC) {
        for_each_pair<T, VEC, kModThreads>(rq, rp, V, [&](int, const float (&zq)[PV], const float (&zp)[PV]) {
            aq.add(zq, c);
            ap.add(zp, c);
        });
    } else {
        for (int x = threadIdx.x; x < V; x += kModThreads) {
            const float zq[1] = {Elem<T>::scalar(rq + x)}, zp[1] = {Elem<T>::scalar(rp + x)};
            aq.add(zq, c); ap.add(zp, c);
        }
    }
    const float Mq = block_max(aq.m2, sh_f);
    const double Zq = block_sum(static_cast<double>(aq.Z * exp2_fast(aq.m2 - Mq)), sh_d);
    const float Mp = block_max(ap.m2, sh_f);
    const double Zp = block_sum(static_cast<double>(ap.Z * exp2_fast(ap.m2 - Mp)), sh_d);
    if (threadIdx.x == 0) {
        const double l2q = static_cast<double>(Elem<T>::scalar(rq + e)) * static_cast<double>(c) - (static_cast<double>(Mq) + log2(Zq));
        const double l2p = static_cast<double>(Elem<T>::scalar(rp + e)) * static_cast<double>(c) - (static_cast<double>(Mp) + log2(Zp));
        delta[static_cast<long long>(b) * M + j] = (l2q - l2p) * 0.693147180559945309417;
    }
}

// one thread per prefix: sums the log-ratios in position order and shortens the row count
__global__ void k_carry_apply(const int32_t *__restrict__ accepted_len, int M, int batch, const double *__restrict__ delta,
                              double *__restrict__ carry, int32_t *__restrict__ count)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= batch) return;
    const int tau = accepted_len[b], n = count[b];
    if (tau < M && n > tau + 1) {
        double a = carry[b];
        for (int j = 0; j <= tau; ++j) a += delta[static_cast<long long>(b) * M + j];
        carry[b] = a;
        count[b] = n - (tau + 1);
    } else {
        count[b] = 0;                                     // expired: its ratio is not used again
    }
}

template <typename T>
hipError_t launch_carry_typed(const void *rows_q, const void *rows_p, const int32_t *tokens, const int32_t *accepted_len,
                              const int32_t *accepted_idx, const int32_t *out_tokens, int K, int M, int bonus, int V,
                              int batch, float c, double *carry, int32_t *count, double *delta, hipStream_t stream)
{
    const bool vec = read_by_vectors<T>(V);
    const dim3 g(static_cast<unsigned>(M), static_cast<unsigned>(batch));
    if (vec)
        hipLaunchKernelGGL((k_carry_rows<T, true>), g, dim3(kModThreads), 0, stream, static_cast<const T *>(rows_q),
                           static_cast<const T *>(rows_p), tokens, accepted_len, accepted_idx, out_tokens, count, K, M,
                           M + bonus, V, c, delta);
    else
        hipLaunchKernelGGL((k_carry_rows<T, false>), g, dim3(kModThreads), 0, stream, static_cast<const T *>(rows_q),
                           static_cast<const T *>(rows_p), tokens, accepted_len, accepted_idx, out_tokens, count, K, M,
                           M + bonus, V, c, delta);
    hipLaunchKernelGGL(k_carry_apply, dim3((batch + 255) / 256), dim3(256), 0, stream, accepted_len, M, batch, delta, carry,
                       count);
    return hipGetLastError();
}

}  // namespace

size_t modify_workspace_bytes(int batch, int K, int M, int bonus) { return mod_layout(batch, K, M, bonus).total; }

hipError_t launch_modify(const void *target, const void *draft, const int32_t *tokens, int K, int M, int bonus, int V,
                         int batch, int dtype, float c, const double *carry, const int32_t *count, float *out_logq,
                         float *out_logp, double *norm_out, int32_t *fallback_out, char *ws, hipStream_t stream)
{
    return dtype == 1 ? launch_modify_typed<uint16_t>(target, draft, tokens, K, M, bonus, V, batch, c, carry, count,
                                                      out_logq, out_logp, norm_out, fallback_out, ws, stream)
                      : launch_modify_typed<float>(target, draft, tokens, K, M, bonus, V, batch, c, carry, count,
                                                   out_logq, out_logp, norm_out, fallback_out, ws, stream);
}

hipError_t launch_carry_advance(const void *rows_q, const void *rows_p, const int32_t *tokens, const int32_t *accepted_len,
                                const int32_t *accepted_idx, const int32_t *out_tokens, int K, int M, int bonus, int V,
                                int batch, int dtype, float c, double *carry, int32_t *count, double *delta,
                                hipStream_t stream)
{
    return dtype == 1 ? launch_carry_typed<uint16_t>(rows_q, rows_p, tokens, accepted_len, accepted_idx, out_tokens, K, M,
                                                     bonus, V, batch, c, carry, count, delta, stream)
                      : launch_carry_typed<float>(rows_q, rows_p, tokens, accepted_len, accepted_idx, out_tokens, K, M,
                                                  bonus, V, batch, c, carry, count, delta, stream);
}

}  // namespace specgbv
