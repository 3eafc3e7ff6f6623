// Draft-side sampling (the drafting step of Algorithm 3): one token per row from
// softmax(logits[row, :] / T) by inverse CDF in token-id order.
//
// One workgroup streams one row.  The row is cut into 512-entry segments (one wave x 8 entries per lane, so lane order
// is token order); wave w takes every kWaves-th segment from w on; each segment's weight sum goes to LDS together with
// the integral reference exponent of the batch of segments it was loaded with, so no row-wide maximum is needed before
// the pass.  Then one wave brings the sums to a common scale, finds the segment in which the running sum first exceeds
// u * total by a scan, re-reads that one segment and finds the entry.  The row is read once (plus one segment); nothing
// is exchanged between workgroups.
//
// What bounds it: a workgroup alone on its compute unit, so the loads in flight and, after the last one has come, the
// chain sum - barrier - scan - segment.  With up to one row per compute unit 16 waves take 16 segments each, so that a
// row of 131072 bfloat16 entries is in flight at once; with more rows two workgroups of 8 waves share a unit.  256 rows of
// 128256 bfloat16 entries: 16.3 us a call (17.9 with 8 waves in two batches and a workgroup-wide search), 2048 rows of 152064
// 116 (150; 5.4 TB/s), 3 rows 10.9 (13.3).
// Rows at odd addresses take the same path (entry by entry before: 24 rows of 32003 14.7, 7.8 now).
#include "specgbv_internal.hpp"

namespace specgbv {
namespace {

constexpr int kSampMaxSeg = 2048;            // V <= 2048 * 512 entries per row

// largest of the logits packed in one 16-byte vector
template <typename T>
__device__ __forceinline__ float vec_max_elem(const U4 &v)
{
    constexpr int PV = Elem<T>::kPerVec;
    float t[PV];
    Elem<T>::unpack(v, t);
    float m = t[0];
#pragma unroll
    for (int j = 1; j < PV; ++j) m = fmaxf(m, t[j]);
    return m;
}

template <typename T, int TH>
__global__ void __launch_bounds__(TH, 4)
k_sample_rows(const T *__restrict__ logits, int V, float c, int nseg, uint64_t seed, uint64_t offset, uint32_t slot,
              int32_t *__restrict__ out_tokens, double *__restrict__ u_out, double *__restrict__ margin_out)
{
    constexpr int kWaves = TH / kWave;
    __shared__ double sh_sum[kSampMaxSeg];
    __shared__ float sh_m2[kSampMaxSeg];
    const int row_id = blockIdx.x, tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wid = __builtin_amdgcn_readfirstlane(tid / kWave);    // (scalar: so are the segments' addresses)
    const T *row = logits + static_cast<long long>(row_id) * V;

    // ---- pass over the row, UN segments of this wave in flight at a time (every slot loads: a load under a branch is
    // waited for where the branch ends; slots beyond the row repeat its last segment)
    constexpr int PV = Elem<T>::kPerVec;
    constexpr int NV = 8 / PV;                              // vectors per lane and segment
    constexpr int UN = 16 / NV;
    for (int s0 = wid; s0 < nseg; s0 += UN * kWaves) {
        SegVec<T> raw[UN];
#pragma unroll
        for (int i = 0; i < UN; ++i) {
            const int s = s0 + i * kWaves < nseg ? s0 + i * kWaves : nseg - 1;
            raw[i] = seg_load(row, s, lane, V);
        }
        // one reference exponent for the whole batch (its largest logit): a wave-wide maximum per batch instead
        // of one per segment.  Entries 2^-126 below it round to weight 0, which they are against the total anyway.
        // (Lanes beyond the row's end hold its last entries: at worst a larger reference, that of an entry of the row.)
        float mb = -3.0e38f;
        if (V >= 8) {
#pragma unroll
            for (int i = 0; i < UN; ++i)
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    mb = fmaxf(mb, vec_max_elem<T>(raw[i].v[v]));
                    // (opaque touch: the floats unpacked for the maximum are not kept for the weights)
                    asm volatile("" : "+v"(raw[i].v[v].x), "+v"(raw[i].v[v].y), "+v"(raw[i].v[v].z), "+v"(raw[i].v[v].w), "+v"(mb));
                }
        }
        if (V < 8)                                          // uniform
            for (int e = 0; e < V; ++e) mb = fmaxf(mb, Elem<T>::scalar(row + e));
        const float m2 = integral_reference(wave_max(mb), c);
#pragma unroll
        for (int i = 0; i < UN; ++i) {
            const int s = s0 + i * kWaves;
            if (s < nseg) {                                 // wave-uniform
                float z[8], w[8];
                seg_unpack(raw[i], row, s, lane, V, -INFINITY, z);
#pragma unroll
                for (int j = 0; j < 8; ++j) w[j] = exp2_fast(fmaf(z[j], c, -m2));
                // 512 weights of at most 2^1 each: float32 sums (8 per lane, then over the wave) are good to a few 1e-7 of
                // the segment, far inside the 1e-6 of the total below which a draw counts as undecided
                const float a = wave_sum_f32(((w[0] + w[1]) + (w[2] + w[3])) + ((w[4] + w[5]) + (w[6] + w[7])));
                if (lane == 0) { sh_sum[s] = static_cast<double>(a); sh_m2[s] = m2; }
            }
        }
    }
    const double u = philox_uniform(seed, offset, static_cast<uint32_t>(row_id), slot);
    __syncthreads();
    if (wid != 0) return;

    // ---- one wave: common scale, total, and the lane whose contiguous segments contain the goal
    const int chunk = (nseg + kWave - 1) / kWave;
    const int s0 = lane * chunk < nseg ? lane * chunk : nseg, s1 = min(nseg, s0 + chunk);
    float mloc = -3.0e38f;
    for (int s = s0; s < s1; ++s) mloc = fmaxf(mloc, sh_m2[s]);
    const float M = wave_max(mloc);
    double mine_seg = 0.0;
    for (int s = s0; s < s1; ++s) mine_seg += ldexp(sh_sum[s], reference_shift(sh_m2[s], M));
    const double incl_t = wave_inclusive_sum(mine_seg);
    const double W = lane_value(incl_t, kWave - 1);
    const double goal = u * W;
    const double excl_t = incl_t - mine_seg;
    const unsigned long long has = __ballot(mine_seg > 0.0);
    const unsigned long long over = __ballot(mine_seg > 0.0 && excl_t + mine_seg > goal);
    const int win_l = over ? __ffsll(static_cast<long long>(over)) - 1
                           : (has ? 63 - __clzll(static_cast<long long>(has)) : 0);     // (rounding pushed the goal past the end)
    int seg_w = 0;
    double cum_w = 0.0;
    if (lane == win_l) {
        double cum = excl_t, cum_before = excl_t, cum_before_last = excl_t;
        int found = -1, last_pos = s0 < nseg ? s0 : 0;
        for (int s = s0; s < s1; ++s) {
            const double v = ldexp(sh_sum[s], reference_shift(sh_m2[s], M));
            if (v > 0.0) { last_pos = s; cum_before_last = cum; }
            if (cum + v > goal) { found = s; cum_before = cum; break; }
            cum += v;
        }
        if (found < 0) { found = last_pos; cum_before = cum_before_last; }
        seg_w = found; cum_w = cum_before;
    }
    const int seg = __builtin_amdgcn_readlane(seg_w, win_l);
    const float seg_m2 = sh_m2[seg];
    const int up = -reference_shift(seg_m2, M);
    const double local_target = ldexp(goal - lane_value(cum_w, win_l), up);        // goal in the segment's own scale
    const double total_here = ldexp(W, up);

    // ---- inside the segment: lane order = token-id order
    float z[8], w[8];
    seg_unpack(seg_load(row, seg, lane, V), row, seg, lane, V, -INFINITY, z);
#pragma unroll
    for (int j = 0; j < 8; ++j) w[j] = exp2_fast(fmaf(z[j], c, -seg_m2));
    double mine = 0.0;
#pragma unroll
    for (int j = 0; j < 8; ++j) mine += static_cast<double>(w[j]);
    const double incl = wave_inclusive_sum(mine);
    const double excl = incl - mine;
    const unsigned long long cross = __ballot(mine > 0.0 && incl > local_target);
    const unsigned long long pos = __ballot(mine > 0.0);
    int winner;
    if (cross) winner = __ffsll(static_cast<long long>(cross)) - 1;
    else if (pos) winner = 63 - __clzll(static_cast<long long>(pos));
    else winner = 0;
    if (lane == winner) {
        double run = excl, mg = 0.0;
        int y = -1, last = -1;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const double prev = run;
            run += static_cast<double>(w[j]);
            if (w[j] > 0.0f) last = j;
            if (y < 0 && run > local_target) {
                y = j;
                const double lo = local_target - prev, hi = run - local_target;
                mg = (lo < hi ? lo : hi) / total_here;
            }
        }
        if (y < 0) { y = last < 0 ? 0 : last; mg = 0.0; }
        long long tokid = static_cast<long long>(seg) * kSegElems + lane * 8 + y;
        if (tokid >= V) tokid = V - 1;
        out_tokens[row_id] = static_cast<int32_t>(tokid);
        u_out[row_id] = u;
        margin_out[row_id] = mg;
    }
}

template <typename T>
hipError_t launch_sample_typed(const void *logits, int rows, int V, float c, uint64_t seed, uint64_t offset,
                               uint32_t slot, int32_t *out_tokens, double *u_out, double *margin_out, hipStream_t stream)
{
    const int nseg = (V + kSegElems - 1) / kSegElems;
#define SPECGBV_SAMPLE_LAUNCH(TH)                                                                                      \
    hipLaunchKernelGGL((k_sample_rows<T, TH>), dim3(rows), dim3(TH), 0, stream, static_cast<const T *>(logits), V, c, nseg, \
                       seed, offset, slot, out_tokens, u_out, margin_out)
    if (rows <= compute_units() && nseg > 64) SPECGBV_SAMPLE_LAUNCH(1024);
    else SPECGBV_SAMPLE_LAUNCH(512);
#undef SPECGBV_SAMPLE_LAUNCH
    return hipGetLastError();
}

}  // namespace

int sample_max_vocab() { return kSampMaxSeg * kSegElems; }

hipError_t launch_sample_rows(const void *logits, int rows, int V, int dtype, float c, uint64_t seed, uint64_t offset,
                              uint32_t slot, int32_t *out_tokens, double *u_out, double *margin_out, hipStream_t stream)
{
    return dtype == 1 ? launch_sample_typed<uint16_t>(logits, rows, V, c, seed, offset, slot, out_tokens, u_out, margin_out, stream)
                      : launch_sample_typed<float>(logits, rows, V, c, seed, offset, slot, out_tokens, u_out, margin_out, stream);
}

}  // namespace specgbv
