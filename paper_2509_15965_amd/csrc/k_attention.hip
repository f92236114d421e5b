// k_attention.hip -- grouped-query attention over the per-sequence KV cache.
//
// bf16 path (split-KV, MFMA).  One wave owns one work item: up to 16 query
// columns (query tokens x the q-heads of one kv-head) against one chunk of
// key positions of one KV slot.  Every K and V byte of the chunk is read
// once for all q-heads of the group.  A pair item serves the single decode
// tokens of two sequences that read the same shared prompt chunk (2 x group
// columns), so that chunk is read once for both.
//   scores   S^T[t][c] = K[t] . Q[c]     (A = 16 key rows, B = 16 columns)
//   output   O^T[d][c] += V^T[d][t] P^T[t][c]
// Key rows of the two 16-row score tiles of a 32-position step are permuted
// so that the lane holding column c and k-group q owns the scores of
// positions t0 + 8q .. t0 + 8q + 7; those eight probabilities are exactly
// the lane's B operand of the P.V product, and the matching A operand is one
// 16-byte load from the V cache's 8-position blocks.  No LDS, no transposes.
// Online softmax in the exp2 domain, fp32 state; the hardware's exp2 returns 0
// below 2^-126, where a weight is nothing beside the row's largest (1); the
// probabilities enter the P.V MFMA as a bf16 hi/lo pair, so they are not
// rounded to bf16.  A work
// item that covers all keys of its tokens writes the normalised output;
// otherwise it writes (max, sum, unnormalised output) partials that
// attn_combine merges in item order.  (Merging in the last-arriving wave
// would need device-scope fences, which on this multi-XCD part write back and
// invalidate the whole L2 and slow every co-running wave.)
//
// fp32 path: one workgroup per (row, q-head), plain VALU (tiny model only).
#include <hip/hip_ext.h>

#include "rl_device.h"
#include "rl_internal.h"

#include <type_traits>

namespace rl {

// Zero the bf16 elements e >= nvalid of an 8-element vector (0 <= nvalid <= 8).
__device__ __forceinline__ u32x4 mask_tail8(u32x4 v, int nvalid) {
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const int e0 = 2 * w;
        uint32_t keep = (e0 < nvalid ? 0x0000FFFFu : 0u) | (e0 + 1 < nvalid ? 0xFFFF0000u : 0u);
        v[w] &= keep;
    }
    return v;
}

// Two floats as bf16 (round to nearest even) in one word, the first in the low half.
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
}

// Probabilities of one 32-position step for a lane's column, as P.V operands.
struct StepProbs {
    u32x4 hi, lo;   // bf16 pair: hi = rne(p), lo = rne(p - hi)
    float alpha;    // rescale of the running sum and output
};

// First half of a 32-position step of the online-softmax attention of a wave's
// 16 query columns: scores of positions t0..t0+31 from the K rows (k0: tile 0,
// k1: tile 1), positions past min(hi - 1, limit) masked (full: none is, for
// any lane), running max and sum updated.  after_qk runs once the K registers
// are consumed, so that the caller can refill them under the softmax.
template <int D, typename AfterQk>
__device__ __forceinline__ StepProbs attn_scores(const u32x4 (&k0)[D / 32], const u32x4 (&k1)[D / 32],
                                                 const u32x4 (&qf)[D / 32], int t0, int hi, int limit, bool full,
                                                 int kq, float scale_log2, float& m, float& l, AfterQk after_qk) {
    constexpr int KG = D / 32;
    const int pb = t0 + 8 * kq;
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < KG; ++j) {
        s0 = mfma16x16x32(as_bf16x8(k0[j]), as_bf16x8(qf[j]), s0);
        s1 = mfma16x16x32(as_bf16x8(k1[j]), as_bf16x8(qf[j]), s1);
    }
    after_qk();
    // this lane now holds the scores of its column at positions pb + 0..7
    float sv[8];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        sv[e] = s0[e] * scale_log2;
        sv[4 + e] = s1[e] * scale_log2;
    }
    if (!full) {
        const int lim = min(hi - 1, limit);
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (pb + e > lim) sv[e] = -INFINITY;
    }
    float mx = sv[0];
#pragma unroll
    for (int e = 1; e < 8; ++e) mx = fmaxf(mx, sv[e]);
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float m_new = fmaxf(m, mx);
    const float m_use = m_new == -INFINITY ? 0.0f : m_new;
    StepProbs r;
    r.alpha = __builtin_amdgcn_exp2f(m - m_use);
    // the P.V product carries ~16 significant bits of p (hi + lo), so the only
    // storage rounding left is the one of the attention output
    float psum = 0.0f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const float p0 = __builtin_amdgcn_exp2f(sv[2 * w] - m_use);
        const float p1 = __builtin_amdgcn_exp2f(sv[2 * w + 1] - m_use);
        psum += p0 + p1;
        const uint32_t h = pack_bf16(p0, p1);
        r.hi[w] = h;
        r.lo[w] = pack_bf16(p0 - __uint_as_float(h << 16), p1 - __uint_as_float(h & 0xFFFF0000u));
    }
    l = l * r.alpha + psum;
    m = m_new;
    return r;
}

// Second half: the output rescaled and updated with the V blocks vf
// (positions >= hi zeroed unless full).
template <int D>
__device__ __forceinline__ void attn_pv(const u32x4 (&vf)[D / 16], const StepProbs& p, int t0, int hi, bool full,
                                        int kq, f32x4 (&o)[D / 16]) {
    constexpr int DT = D / 16;
    const int nvalid = hi - (t0 + 8 * kq);   // keys past the chunk end carry no data
#pragma unroll
    for (int i = 0; i < DT; ++i) {
        u32x4 v = vf[i];
        if (!full && nvalid < 8) v = mask_tail8(v, nvalid < 0 ? 0 : nvalid);
        o[i] = o[i] * p.alpha;
        o[i] = mfma16x16x32(as_bf16x8(v), as_bf16x8(p.hi), o[i]);
        o[i] = mfma16x16x32(as_bf16x8(v), as_bf16x8(p.lo), o[i]);
    }
}

template <int D>
__device__ __forceinline__ void attn_step(const u32x4 (&k0)[D / 32], const u32x4 (&k1)[D / 32],
                                          const u32x4 (&vf)[D / 16], const u32x4 (&qf)[D / 32], int t0, int hi,
                                          int limit, bool full, int kq, float scale_log2, float& m, float& l,
                                          f32x4 (&o)[D / 16]) {
    const StepProbs p = attn_scores<D>(k0, k1, qf, t0, hi, limit, full, kq, scale_log2, m, l, [] {});
    attn_pv<D>(vf, p, t0, hi, full, kq, o);
}

// 16-byte chunk permutation of K row r (of a 32-position step) in LDS:
// logical chunk c sits at c ^ kswz(r), which makes the fragment reads of one
// 16-lane group hit 16 different 16-byte bank groups.
template <int D>
__device__ __forceinline__ int kswz(int r) {
    return D == 128 ? ((r & 3) | ((r >> 1) & 12)) : (((r >> 1) & 1) | ((r >> 2) & 6));
}

// The same for the 32-row fragment reads of the prefill kernel, whose lane
// groups read 16 consecutive positions.
template <int D>
__device__ __forceinline__ int kswz32(int r) {
    return D == 128 ? (r & 15) : ((r >> 1) & 7);
}

__device__ __forceinline__ void lds_dma16(const void* g, uint8_t* lds_wave_base) {
    __builtin_amdgcn_global_load_lds(g, (__attribute__((address_space(3))) void*)(lds_wave_base), 16, 0, 0);
}

// The K rows and V blocks of positions t0..t0+31 of one (slot, kv-head) into
// an LDS step buffer (K [32][D] chunk-permuted, V [4][D][8]), spread over the
// kWaves waves of the workgroup: wave w moves KB w, w + kWaves, ... of each
// (waves past the step's KB count move none).  One global_load_lds per KB per
// lane.
template <int D, int kWaves, bool kRows32 = false>
__device__ __forceinline__ void step_dma(const uint16_t* kb, const uint16_t* vb, int t0, int wave, int lane,
                                         uint8_t* kl, uint8_t* vl) {
    constexpr int STEPB = 32 * D * 2;
    constexpr int NKB = STEPB / 1024;     // KB of K (and of V) per step
    constexpr int RPK = 1024 / (D * 2);   // K rows per KB
    constexpr int CPR = D / 8;            // 16-byte chunks per row
#pragma unroll
    for (int j = 0; j < (NKB + kWaves - 1) / kWaves; ++j) {
        const int kb_ = wave + kWaves * j;
        if (kb_ >= NKB) break;
        const int r = kb_ * RPK + lane / CPR;
        const int c = (lane % CPR) ^ (kRows32 ? kswz32<D>(r) : kswz<D>(r));
        lds_dma16(kb + static_cast<size_t>(t0 + r) * D + 8 * c, kl + kb_ * 1024);
        lds_dma16(reinterpret_cast<const uint8_t*>(vb + static_cast<size_t>(t0) * D) + kb_ * 1024 + lane * 16,
                  vl + kb_ * 1024);
    }
}

// A wave's K / V fragments of one step from an LDS step buffer.
template <int D>
__device__ __forceinline__ void step_frags(const uint8_t* kl, const uint8_t* vl, int krow, int kq, int col,
                                           u32x4 (&k0)[D / 32], u32x4 (&k1)[D / 32], u32x4 (&vf)[D / 16]) {
#pragma unroll
    for (int j = 0; j < D / 32; ++j) {
        const int c = kq + 4 * j;
        k0[j] = *reinterpret_cast<const u32x4*>(kl + krow * (2 * D) + 16 * (c ^ kswz<D>(krow)));
        k1[j] = *reinterpret_cast<const u32x4*>(kl + (krow + 4) * (2 * D) + 16 * (c ^ kswz<D>(krow + 4)));
    }
#pragma unroll
    for (int i = 0; i < D / 16; ++i) vf[i] = *reinterpret_cast<const u32x4*>(vl + (kq * D + col + 16 * i) * 16);
}

// vmcnt(0) with expcnt and lgkmcnt left alone (gfx9 encoding)
__device__ __forceinline__ void wait_vm0() { __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8)); }

// PAGED: the item's key range may cross pages, so each 32-position step
// looks its page up; otherwise the slot's block is fixed for the item.
template <int D, bool PAGED>
__global__ void __launch_bounds__(256, 2) attn_bf16_kernel(const AttnItem* __restrict__ items,
        const int32_t* __restrict__ wave_first, int n_waves, const uint16_t* __restrict__ q,
        const uint16_t* __restrict__ kc, const uint16_t* __restrict__ vc, KvPages kp, int Hq, int Hkv, int layer,
        float scale_log2, uint16_t* __restrict__ out, float* __restrict__ part) {
    constexpr int KG = D / 32;   // 32-wide k groups of a head
    constexpr int DT = D / 16;   // 16-wide d tiles of the output
    constexpr int STEPB = 32 * D * 2;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[2][2][STEPB];   // [buffer][K | V], shared-chunk units
    // the wave index as a scalar: the item, its addresses and its page table
    // reads then are scalar too
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wid = blockIdx.x * 4 + wave;
    if (wid >= n_waves) return;
    const int kvh = blockIdx.y;
    const int G = Hq / Hkv;
    // the wave's items: consecutive ones up to the next wave's first, or the
    // wave's own number without a list
    const int first = wave_first ? wave_first[wid] : wid, last = wave_first ? wave_first[wid + 1] : wid + 1;
    // a unit of four items over one shared prompt chunk (same slot and key
    // range; the host flags its first item): every K/V step goes through LDS
    // once for the four waves
    const bool wg_lds = !wave_first && blockIdx.x * 4 + 3 < n_waves && (items[blockIdx.x * 4].flags & kAttnLds) != 0;
    for (int item_id = first; item_id < last; ++item_id) {
        const AttnItem it = items[item_id];

        const int col = lane & 15, kq = lane >> 4;
        const int ncols = it.nq * G;
        const bool cvalid = col < ncols;
        const int tau = cvalid ? col / G : 0;
        const int head = kvh * G + (cvalid ? col - tau * G : 0);
        const bool second = it.qrow_b >= 0 && tau == 1;   // second sequence of a pair item
        const int qrow = second ? it.qrow_b : it.qrow + tau;
        const int limit = cvalid ? it.pos0 + tau : -1;   // last key this column sees

        const u32x4 zero = {0u, 0u, 0u, 0u};
        u32x4 qf[KG];
        {
            const uint16_t* qp = q + (static_cast<size_t>(qrow) * Hq + head) * D + 8 * kq;
#pragma unroll
            for (int j = 0; j < KG; ++j) qf[j] = cvalid ? ld16(qp + 32 * j) : zero;
        }

        // The K / V block of the current step and the step's position inside it.
        // Steps ascend 32 positions at a time and pages are multiples of 32, so a
        // paged item enters its pages in order; each table entry is read one page
        // ahead.
        size_t base = 0;
        int lt = it.kv_lo, page_j = 0, next_pid = 0;
        if (!PAGED) {
            base = kv_block(kp, layer, Hkv, it.slot, kvh);
        } else {
            page_j = it.kv_lo / kp.page;
            lt = it.kv_lo - page_j * kp.page;
            if (page_j < kp.maxp) base = kv_block(kp, layer, Hkv, kv_clamp(kp, kv_table(kp, it.slot, page_j)), kvh);
            if (page_j + 1 < kp.maxp) next_pid = kv_table(kp, it.slot, page_j + 1);
        }
        auto advance = [&] {
            lt += 32;
            if (PAGED && lt == kp.page) {
                lt = 0;
                ++page_j;
                base = kv_block(kp, layer, Hkv, kv_clamp(kp, next_pid), kvh);
                next_pid = page_j + 1 < kp.maxp ? kv_table(kp, it.slot, page_j + 1) : 0;
            }
        };

        float m = -INFINITY, l = 0.0f;
        f32x4 o[DT];
#pragma unroll
        for (int i = 0; i < DT; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};

        const int hi = it.kv_hi;
        // a step before this position masks no key of any valid column (columns
        // without a query are never stored)
        const int full_end = min(hi, it.pos0 + 1);
        // key row r of score tile 0 is position t0 + 8(r/4) + r%4; tile 1 adds 4
        const int krow = 8 * (col >> 2) + (col & 3);
        const uint32_t koff = krow * D + 8 * kq, voff = (kq * D + col) * 8;   // this lane's element in a step
        u32x4 k0[KG], k1[KG], vf[DT];
        if (wg_lds) {
            const int nsteps = (hi - it.kv_lo + 31) / 32;
            if (nsteps > 0) step_dma<D, 4>(kc + base, vc + base, lt, wave, lane, lds[0][0], lds[0][1]);
            for (int s = 0; s < nsteps; ++s) {
                wait_vm0();        // this wave's DMAs (and q loads) landed
                __syncthreads();   // every wave's part of step s is in LDS; step s-1 retired
                if (s + 1 < nsteps) {
                    advance();
                    step_dma<D, 4>(kc + base, vc + base, lt, wave, lane, lds[(s + 1) & 1][0], lds[(s + 1) & 1][1]);
                }
                const int t0 = it.kv_lo + 32 * s;
                step_frags<D>(lds[s & 1][0], lds[s & 1][1], krow, kq, col, k0, k1, vf);
                attn_step<D>(k0, k1, vf, qf, t0, hi, limit, t0 + 32 <= full_end, kq, scale_log2, m, l, o);
            }
        } else if (hi > it.kv_lo) {
            // K and V registers are refilled for the next step as soon as this
            // one has consumed them, so a wave always has loads in flight under
            // its math, in the same registers.  Keys that this item alone reads
            // carry the non-temporal hint: streaming them through the memory-side
            // cache evicts the activations and partial sums written there, which
            // then cross HBM twice.
            auto run = [&](auto once) {
                constexpr bool NT = decltype(once)::value;
                auto ld = [](const uint16_t* q_) { return NT ? ld16_nt(q_) : ld16(q_); };
                auto load_k = [&] {
                    const uint16_t* kb = kc + base + static_cast<size_t>(lt) * D;
#pragma unroll
                    for (int j = 0; j < KG; ++j) {
                        k0[j] = ld(kb + koff + 32 * j);
                        k1[j] = ld(kb + koff + 4 * D + 32 * j);
                    }
                };
                auto load_v = [&] {
                    const uint16_t* vb = vc + base + static_cast<size_t>(lt) * D;
#pragma unroll
                    for (int i = 0; i < DT; ++i) vf[i] = ld(vb + voff + 128 * i);
                };
                load_k();
                load_v();
                for (int t0 = it.kv_lo; t0 < hi; t0 += 32) {
                    const bool more = t0 + 32 < hi, full = t0 + 32 <= full_end;
                    const StepProbs p = attn_scores<D>(k0, k1, qf, t0, hi, limit, full, kq, scale_log2, m, l, [&] {
                        if (more) {
                            advance();
                            load_k();
                        }
                    });
                    attn_pv<D>(vf, p, t0, hi, full, kq, o);
                    if (more) load_v();
                }
            };
            if (it.flags & kAttnOnce) run(std::true_type{});
            else run(std::false_type{});
        }
        l += __shfl_xor(l, 16, 64);
        l += __shfl_xor(l, 32, 64);

        // lane holds O^T[d = 16 i + 4 kq + e][col]
        if (it.part < 0) {
            if (!cvalid) continue;
            const float inv = 1.0f / l;
            uint16_t* op = out + (static_cast<size_t>(qrow) * Hq + head) * D + 4 * kq;
#pragma unroll
            for (int i = 0; i < DT; ++i) {
                const uint32_t w0 = static_cast<uint32_t>(f32_to_bf16(o[i][0] * inv)) |
                                    (static_cast<uint32_t>(f32_to_bf16(o[i][1] * inv)) << 16);
                const uint32_t w1 = static_cast<uint32_t>(f32_to_bf16(o[i][2] * inv)) |
                                    (static_cast<uint32_t>(f32_to_bf16(o[i][3] * inv)) << 16);
                *reinterpret_cast<uint2*>(op + 16 * i) = make_uint2(w0, w1);
            }
            continue;
        }
        // split block: (unnormalised o, then m and l) partials, merged by attn_combine
        if (!cvalid) continue;
        // a pair item's second sequence owns its own partial slot (columns from 0)
        const int pidx = second ? it.part_b : it.part;
        const int pcol = second ? col - G : col;
        float* pb = part + (static_cast<size_t>(pidx) * Hkv + kvh) * 16 * (D + 2);
#pragma unroll
        for (int i = 0; i < DT; ++i) *reinterpret_cast<f32x4*>(pb + pcol * D + 16 * i + 4 * kq) = o[i];
        if (kq == 0) *reinterpret_cast<float2*>(pb + 16 * D + 2 * pcol) = make_float2(m, l);
    }
}

hipError_t launch_attention_bf16(const AttnItem* items, const int32_t* wave_first, int n_waves, const void* q,
                                 const void* kc, const void* vc, const KvPages& kp, int Hq, int Hkv,
                                 int D, int layer, void* out, float* part,
                                 hipStream_t s, hipEvent_t ev_start, hipEvent_t ev_stop) {
    if (n_waves <= 0) return hipSuccess;
    const float scale_log2 = 1.4426950408889634f / sqrtf(static_cast<float>(D));
    dim3 grid((n_waves + 3) / 4, Hkv), block(256);
    auto go = [&](auto kern) {
        if (ev_start || ev_stop)
            hipExtLaunchKernelGGL(kern, grid, block, 0, s, ev_start, ev_stop, 0, items, wave_first, n_waves,
                                  static_cast<const uint16_t*>(q), static_cast<const uint16_t*>(kc),
                                  static_cast<const uint16_t*>(vc), kp, Hq, Hkv, layer, scale_log2,
                                  static_cast<uint16_t*>(out), part);
        else
            hipLaunchKernelGGL(kern, grid, block, 0, s, items, wave_first, n_waves, static_cast<const uint16_t*>(q),
                               static_cast<const uint16_t*>(kc), static_cast<const uint16_t*>(vc), kp, Hq,
                               Hkv, layer, scale_log2, static_cast<uint16_t*>(out), part);
    };
    if (kp.table) {
        if (D == 128) go(attn_bf16_kernel<128, true>); else go(attn_bf16_kernel<64, true>);
    } else {
        if (D == 128) go(attn_bf16_kernel<128, false>); else go(attn_bf16_kernel<64, false>);
    }
    return hipGetLastError();
}


// ---------------------------------------------------------------------------
// Prefill / scoring attention: a workgroup of WAVES waves shares each
// K/V step through LDS, each wave with its own kPrefillCols query columns
// (tokens x the q-heads of one kv-head).  Per 32-position step the workgroup
// DMAs the step's K rows ([32][D], 16-byte chunks permuted by row so that the
// fragment reads are free of bank conflicts) and its four V blocks
// ([4][D][8], contiguous in the cache) into one of two LDS buffers with
// global_load_lds, the next step's right after the barrier that retires the
// previous one.  32x32x16 MFMAs: a wave's fragment reads (16 KB a step at D =
// 128) then serve 32 columns; with 16 columns and 16x16x32 MFMAs those reads
// bound the kernel (20.8k rows of one 7B group, 640 + 16 x 1100 tokens: 1748 ->
// 1057 us a layer).  K rows are read in the order that leaves each lane with
// the scores of the eight consecutive positions its P.V operand takes: output
// row 8q + 4h + i of the score tile is position 16(q/2) + 8h + 4(q%2) + i.
// ---------------------------------------------------------------------------
constexpr int kPrefillCols = 32;

template <int D, int WAVES>
__global__ void __launch_bounds__(64 * WAVES) attn_prefill_kernel(const PrefillTile* __restrict__ tiles,
        const uint16_t* __restrict__ q, const uint16_t* __restrict__ kc, const uint16_t* __restrict__ vc,
        KvPages kp, int Hq, int Hkv, int layer, float scale_log2, uint16_t* __restrict__ out) {
    constexpr int KS = D / 16, DT = D / 32;
    constexpr int STEPB = 32 * D * 2;               // bytes of K (and of V) per 32-position step
    static_assert(STEPB % 1024 == 0, "whole 1 KB DMA instructions per step");
    __shared__ __attribute__((aligned(1024))) uint8_t lds[2][2][STEPB];   // [buffer][K | V]

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kvh = blockIdx.y;
    const int G = Hq / Hkv;
    const int tq = kPrefillCols / G;
    const PrefillTile tl = tiles[blockIdx.x];
    const int tok0 = wave * tq;
    const int nq = max(0, min(tq, tl.ntok - tok0));
    const int col = lane & 31, kh = lane >> 5;
    const bool cvalid = col < nq * G;
    const int tau = cvalid ? col / G : 0;
    const int head = kvh * G + (cvalid ? col - tau * G : 0);
    const int qrow = cvalid ? tl.qrow0 + tok0 + tau : tl.qrow0;
    const int limit = cvalid ? tl.pos0 + tok0 + tau : -1;
    const int hi = tl.pos0 + tl.ntok;               // keys [0, hi)
    const int wave_last = tl.pos0 + tok0 + nq - 1;  // last key any column of this wave sees
    const int full_end = min(hi, tl.pos0 + tok0 + 1);   // steps that end here mask nothing
    const int nsteps = (hi + 31) / 32;

    // the K/V of the step at position t0: its page's blocks and t0 inside the page
    auto dma_step = [&](int t0, int buf) {
        int lt;
        const size_t b = kv_block(kp, layer, Hkv, kv_page(kp, tl.slot, t0, &lt), kvh);
        step_dma<D, WAVES, true>(kc + b, vc + b, lt, wave, lane, lds[buf][0], lds[buf][1]);
    };

    const u32x4 zero = {0u, 0u, 0u, 0u};
    u32x4 qf[KS];
    {
        const uint16_t* qp = q + (static_cast<size_t>(qrow) * Hq + head) * D + 8 * kh;
#pragma unroll
        for (int j = 0; j < KS; ++j) qf[j] = cvalid ? ld16(qp + 16 * j) : zero;
    }
    float m = -INFINITY, l = 0.0f;
    f32x16 o[DT];
#pragma unroll
    for (int i = 0; i < DT; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[i][e] = 0.f;
    // the position in the step that this lane's K row holds, and its LDS bytes
    const int kpos = 16 * (col >> 4) + 8 * ((col >> 2) & 1) + 4 * ((col >> 3) & 1) + (col & 3);
    const int krow = kpos * (2 * D), kx = kswz32<D>(kpos);

    if (nsteps > 0) dma_step(0, 0);
    for (int s = 0; s < nsteps; ++s) {
        wait_vm0();        // this wave's DMAs (and q loads) landed
        __syncthreads();   // every wave's part of step s is in LDS; step s-1 retired
        if (s + 1 < nsteps) dma_step(32 * (s + 1), (s + 1) & 1);
        const int t0 = 32 * s;
        if (nq == 0 || t0 > wave_last) continue;       // wave-uniform: nothing of this step is visible
        const uint8_t *kl = lds[s & 1][0], *vl = lds[s & 1][1];
        f32x16 sc;
#pragma unroll
        for (int e = 0; e < 16; ++e) sc[e] = 0.f;
#pragma unroll
        for (int j = 0; j < KS; ++j) {
            const u32x4 kf = *reinterpret_cast<const u32x4*>(kl + krow + 16 * ((2 * j + kh) ^ kx));
            sc = mfma32x32x16(as_bf16x8(kf), as_bf16x8(qf[j]), sc);
        }
        // this lane holds the scores of its column at positions t0 + 16(e/8) + 8 kh + e%8
        const bool full = t0 + 32 <= full_end;
#pragma unroll
        for (int e = 0; e < 16; ++e) sc[e] *= scale_log2;
        if (!full) {
            const int lim = min(hi - 1, limit) - t0 - 8 * kh;
#pragma unroll
            for (int e = 0; e < 16; ++e)
                if (16 * (e >> 3) + (e & 7) > lim) sc[e] = -INFINITY;
        }
        float mx = sc[0];
#pragma unroll
        for (int e = 1; e < 16; ++e) mx = fmaxf(mx, sc[e]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float m_new = fmaxf(m, mx);
        const float m_use = m_new == -INFINITY ? 0.0f : m_new;
        const float alpha = __builtin_amdgcn_exp2f(m - m_use);
        // probabilities as a bf16 pair hi + lo (~16 significant bits)
        float psum = 0.0f;
        u32x4 ph[2], pl[2];
#pragma unroll
        for (int w = 0; w < 8; ++w) {
            const float p0 = __builtin_amdgcn_exp2f(sc[2 * w] - m_use);
            const float p1 = __builtin_amdgcn_exp2f(sc[2 * w + 1] - m_use);
            psum += p0 + p1;
            const uint32_t h = pack_bf16(p0, p1);
            ph[w >> 2][w & 3] = h;
            pl[w >> 2][w & 3] = pack_bf16(p0 - __uint_as_float(h << 16), p1 - __uint_as_float(h & 0xFFFF0000u));
        }
        l = l * alpha + psum;
        m = m_new;
        if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {   // a new maximum: rare after the first steps
#pragma unroll
            for (int i = 0; i < DT; ++i) o[i] = o[i] * alpha;
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int nvalid = hi - (t0 + 16 * c + 8 * kh);   // keys past the end carry no data
#pragma unroll
            for (int i = 0; i < DT; ++i) {
                u32x4 v = *reinterpret_cast<const u32x4*>(vl + ((2 * c + kh) * D + 32 * i + col) * 16);
                if (!full && nvalid < 8) v = mask_tail8(v, nvalid < 0 ? 0 : nvalid);
                o[i] = mfma32x32x16(as_bf16x8(v), as_bf16x8(ph[c]), o[i]);
                o[i] = mfma32x32x16(as_bf16x8(v), as_bf16x8(pl[c]), o[i]);
            }
        }
    }
    l += __shfl_xor(l, 32, 64);
    if (!cvalid) return;
    const float inv = 1.0f / l;
    uint16_t* op = out + (static_cast<size_t>(qrow) * Hq + head) * D + 4 * kh;
    // lane holds O^T[d = 32 i + 8 w + 4 kh + e][col]
#pragma unroll
    for (int i = 0; i < DT; ++i)
#pragma unroll
        for (int w = 0; w < 4; ++w)
            *reinterpret_cast<uint2*>(op + 32 * i + 8 * w) =
                make_uint2(pack_bf16(o[i][4 * w] * inv, o[i][4 * w + 1] * inv),
                           pack_bf16(o[i][4 * w + 2] * inv, o[i][4 * w + 3] * inv));
}

hipError_t launch_attention_prefill(const PrefillTile* tiles, int n_tiles, int waves, const void* q, const void* kc,
                                    const void* vc, const KvPages& kp, int Hq, int Hkv, int D, int layer,
                                    void* out, hipStream_t s) {
    if (n_tiles <= 0) return hipSuccess;
    const float scale_log2 = 1.4426950408889634f / sqrtf(static_cast<float>(D));
    const dim3 grid(n_tiles, Hkv), block(64 * waves);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, block, 0, s, tiles, static_cast<const uint16_t*>(q),
                           static_cast<const uint16_t*>(kc), static_cast<const uint16_t*>(vc), kp, Hq, Hkv,
                           layer, scale_log2, static_cast<uint16_t*>(out));
    };
    if (waves == 4) {
        if (D == 128) go(attn_prefill_kernel<128, 4>); else go(attn_prefill_kernel<64, 4>);
    } else if (waves == 8) {
        if (D == 128) go(attn_prefill_kernel<128, 8>); else go(attn_prefill_kernel<64, 8>);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Merge the split partials of one query block and kv-head: one workgroup per
// (split block, kv-head), one thread per four output dimensions of a q-head,
// the block's tokens in turn.  Partials are taken eight at a time, in item
// order, with every load of the eight in flight at once; weights 2^(m_j - M).
// Latency bound (two round trips up to eight partials).
template <int D>
__global__ void __launch_bounds__(16 * D / 4) attn_combine_kernel(const int32_t* __restrict__ blocks,
        const AttnItem* __restrict__ items, const float* __restrict__ part, int Hq, int Hkv,
        uint16_t* __restrict__ out) {
    const AttnItem it = items[blocks[blockIdx.x]];
    const int kvh = blockIdx.y, G = Hq / Hkv;
    const int g = threadIdx.x / (D / 4), d4 = threadIdx.x % (D / 4);
    if (g >= G) return;
    const int np = it.nparts;
    const size_t pstride = static_cast<size_t>(Hkv) * 16 * (D + 2);
    const float* pb = part + (static_cast<size_t>(it.part0) * Hkv + kvh) * 16 * (D + 2);
    for (int t = 0; t < it.nq; ++t) {
        const int c = t * G + g;
        const float* po = pb + c * D + 4 * d4;
        const float* pm = pb + 16 * D + 2 * c;
        float M = -INFINITY, L = 0.0f;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        for (int j = 0; j < np; j += 8) {
            float2 ml[8];
            f32x4 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const bool in = j + u < np;
                ml[u] = in ? *reinterpret_cast<const float2*>(pm + (j + u) * pstride) : make_float2(-INFINITY, 0.f);
                v[u] = in ? *reinterpret_cast<const f32x4*>(po + (j + u) * pstride) : f32x4{0.f, 0.f, 0.f, 0.f};
            }
            float Mn = M;
#pragma unroll
            for (int u = 0; u < 8; ++u) Mn = fmaxf(Mn, ml[u].x);
            const float Mu = Mn == -INFINITY ? 0.0f : Mn;
            const float al = exp2f(M - Mu);
            L *= al;
            acc = acc * al;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const float w = exp2f(ml[u].x - Mu);
                L += w * ml[u].y;
                acc += v[u] * w;
            }
            M = Mn;
        }
        const float inv = 1.0f / L;
        *reinterpret_cast<uint2*>(out + (static_cast<size_t>(it.qrow + t) * Hq + kvh * G + g) * D + 4 * d4) =
            make_uint2(pack_bf16(acc[0] * inv, acc[1] * inv), pack_bf16(acc[2] * inv, acc[3] * inv));
    }
}

hipError_t launch_attn_combine(const int32_t* blocks, int n_blocks, const AttnItem* items, const float* part,
                               int Hq, int Hkv, int D, void* out, hipStream_t s) {
    if (n_blocks <= 0) return hipSuccess;
    const int threads = (Hq / Hkv * (D / 4) + 63) / 64 * 64;
    dim3 grid(n_blocks, Hkv), block(threads);
    if (D == 128)
        hipLaunchKernelGGL(attn_combine_kernel<128>, grid, block, 0, s, blocks, items, part, Hq, Hkv,
                           static_cast<uint16_t*>(out));
    else
        hipLaunchKernelGGL(attn_combine_kernel<64>, grid, block, 0, s, blocks, items, part, Hq, Hkv,
                           static_cast<uint16_t*>(out));
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// fp32: one 64-lane workgroup per (row, q-head); keys 0..pos of the row's slot.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(64) attn_f32_kernel(const int32_t* __restrict__ row_slot,
        const int32_t* __restrict__ row_pos, const float* __restrict__ q,
        const float* __restrict__ kc, const float* __restrict__ vc, KvPages kp, int Hq, int Hkv, int D,
        int layer, float* __restrict__ out) {
    __shared__ float qs[128];
    __shared__ float ps[64];
    const int r = blockIdx.x, h = blockIdx.y, lane = threadIdx.x;
    const int G = Hq / Hkv, kvh = h / G;
    const int pos = row_pos[r], slot = row_slot[r];
    const float* qr = q + (static_cast<size_t>(r) * Hq + h) * D;
    for (int i = lane; i < D; i += 64) qs[i] = qr[i];
    __syncthreads();
    // K row and V block start of position t (its page's block, t inside it)
    auto krow_of = [&](int t) {
        int lt;
        const size_t b = kv_block(kp, layer, Hkv, kv_page(kp, slot, t, &lt), kvh);
        return kc + b + static_cast<size_t>(lt) * D;
    };
    auto vblk_of = [&](int t) {
        int lt;
        const size_t b = kv_block(kp, layer, Hkv, kv_page(kp, slot, t, &lt), kvh);
        return vc + b + static_cast<size_t>(lt >> 3) * D * 8 + (lt & 7);
    };
    const float scale = 1.0f / sqrtf(static_cast<float>(D));
    float m = -INFINITY, l = 0.0f;
    float acc0 = 0.0f, acc1 = 0.0f;   // d = lane, lane + 64
    for (int t0 = 0; t0 <= pos; t0 += 64) {
        const int t = t0 + lane;
        float s = -INFINITY;
        if (t <= pos) {
            const float* kr = krow_of(t);
            float d = 0.0f;
            for (int i = 0; i < D; ++i) d = fmaf(qs[i], kr[i], d);
            s = d * scale;
        }
        const float mx = wave_max(s);
        const float m_new = fmaxf(m, mx);
        const float alpha = expf(m - m_new);
        const float p = t <= pos ? expf(s - m_new) : 0.0f;
        l = l * alpha + wave_sum(p);
        m = m_new;
        ps[lane] = p;
        __syncthreads();
        acc0 *= alpha;
        acc1 *= alpha;
        const int nt = min(64, pos + 1 - t0);
        for (int tt = 0; tt < nt; ++tt) {
            const float* vblk = vblk_of(t0 + tt);
            if (lane < D) acc0 = fmaf(ps[tt], vblk[static_cast<size_t>(lane) * 8], acc0);
            if (lane + 64 < D) acc1 = fmaf(ps[tt], vblk[static_cast<size_t>(lane + 64) * 8], acc1);
        }
        __syncthreads();
    }
    float* orow = out + (static_cast<size_t>(r) * Hq + h) * D;
    if (lane < D) orow[lane] = acc0 / l;
    if (lane + 64 < D) orow[lane + 64] = acc1 / l;
}

hipError_t launch_attention_f32(int n_rows, const int32_t* row_slot, const int32_t* row_pos,
                                const float* q, const float* kc, const float* vc, const KvPages& kp,
                                int Hq, int Hkv, int D, int layer, float* out,
                                hipStream_t s) {
    if (n_rows <= 0) return hipSuccess;
    hipLaunchKernelGGL(attn_f32_kernel, dim3(n_rows, Hq), dim3(64), 0, s, row_slot, row_pos, q, kc,
                       vc, kp, Hq, Hkv, D, layer, out);
    return hipGetLastError();
}

}  // namespace rl
