// gockpt_kernels.hip -- device side of the GoCkpt hot path for gfx950.
//
//   prepass_kernel   one read of the 16-bit gradients (bf16 or fp16, Sec. 2.2):
//                    inf/NaN test on the raw bits (loss-scale skip) and the
//                    sum of squares of the unscaled gradient; one partial per
//                    block.
//   scan_kernel      the prepass over one bucket of gradients [begin, end),
//                    run by the caller as soon as the backward has written
//                    it: inf/NaN test and the sum of squares of the scaled
//                    gradient in fp64 (the scale is applied at the finalize,
//                    so the scan does not depend on the previous step).  Also
//                    the prepass of a small space whose step is not one launch.
//   finalize_kernel  one block: reduces the partials (of the prepass or of the
//                    bucket scans) in a fixed order, moves the loss scaler
//                    and the step count, computes the step's scalars and
//                    writes the step record (and, inside a window, the skip
//                    decision to the host).
//   gate_kernel      one wavefront on the copy stream that waits until the
//                    host has emptied a staging slot before a copy reuses it.
//   step_kernel      a small space's whole step in one launch, or its end
//                    (finalize and update) behind a prepass or bucket scans.
//   gather_kernel    the copies of a small window step to pinned host memory.
//   init_kernel      the workspace of a new context.
//   fused_kernel     the mixed-precision AdamW update of every element
//                    (Sec. 2.2, AdamW of Sec. 4.3.1) fused with the window's
//                    pack (Sec. 4.2.1): the step's part of the updated state
//                    and the gradients of the parts already sent are written
//                    into the staging ring in the same pass over HBM.
//
// Memory layout: flat structure-of-arrays -- master, exp_avg, exp_avg_sq
// (fp32), working weights (bf16) and gradients (bf16 or fp16), each
// contiguous over the flat parameter space.  The fused kernel gives each lane
// one quad of 4 consecutive elements per tile (see fused_kernel); the prepass
// reads 8 gradients per lane per iteration.  The large kernels are HBM-bound
// (28 bytes per element per step plus the pack) and the work is elementwise:
// no matrix cores, and LDS only where blocks reduce a sum, in step_kernel to
// hand the step's scalars and the exchange's result around, and in
// fused_kernel as an allocation that limits how many blocks share a compute
// unit.

#include <hip/hip_runtime.h>

#include "gockpt_internal.h"

#pragma clang fp contract(off)

namespace gockpt {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ u32x4 ld_u32x4(const void* p) {
    return *reinterpret_cast<const u32x4*>(p);
}

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// State streams of the fused kernel: every byte is touched once per step and
// next used a whole training step later, far beyond what the caches hold, so
// loads and stores carry the nontemporal hint (measured on the update's
// memory twin: 6.19 -> 6.49 TB/s with the state spread over HBM).
template <bool kNT, class T>
__device__ __forceinline__ T ld_stream(const T* p) {
    if constexpr (kNT)
        return __builtin_nontemporal_load(p);
    else
        return *p;
}
// A store of 8 or 16 bytes at a byte offset into a tile whose base is the same
// for the whole block.  kThrough: beside the hint it is written through the L2
// (sc1), so that no line waits there for its turn.  For the bandwidth-bound
// shape, the update from 4.2e6 elements on; us a step with the hint alone and
// written through: 5.0e6 elements 31.2 and 31.2, 6.3e6 35.5 and 35.4, 8.4e6
// 46.2 and 45.7, 10.5e6 55.8 and 54.9, 12.6e6 65.2 and 63.8, 16.8e6 77.9 and
// 76.5, 33.6e6 151.5 and 149.5, 124e6 573 and 562, 350e6 1660 and 1635, 1.63e9
// the same within 0.5%.  Not for 2.1e6 elements, whose lines the next step
// still finds in the L2: 17.1 and 17.9.
template <bool kNT, bool kThrough, uint32_t kTileBytes, class T>
__device__ __forceinline__ void st_tile(void* base, uint32_t off, T v) {
    static_assert(sizeof(T) == 16 || sizeof(T) == 8, "8 or 16 bytes");
    if constexpr (!kNT) {
        *reinterpret_cast<T*>(static_cast<uint8_t*>(base) + off) = v;
    } else {
        constexpr int kBits = kThrough ? 2 | 16 : 2;  // nt, sc1
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(base, 0, kTileBytes, 0x00020000);
        if constexpr (sizeof(T) == 16)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rsrc, off, 0, kBits);
        else
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), rsrc, off, 0, kBits);
    }
}

// Ring stores: the ring is only read back by the copy engine, so bypass the
// caches' retention policy with nontemporal stores.  `off` < 2*ring_bytes.
__device__ __forceinline__ void ring_st16(const PackPlan& pk, uint64_t off, u32x4 v) {
    if (off >= pk.ring_bytes) off -= pk.ring_bytes;
    u32x4* dst = reinterpret_cast<u32x4*>(pk.ring + off);
    if (pk.ring_nt)
        __builtin_nontemporal_store(v, dst);
    else
        *dst = v;
}
__device__ __forceinline__ void ring_st_u16(const PackPlan& pk, uint64_t off, uint16_t v) {
    if (off >= pk.ring_bytes) off -= pk.ring_bytes;
    *reinterpret_cast<uint16_t*>(pk.ring + off) = v;
}
__device__ __forceinline__ void ring_st_f32(const PackPlan& pk, uint64_t off, float v) {
    if (off >= pk.ring_bytes) off -= pk.ring_bytes;
    *reinterpret_cast<float*>(pk.ring + off) = v;
}

// ---------------------------------------------------------------------------
// Block reductions (4 wavefronts of 64).
// ---------------------------------------------------------------------------
__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}

template <int kThreads>
__device__ __forceinline__ void block_reduce(double& sum, uint32_t& flag) {
    static_assert(kThreads % 64 == 0, "wave multiple");
    constexpr int kWaves = kThreads / 64;
    __shared__ double s_sum[kWaves];
    __shared__ uint32_t s_flag[kWaves];
    sum = wave_sum(sum);
    flag = __any(flag != 0u) ? 1u : 0u;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    if (lane == 0) {
        s_sum[wave] = sum;
        s_flag[wave] = flag;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        uint32_t f = 0u;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            t += s_sum[w];
            f |= s_flag[w];
        }
        sum = t;
        flag = f;
    }
}

// ---------------------------------------------------------------------------
// Prepass: inf/NaN flag + sum of squares of the unscaled gradient.
// ---------------------------------------------------------------------------
// Gradient value for the norm: fp16 through the hardware conversion, which
// is exact for every finite value and infinity (the norm is telemetry; the
// update uses the contract's widening).
template <int kKind>
__device__ __forceinline__ float norm_value(uint16_t h) {
    if constexpr (kKind == kGradFP16)
        return static_cast<float>(__builtin_bit_cast(_Float16, h));
    else
        return bf16_to_f32(h);
}

template <int kKind>
__device__ __forceinline__ uint32_t word_nonfinite(uint32_t w) {
    // two 16-bit values; exponent field all ones means inf or NaN
    return (grad_nonfinite<kKind>(static_cast<uint16_t>(w & 0xFFFFu)) ? 1u : 0u) |
           (grad_nonfinite<kKind>(static_cast<uint16_t>(w >> 16)) ? 1u : 0u);
}

// ---------------------------------------------------------------------------
// End of a step, by one thread: skip decision, loss scaler, step count,
// scalars, record.  `in` is the state before the step; acc and bad are the
// step's sum of squares and inf/NaN flag.
// ---------------------------------------------------------------------------
struct StepState {
    int64_t t, tracker;
    float scale;
};

__device__ void finish_step(uint8_t* __restrict__ ws, const FinalizeArgs& fa, StepState in, double acc,
                            uint32_t bad) {
    const ScalerCfg& sc = fa.sc;
    DevScaler* st = reinterpret_cast<DevScaler*>(ws + kWsScalerOff);
    gockpt_step_record* rec = reinterpret_cast<gockpt_step_record*>(ws + kWsRecordsOff) + fa.slot;
    const float scale_used = in.scale;
    int64_t t = in.t;
    int64_t tracker = in.tracker;
    float scale = scale_used;
    const int skip = (sc.check_overflow != 0 && bad != 0u) ? 1 : 0;
    if (skip) {
        if (sc.dynamic_scale) {
            const float reduced = scale * sc.backoff_factor;
            scale = reduced < sc.min_scale ? sc.min_scale : reduced;
            tracker = 0;
        }
    } else {
        t = t + 1;
        if (sc.dynamic_scale) {
            tracker = tracker + 1;
            if (tracker == sc.growth_interval) {
                scale = scale * sc.growth_factor;
                tracker = 0;
            }
        }
    }
    st->t = t;
    st->tracker = tracker;
    st->scale = scale;

    const StepScalars s = step_scalars(fa.hp, fa.lr, t, scale_used);
    if (fa.raw) {  // bucket scans summed squares of the scaled gradients
        const double inv = static_cast<double>(s.inv_scale);
        acc = acc * inv * inv;
    }
    rec->t = t;
    rec->tracker = tracker;
    rec->scale_used = scale_used;
    rec->scale_next = scale;
    rec->lr = fa.lr;
    rec->skip = skip;
    rec->nonfinite = static_cast<int32_t>(bad);
    rec->window_step = fa.window_step;
    rec->gnorm2 = fa.norm_off ? -1.0 : acc;
    rec->step_size = s.step_size;
    rec->sqrt_bc2 = s.sqrt_bc2;
    rec->decay = s.decay;
    rec->inv_scale = s.inv_scale;
    // the host reads the decision from its own memory once the step's
    // finalize has completed (vector store, system scope)
    if (fa.skip_out != nullptr) __hip_atomic_store(fa.skip_out, skip, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---------------------------------------------------------------------------
// Finalize: one whole block of kBlock threads reduces the partials of the
// step and ends it.
// ---------------------------------------------------------------------------
__device__ void finalize_block(uint8_t* __restrict__ ws, const Partial* __restrict__ parts, int nparts,
                               const FinalizeArgs& fa) {
    // Thread t sums partials t, t + kBlock, ... in that order; the loads of
    // eight of them are issued before any is added, so one block does not
    // wait out eight memory latencies in a row.
    double acc = 0.0;
    uint32_t bad = 0u;
    constexpr int kBatch = 8;
    for (int b0 = 0; b0 < nparts; b0 += kBlock * kBatch) {
        double v[kBatch];
        int32_t f[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            const int b = b0 + k * kBlock + static_cast<int>(threadIdx.x);
            v[k] = b < nparts ? parts[b].sumsq : 0.0;
            f[k] = b < nparts ? parts[b].nonfinite : 0;
        }
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            acc += v[k];
            bad |= static_cast<uint32_t>(f[k]);
        }
    }
    block_reduce<kBlock>(acc, bad);
    if (threadIdx.x != 0) return;
    // a caller-side overflow test replaces the scan (NaN counts as set)
    if (fa.found_inf != nullptr) bad = (*fa.found_inf != 0.0f) ? 1u : 0u;

    const DevScaler* st = reinterpret_cast<const DevScaler*>(ws + kWsScalerOff);
    finish_step(ws, fa, StepState{st->t, st->tracker, st->scale}, acc, bad);
}

// One 8-element group of gradients (16 B), nontemporal or cached.
template <bool kNT>
__device__ __forceinline__ u32x4 ld_group(const uint16_t* p) {
    return kNT ? __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p)) : ld_u32x4(p);
}

// Calls f(group) for this thread's groups gi, gi + stride, ... below ngroups
// (a multiple of kAhead of them: zeros stand in beyond the end).  The next
// kAhead loads are issued before the arithmetic of the current ones.
template <bool kNT, int kAhead, class F>
__device__ __forceinline__ void each_group(const uint16_t* g, int64_t gi, int64_t stride, int64_t ngroups, F&& f) {
    u32x4 next[kAhead];
    auto load = [&](int64_t first) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            next[u] = (u32x4){0u, 0u, 0u, 0u};
            if (first + u * stride < ngroups) next[u] = ld_group<kNT>(g + (first + u * stride) * kVec);
        }
    };
    load(gi);
    for (; gi < ngroups; gi += kAhead * stride) {
        u32x4 raw[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) raw[u] = next[u];
        load(gi + kAhead * stride);
#pragma unroll
        for (int u = 0; u < kAhead; ++u) f(raw[u]);
    }
}

template <bool kNT, int kKind>
__global__ __launch_bounds__(kBlock) void prepass_kernel(const uint16_t* __restrict__ g, int64_t n,
                                                         uint8_t* __restrict__ ws) {
    const DevScaler* st = reinterpret_cast<const DevScaler*>(ws + kWsScalerOff);
    Partial* parts = reinterpret_cast<Partial*>(ws + kWsPartialsOff);
    const float inv_scale = 1.0f / st->scale;
    const int64_t ngroups = n / kVec;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    double acc = 0.0;
    uint32_t bad = 0u;
    each_group<kNT, kPrepassAhead>(g, static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x, stride, ngroups, [&](u32x4 raw) {
        float s = 0.0f;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t w = raw[k];
            bad |= word_nonfinite<kKind>(w);
            const float a = norm_value<kKind>(static_cast<uint16_t>(w & 0xFFFFu)) * inv_scale;
            const float b = norm_value<kKind>(static_cast<uint16_t>(w >> 16)) * inv_scale;
            s = s + a * a;
            s = s + b * b;
        }
        acc += static_cast<double>(s);
    });
    if (blockIdx.x == 0) {
        const int64_t i = ngroups * kVec + threadIdx.x;
        if (threadIdx.x < kVec && i < n) {
            const uint16_t h = g[i];
            bad |= grad_nonfinite<kKind>(h) ? 1u : 0u;
            const float a = norm_value<kKind>(h) * inv_scale;
            acc += static_cast<double>(a * a);
        }
    }
    block_reduce<kBlock>(acc, bad);
    // One partial per block; the finalize kernel reduces them.  (Having the
    // last block to finish run the finalize instead saves a launch, but needs
    // an agent-scope release per block, which on this chip writes back the
    // XCD's L2 each time: measured slower at every size.)
    if (threadIdx.x == 0) {
        parts[blockIdx.x].sumsq = acc;
        parts[blockIdx.x].nonfinite = static_cast<int32_t>(bad);
        parts[blockIdx.x].pad = 0;
    }
}

// ---------------------------------------------------------------------------
// Bucket scan: the prepass over [begin, end), begin a multiple of kVec (end
// too, unless it is n).  Squares are taken of the scaled values in fp64, so
// they cannot overflow; the finalize applies the step's inv_scale.
// ---------------------------------------------------------------------------
template <bool kNT, int kKind>
__global__ __launch_bounds__(kBlock) void scan_kernel(const uint16_t* __restrict__ g, int64_t begin, int64_t end,
                                                      Partial* __restrict__ parts) {
    const int64_t ngroups = (end - begin) / kVec;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    const uint16_t* base = g + begin;
    double acc = 0.0;
    uint32_t bad = 0u;
    each_group<kNT, kScanAhead>(base, static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x, stride, ngroups, [&](u32x4 raw) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t w = raw[k];
            bad |= word_nonfinite<kKind>(w);
            const double a = static_cast<double>(norm_value<kKind>(static_cast<uint16_t>(w & 0xFFFFu)));
            const double b = static_cast<double>(norm_value<kKind>(static_cast<uint16_t>(w >> 16)));
            acc += a * a;
            acc += b * b;
        }
    });
    if (blockIdx.x == 0) {
        const int64_t i = begin + ngroups * kVec + threadIdx.x;
        if (threadIdx.x < kVec && i < end) {
            const uint16_t h = g[i];
            bad |= grad_nonfinite<kKind>(h) ? 1u : 0u;
            const double a = static_cast<double>(norm_value<kKind>(h));
            acc += a * a;
        }
    }
    block_reduce<kBlock>(acc, bad);
    if (threadIdx.x == 0) {
        parts[blockIdx.x].sumsq = acc;
        parts[blockIdx.x].nonfinite = static_cast<int32_t>(bad);
        parts[blockIdx.x].pad = 0;
    }
}

// ---------------------------------------------------------------------------
// Finalize on its own: above kAfterMaxElems, in timed and HOST_WAIT windows,
// with a launch knob, and behind more than kAfterMaxParts scan partials.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void finalize_kernel(uint8_t* __restrict__ ws, const Partial* __restrict__ parts,
                                                          int nparts, FinalizeArgs fa) {
    finalize_block(ws, parts, nparts, fa);
}

// ---------------------------------------------------------------------------
// The workspace of a new context, in one block (a caller's need not be
// cleared, and the library's own holds what its last context left).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void init_kernel(uint8_t* __restrict__ ws, int64_t t, int64_t tracker,
                                                      float scale) {
    uint32_t* words = reinterpret_cast<uint32_t*>(ws + kWsSlotsOff);
    for (size_t i = threadIdx.x; i < (kWsStepEnd - kWsSlotsOff) / 4; i += kBlock) words[i] = 0u;
    if (threadIdx.x != 0) return;
    *reinterpret_cast<DevScaler*>(ws + kWsScalerOff) = DevScaler{t, tracker, scale, 0, {}};
    *reinterpret_cast<StepSync*>(ws + kWsSyncOff) = StepSync{1u, 0u, 0u, {}};
}

// ---------------------------------------------------------------------------
// Gate of the staged copies: the copy stream goes on once the host has moved
// enough earlier copies out of their staging slots.  One wavefront polls the
// host's counter (system-scope loads, never cached) and sleeps between polls;
// every wave leaves after the deadline or an iteration cap at the latest.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void gate_kernel(const uint64_t* released, uint64_t target, uint64_t max_ticks,
                                                  uint32_t* timed_out) {
    const uint64_t t0 = wall_clock64();
    const uint64_t max_iter = max_ticks;  // at least one clock tick per iteration
    bool ok = false;
    for (uint64_t it = 0; it < max_iter; ++it) {
        const uint64_t v = __hip_atomic_load(released, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_SYSTEM);
        if (v >= target) {
            ok = true;
            break;
        }
        if (wall_clock64() - t0 >= max_ticks) break;
        __builtin_amdgcn_s_sleep(16);
    }
    if (!ok && threadIdx.x == 0) __hip_atomic_store(timed_out, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---------------------------------------------------------------------------
// The copies of a small window step to pinned host memory, one launch instead
// of a DMA transfer per range, blockIdx.y per range.  The link bounds the
// bytes (57 GB/s), the calls a small step: a window of 4 steps over 65560
// elements took 378 us to its drain with 19 transfers and 193 with 4 launches,
// over 262144 elements 378 and 205.  See kGatherMaxBytes for where it stops.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void gather_kernel(GatherArgs a) {
    const uint8_t* src = a.seg[blockIdx.y].src;
    uint8_t* dst = a.seg[blockIdx.y].dst;
    const uint64_t bytes = a.seg[blockIdx.y].bytes;
    const uint64_t units = bytes / 16;
    for (uint64_t u = static_cast<uint64_t>(blockIdx.x) * kBlock + threadIdx.x; u < units;
         u += static_cast<uint64_t>(gridDim.x) * kBlock)
        __builtin_nontemporal_store(ld_u32x4(src + u * 16), reinterpret_cast<u32x4*>(dst + u * 16));
    if (blockIdx.x == 0 && threadIdx.x < bytes % 16) dst[units * 16 + threadIdx.x] = src[units * 16 + threadIdx.x];
}

// ---------------------------------------------------------------------------
// Fused AdamW update + window pack.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t pack2_bf16(float a, float b) {
    return static_cast<uint32_t>(f32_to_bf16_rne(a)) | (static_cast<uint32_t>(f32_to_bf16_rne(b)) << 16);
}

__device__ __forceinline__ void ring_st8(const PackPlan& pk, uint64_t off, u32x2 v) {
    if (off >= pk.ring_bytes) off -= pk.ring_bytes;
    u32x2* dst = reinterpret_cast<u32x2*>(pk.ring + off);
    if (pk.ring_nt)
        __builtin_nontemporal_store(v, dst);
    else
        *dst = v;
}

__device__ __forceinline__ void ring_st_f32x4(const PackPlan& pk, uint64_t off, f32x4 v) {
    ring_st16(pk, off, __builtin_bit_cast(u32x4, v));
}

// Where a tile of kTile elements from element i0 meets the ends of the
// arrays and of the pack ranges: offsets inside the tile, the same for every
// lane of the block (they stay in scalar registers).
struct TileSpan {
    uint32_t g_end;     // gradients below it are packed
    uint32_t c_beg;     // state from it on may be packed...
    uint32_t s_end[3];  // ...up to here, per state array
};

template <uint32_t kTile>
__device__ __forceinline__ uint32_t tile_cut(int64_t x, int64_t i0) {
    const int64_t d = x - i0;
    return d <= 0 ? 0u : (d >= static_cast<int64_t>(kTile) ? kTile : static_cast<uint32_t>(d));
}

template <uint32_t kTile>
__device__ __forceinline__ TileSpan tile_span(const FusedArgs& a, int64_t i0, int skip) {
    TileSpan t;
    t.g_end = skip ? 0u : tile_cut<kTile>(a.pack.g_end, i0);  // a skipped step's gradients are never replayed
    t.c_beg = tile_cut<kTile>(a.pack.cb, i0);
#pragma unroll
    for (int k = 0; k < 3; ++k) t.s_end[k] = tile_cut<kTile>(a.pack.s_end[k], i0);
    return t;
}

__device__ __forceinline__ bool tile_packs_state(const TileSpan& t) {
    return t.c_beg < t.s_end[0] || t.c_beg < t.s_end[1] || t.c_beg < t.s_end[2];
}

// AdamW of one quad in registers.
template <int kKind>
__device__ __forceinline__ void update_quad(const StepScalars& s, u32x2 graw, f32x4& pv, f32x4& mv, f32x4& vv) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const uint32_t word = graw[e >> 1];
        const uint16_t gb = static_cast<uint16_t>((e & 1) ? (word >> 16) : (word & 0xFFFFu));
        float p = pv[e], m = mv[e], v = vv[e];
        adamw_update<kKind>(s, gb, p, m, v);
        pv[e] = p;
        mv[e] = m;
        vv[e] = v;
    }
}

// The quad at tile offset o into the ring, as far as the pack ranges reach
// (they are multiples of 8 elements, so a quad lies inside one or outside).
__device__ __forceinline__ void pack_quad(const PackPlan& pk, const TileSpan& t, int64_t i0, uint32_t o, u32x2 graw,
                                          f32x4 pv, f32x4 mv, f32x4 vv) {
    if (o < t.g_end) ring_st8(pk, pk.off_g + 2ull * static_cast<uint64_t>(i0) + 2u * o, graw);
    if (o >= t.c_beg) {
        const uint64_t rel = 4ull * static_cast<uint64_t>(i0 - pk.cb) + 4u * o;
        if (o < t.s_end[0]) ring_st_f32x4(pk, pk.off_s[0] + rel, pv);
        if (o < t.s_end[1]) ring_st_f32x4(pk, pk.off_s[1] + rel, mv);
        if (o < t.s_end[2]) ring_st_f32x4(pk, pk.off_s[2] + rel, vv);
    }
}

// The last n % 4 elements, one per thread.
template <bool kHasW, int kKind>
__device__ __forceinline__ void update_tail(const FusedArgs& a, const StepScalars& s, int skip) {
    const PackPlan& pk = a.pack;
    const int64_t i = a.n / 4 * 4 + threadIdx.x;
    if (threadIdx.x >= 4 || i >= a.n) return;
    const bool pack_g = !skip && i < pk.g_end;
    const bool in_c = i >= pk.cb;
    const uint16_t gb = a.g[i];
    float p = a.p[i], m = a.m[i], v = a.v[i];
    if (!skip) {
        adamw_update<kKind>(s, gb, p, m, v);
        a.p[i] = p;
        a.m[i] = m;
        a.v[i] = v;
        if (kHasW) a.w[i] = f32_to_bf16_rne(p);
    }
    if (pack_g) ring_st_u16(pk, pk.off_g + 2ull * static_cast<uint64_t>(i), gb);
    if (in_c) {
        const uint64_t rel = 4ull * static_cast<uint64_t>(i - pk.cb);
        if (i < pk.s_end[0]) ring_st_f32(pk, pk.off_s[0] + rel, p);
        if (i < pk.s_end[1]) ring_st_f32(pk, pk.off_s[1] + rel, m);
        if (i < pk.s_end[2]) ring_st_f32(pk, pk.off_s[2] + rel, v);
    }
}

// A quad is 4 consecutive elements.  A block of kB threads owns a tile of
// kB * kQ quads; thread t takes quads t, t + kB, ..., so every load and store
// instruction of a wavefront covers 64 consecutive quads (1 KiB of fp32,
// 512 B of bf16) and concurrently running blocks walk memory in order.  All
// loads of a thread are issued before any arithmetic.  Whether a tile is
// whole, is skipped or packs anything is the same for the whole block, so the
// tiles that only update -- nearly all outside a window -- run without a
// predicate, on one base address per array.
//
// HBM bounds it, and how much of HBM's rate it gets depends on how many
// wavefronts stream at once: with every wave slot filled (32 a compute unit)
// the reads and writes of the five arrays disturb each other in the memory.
// See launch_fused_q for the residency and what it measured.
template <bool kHasW, int kQ, int kKind, bool kNT, int kB>
__global__ __launch_bounds__(kB) void fused_kernel(FusedArgs a) {
    constexpr uint32_t kTile = kB * kQ * 4;
    const gockpt_step_record* rec = a.rec;
    const int skip = rec->skip;
    StepScalars s;
    s.b1 = a.b1;
    s.b2 = a.b2;
    s.omb1 = a.omb1;
    s.omb2 = a.omb2;
    s.eps = a.eps;
    s.decay = rec->decay;
    s.step_size = rec->step_size;
    s.sqrt_bc2 = rec->sqrt_bc2;
    s.inv_scale = rec->inv_scale;

    const int64_t i0 = static_cast<int64_t>(blockIdx.x) * kTile;
    const uint32_t live = tile_cut<kTile>(a.n & ~int64_t{3}, i0);  // the tile's whole quads end here
    const uint16_t* gt = a.g + i0;
    float* pt = a.p + i0;
    float* mt = a.m + i0;
    float* vt = a.v + i0;
    uint16_t* wt = a.w + i0;
    u32x2 graw[kQ];
    f32x4 pv[kQ], mv[kQ], vv[kQ];
    const uint32_t o0 = threadIdx.x * 4u;
    if (!skip && live == kTile) {
#pragma unroll
        for (int h = 0; h < kQ; ++h) {
            const uint32_t o = o0 + h * (kB * 4u);
            graw[h] = ld_stream<kNT>(reinterpret_cast<const u32x2*>(gt + o));
            pv[h] = ld_stream<kNT>(reinterpret_cast<const f32x4*>(pt + o));
            mv[h] = ld_stream<kNT>(reinterpret_cast<const f32x4*>(mt + o));
            vv[h] = ld_stream<kNT>(reinterpret_cast<const f32x4*>(vt + o));
        }
#pragma unroll
        for (int h = 0; h < kQ; ++h) {
            const uint32_t o = o0 + h * (kB * 4u);
            update_quad<kKind>(s, graw[h], pv[h], mv[h], vv[h]);
            st_tile<kNT, kB == kFusedBlock, kTile * 4>(pt, o * 4u, pv[h]);
            st_tile<kNT, kB == kFusedBlock, kTile * 4>(mt, o * 4u, mv[h]);
            st_tile<kNT, kB == kFusedBlock, kTile * 4>(vt, o * 4u, vv[h]);
            if (kHasW) {
                const u32x2 wv = {pack2_bf16(pv[h][0], pv[h][1]), pack2_bf16(pv[h][2], pv[h][3])};
                st_tile<kNT, kB == kFusedBlock, kTile * 2>(wt, o * 2u, wv);
            }
        }
        if (a.pack.any) {
            const TileSpan t = tile_span<kTile>(a, i0, 0);
            if (t.g_end != 0u || tile_packs_state(t)) {
#pragma unroll
                for (int h = 0; h < kQ; ++h)
                    pack_quad(a.pack, t, i0, o0 + h * (kB * 4u), graw[h], pv[h], mv[h], vv[h]);
            }
        }
    } else if (live != 0u) {
        // the last tile, or a skipped step (which only packs its part's
        // unchanged state)
        const TileSpan t = tile_span<kTile>(a, i0, skip);
        const bool packs_state = tile_packs_state(t);
#pragma unroll
        for (int h = 0; h < kQ; ++h) {
            const uint32_t o = o0 + h * (kB * 4u);
            if (o >= live || (skip && !packs_state)) continue;
            graw[h] = (u32x2){0u, 0u};
            if (!skip) graw[h] = ld_stream<kNT>(reinterpret_cast<const u32x2*>(gt + o));
            pv[h] = ld_stream<kNT>(reinterpret_cast<const f32x4*>(pt + o));
            mv[h] = ld_stream<kNT>(reinterpret_cast<const f32x4*>(mt + o));
            vv[h] = ld_stream<kNT>(reinterpret_cast<const f32x4*>(vt + o));
            if (!skip) {
                update_quad<kKind>(s, graw[h], pv[h], mv[h], vv[h]);
                st_tile<kNT, kB == kFusedBlock, kTile * 4>(pt, o * 4u, pv[h]);
                st_tile<kNT, kB == kFusedBlock, kTile * 4>(mt, o * 4u, mv[h]);
                st_tile<kNT, kB == kFusedBlock, kTile * 4>(vt, o * 4u, vv[h]);
                if (kHasW) {
                    const u32x2 wv = {pack2_bf16(pv[h][0], pv[h][1]), pack2_bf16(pv[h][2], pv[h][3])};
                    st_tile<kNT, kB == kFusedBlock, kTile * 2>(wt, o * 2u, wv);
                }
            }
            pack_quad(a.pack, t, i0, o, graw[h], pv[h], mv[h], vv[h]);
        }
    }
    if (blockIdx.x == 0) update_tail<kHasW, kKind>(a, s, skip);
}

// ---------------------------------------------------------------------------
// A whole step in one launch, for small spaces (at most kStepMaxElems).
//
// Prepass, finalize and update as launches of their own cost about 3.7 us
// each however little they do, and the gradients are read twice.  Here each
// block keeps its tile in registers from the inf/NaN test to the update, and
// the blocks exchange their partial sums through memory in between, so every
// byte is read once.  Latency bounds it: the launch, one round of loads, the
// exchange (about 1.3 us) and one round of stores.  Steps one after the other
// on one stream, three launches against one: 11.0 us and 7.6 for 65560
// elements, 11.4 and 8.2 for 524288, 11.1 and 9.8 for 1048579; without
// anything to exchange 6.2, 6.9 and 8.3.  The update's arithmetic runs before
// the exchange and one wavefront polls for all: with the update after it and
// a barrier per poll 7.8, 8.9 and 10.0.
//
// The exchange needs no block to be running beside another one.  A block that
// has waited kStepHelpSpins polls for a partial computes the missing ones
// itself: a partial depends on the gradients alone, which nothing writes
// during the kernel, so whoever computes it publishes the same bits.  Every
// running block can therefore finish on its own, and a block that starts late
// finds all partials there and updates its own tile.  The loss-scaler state
// is read by every block and moved on by the last one to have read it.
//
// A partial is one 64-bit word: a double, and in the place of its sign, which
// a sum of squares has no use for, the step's epoch modulo two, which the last
// block moves on too.  A reader thus needs no order between the partial and a
// flag: no fence, which on this chip would write back an XCD's L2.  Every step
// writes every slot, so a slot whose tag is not this epoch's holds the last
// step's partial: one bit tells them apart, and the sum keeps all of its bits
// (the double in two words with 32 bits of epoch each: 10.1 us against 9.9 for
// 1048579 elements).  A sum of squares in fp64 is finite exactly when every
// gradient is, so the inf/NaN flag needs no bits of its own.
// ---------------------------------------------------------------------------
struct StepIn {  // what a block reads of the workspace
    StepState st;
    uint32_t epoch;
};

template <class T>
__device__ __forceinline__ T ld_agent(const T* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sum over the block, the same bits in every thread.  A barrier follows
// before `lds` is used again.
template <int kB>
__device__ __forceinline__ double block_sum(double x, double* lds) {
    x = wave_sum(x);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = x;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kB / 64; ++w) t += lds[w];
    return t;
}

template <int kKind>
__device__ __forceinline__ double quad_sumsq(u32x2 g) {
    double acc = 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const uint32_t word = g[e >> 1];
        const double x = static_cast<double>(
            norm_value<kKind>(static_cast<uint16_t>((e & 1) ? (word >> 16) : (word & 0xFFFFu))));
        acc += x * x;
    }
    return acc;
}

// Sum of squares of the scaled gradients of tile b (the last n % 4 belong to
// tile 0), given its quads or loading them.
template <int kB, int kQ, int kKind>
__device__ __forceinline__ double tile_sumsq(const FusedArgs& a, int b, const u32x2* graw, double* lds) {
    constexpr uint32_t kTile = kB * kQ * 4;
    const int64_t i0 = static_cast<int64_t>(b) * kTile;
    const uint32_t live = tile_cut<kTile>(a.n & ~int64_t{3}, i0);
    double acc = 0.0;
#pragma unroll
    for (int h = 0; h < kQ; ++h) {
        const uint32_t o = threadIdx.x * 4u + h * (kB * 4u);
        u32x2 g = {0u, 0u};
        if (graw != nullptr)
            g = graw[h];
        else if (o < live)
            g = *reinterpret_cast<const u32x2*>(a.g + i0 + o);
        acc += quad_sumsq<kKind>(g);
    }
    if (b == 0 && threadIdx.x < 4) {
        const int64_t i = (a.n & ~int64_t{3}) + threadIdx.x;
        if (i < a.n) {
            const double x = static_cast<double>(norm_value<kKind>(a.g[i]));
            acc += x * x;
        }
    }
    return block_sum<kB>(acc, lds);
}

constexpr uint64_t kSlotTag = uint64_t{1} << 63;

__device__ __forceinline__ uint64_t slot_tag(uint32_t epoch) { return static_cast<uint64_t>(epoch) << 63; }
__device__ __forceinline__ void publish(uint64_t* slot, uint32_t epoch, double x) {
    __hip_atomic_store(slot, (__builtin_bit_cast(uint64_t, x) & ~kSlotTag) | slot_tag(epoch), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double slot_value(uint64_t w) { return __builtin_bit_cast(double, w & ~kSlotTag); }

// Counts this block in; true for the last of `tiles` blocks.  Two levels: one
// counter for all of them took 12 ns a block, 3 us for 256.
__device__ __forceinline__ bool arrive_last(StepSync* sync, StepArrive* lanes, int tiles) {
    const int lane = blockIdx.x % kStepArriveLanes;
    const uint32_t here = (tiles - lane + kStepArriveLanes - 1) / kStepArriveLanes;  // blocks of this lane
    const uint32_t used = tiles < kStepArriveLanes ? tiles : kStepArriveLanes;
    if (__hip_atomic_fetch_add(&lanes[lane].count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u != here)
        return false;
    return __hip_atomic_fetch_add(&sync->arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == used;
}

// kStepJoint: the step needs the sum over all gradients (overflow test or
// norm) and takes it itself.  kStepAfter: a prepass or bucket scans before it
// have left their partials (at most kAfterMaxParts), which every block reduces
// for itself instead of waiting for a finalize launch; kStepAlone: nothing is
// summed.  In these two no block waits for another's sum (they only count
// their arrivals, as kStepJoint does), so they may have more blocks than the
// device has places, and go up to kAfterMaxElems, where the separate kernels'
// shape changes.  us a step with a finalize launch and without: behind a
// prepass 2.1e6 elements 17.1 and 14.2, 4.2e6 27.6 and 25.4 (1.05e6 the same);
// alone 13.4 and 10.6, 22.1 and 20.7; behind 4 bucket scans 100 and 89.
template <bool kHasW, int kB, int kQ, int kKind, int kMode>
__global__ __launch_bounds__(kB) void step_kernel(FusedArgs a, FinalizeArgs fa, uint8_t* __restrict__ ws,
                                                  const Partial* __restrict__ parts, int nparts, int again) {
    constexpr uint32_t kTile = kB * kQ * 4;
    __shared__ StepScalars s_sc;
    __shared__ uint32_t s_epoch, s_found, s_done;
    __shared__ double s_sum[kB / 64], s_total;
    __shared__ uint32_t s_bad[kB / 64];
    __shared__ uint8_t s_missing[kStepMaxTiles];
    const int tid = threadIdx.x;
    const int tiles = gridDim.x;
    StepSync* sync = reinterpret_cast<StepSync*>(ws + kWsSyncOff);
    uint64_t* slots = reinterpret_cast<uint64_t*>(ws + kWsSlotsOff);
    StepArrive* lanes = reinterpret_cast<StepArrive*>(ws + kWsArriveOff);

    StepIn in{};
    float found = 0.0f;
    if (tid == 0) {
        const DevScaler* st = reinterpret_cast<const DevScaler*>(ws + kWsScalerOff);
        in.st = StepState{st->t, st->tracker, st->scale};
        in.epoch = sync->epoch;
        if (fa.found_inf != nullptr) found = *fa.found_inf;
    }
    const int64_t i0 = static_cast<int64_t>(blockIdx.x) * kTile;
    const uint32_t live = tile_cut<kTile>(a.n & ~int64_t{3}, i0);
    const uint32_t o0 = tid * 4u;
    u32x2 graw[kQ];
    f32x4 pv[kQ], mv[kQ], vv[kQ];
#pragma unroll
    for (int h = 0; h < kQ; ++h) {
        const uint32_t o = o0 + h * (kB * 4u);
        graw[h] = (u32x2){0u, 0u};
        pv[h] = mv[h] = vv[h] = (f32x4){0.f, 0.f, 0.f, 0.f};
        if (o < live) {
            graw[h] = *reinterpret_cast<const u32x2*>(a.g + i0 + o);
            pv[h] = *reinterpret_cast<const f32x4*>(a.p + i0 + o);
            mv[h] = *reinterpret_cast<const f32x4*>(a.m + i0 + o);
            vv[h] = *reinterpret_cast<const f32x4*>(a.v + i0 + o);
        }
    }
    bool last = false;
    if (tid == 0) {
        // the state is in registers before the arrival is counted: the last
        // block to arrive overwrites it
        asm volatile("" : "+v"(in.st.t), "+v"(in.st.tracker), "+v"(in.st.scale), "+v"(in.epoch) : : "memory");
        s_epoch = in.epoch;
        s_found = found != 0.0f ? 1u : 0u;  // a NaN flag counts as set
        s_sc = step_scalars(fa.hp, fa.lr, in.st.t + 1, in.st.scale);
    }

    double acc = 0.0;
    uint32_t bad = 0u;
    if constexpr (kMode == kStepJoint) {
        acc = tile_sumsq<kB, kQ, kKind>(a, blockIdx.x, graw, s_sum);
    } else if constexpr (kMode == kStepAfter) {
        for (int b = tid; b < nparts; b += kB) {
            acc += parts[b].sumsq;
            bad |= static_cast<uint32_t>(parts[b].nonfinite);
        }
        bad = __any(bad != 0u) ? 1u : 0u;
        if ((tid & 63) == 0) s_bad[tid >> 6] = bad;
        acc = block_sum<kB>(acc, s_sum);
#pragma unroll
        for (int w = 0; w < kB / 64; ++w) bad |= s_bad[w];
    } else {
        __syncthreads();
    }
    const uint32_t epoch = s_epoch;
    if (tid == 0) {
        if (kMode == kStepJoint) publish(slots + blockIdx.x, epoch, acc);
        last = arrive_last(sync, lanes, tiles);
    }

    // the update itself while the partials travel, in registers: only its
    // stores wait for the decision
    const StepScalars s = s_sc;
    u32x2 wv[kQ];
#pragma unroll
    for (int h = 0; h < kQ; ++h) {
        update_quad<kKind>(s, graw[h], pv[h], mv[h], vv[h]);
        wv[h] = (u32x2){pack2_bf16(pv[h][0], pv[h][1]), pack2_bf16(pv[h][2], pv[h][3])};
        asm volatile("" : "+v"(pv[h]), "+v"(mv[h]), "+v"(vv[h]), "+v"(wv[h]));  // here, not after the exchange
    }

    if constexpr (kMode == kStepJoint) {
        // the first wavefront polls, a lane for every 64th partial
        constexpr int kPer = kStepMaxTiles / 64;
        for (;; again = 0) {
            if (tid < 64) {
                uint64_t word[kPer];
                uint32_t missing = 0;  // bit k: this lane's k-th partial
                for (int spins = 0; spins < kStepHelpSpins; ++spins) {
                    missing = 0;
#pragma unroll
                    for (int k = 0; k < kPer; ++k) {
                        const int b = tid + 64 * k;
                        word[k] = b < tiles ? ld_agent(slots + b) : 0u;
                    }
#pragma unroll
                    for (int k = 0; k < kPer; ++k)
                        if (tid + 64 * k < tiles && (word[k] & kSlotTag) != slot_tag(epoch)) missing |= 1u << k;
                    if (__all(missing == 0u)) break;
                }
                if (__builtin_expect(again, 0)) {
#pragma unroll
                    for (int k = 0; k < kPer; ++k) missing |= (tid + 64 * k < tiles ? 1u : 0u) << k;
                }
                if (__all(missing == 0u)) {
                    double x = 0.0;
#pragma unroll
                    for (int k = 0; k < kPer; ++k) x += slot_value(word[k]);
                    x = wave_sum(x);
                    if (tid == 0) s_total = x, s_done = 1u;
                } else {
#pragma unroll
                    for (int k = 0; k < kPer; ++k) s_missing[tid + 64 * k] = (missing >> k) & 1u;
                    if (tid == 0) s_done = 0u;
                }
            }
            __syncthreads();
            if (__builtin_expect(s_done != 0u, 1)) break;
            for (int b = 0; b < tiles; ++b) {
                if (!s_missing[b]) continue;
                const double x = tile_sumsq<kB, kQ, kKind>(a, b, nullptr, s_sum);
                if (tid == 0) {
                    publish(slots + b, epoch, x);
                    __hip_atomic_fetch_add(&sync->helped, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                __syncthreads();
            }
            __syncthreads();  // everyone has read s_done and s_missing
        }
        acc = s_total;
        bad = (__builtin_bit_cast(uint64_t, acc) & 0x7FF0000000000000ull) == 0x7FF0000000000000ull ? 1u : 0u;
    }
    if (fa.found_inf != nullptr) bad = s_found;
    const int skip = (fa.sc.check_overflow != 0 && bad != 0u) ? 1 : 0;

    if (__builtin_expect(!skip, 1)) {
#pragma unroll
        for (int h = 0; h < kQ; ++h) {
            const uint32_t o = o0 + h * (kB * 4u);
            if (o >= live) continue;
            *reinterpret_cast<f32x4*>(a.p + i0 + o) = pv[h];
            *reinterpret_cast<f32x4*>(a.m + i0 + o) = mv[h];
            *reinterpret_cast<f32x4*>(a.v + i0 + o) = vv[h];
            if (kHasW) *reinterpret_cast<u32x2*>(a.w + i0 + o) = wv[h];
        }
    }
    if (__builtin_expect(a.pack.any, 0)) {
        const TileSpan t = tile_span<kTile>(a, i0, skip);
        const bool packs_state = tile_packs_state(t);
        if (t.g_end != 0u || packs_state) {
#pragma unroll
            for (int h = 0; h < kQ; ++h) {
                const uint32_t o = o0 + h * (kB * 4u);
                if (o >= live) continue;
                if (skip) {  // the registers hold an update that is not applied
                    pv[h] = *reinterpret_cast<const f32x4*>(a.p + i0 + o);
                    mv[h] = *reinterpret_cast<const f32x4*>(a.m + i0 + o);
                    vv[h] = *reinterpret_cast<const f32x4*>(a.v + i0 + o);
                }
                pack_quad(a.pack, t, i0, o, graw[h], pv[h], mv[h], vv[h]);
            }
        }
    }
    if (blockIdx.x == 0) update_tail<kHasW, kKind>(a, s, skip);

    if (__builtin_expect(last, 0)) {
        for (int k = 0; k < kStepArriveLanes; ++k) lanes[k].count = 0u;
        sync->arrived = 0u;
        if (kMode == kStepJoint) sync->epoch = in.epoch + 1u;
        finish_step(ws, fa, in.st, acc, bad);
    }
}

// ---------------------------------------------------------------------------
// Launchers.
// ---------------------------------------------------------------------------
static int env_int(const char* name, int dflt) {
    const char* s = getenv(name);
    if (s == nullptr || *s == '\0') return dflt;
    return atoi(s);
}

int scan_blocks_for(int64_t count, int max_blocks) {
    // at least four 8-element groups per lane
    int64_t b = (count / kVec + 4 * kBlock - 1) / (4 * kBlock);
    if (b < 1) b = 1;
    if (b > max_blocks) b = max_blocks;
    return static_cast<int>(b);
}

int launch_scan(const uint16_t* g, int64_t begin, int64_t end, void* parts, int nblocks, int nt, int grad_kind,
                void* stream) {
    hipStream_t s = static_cast<hipStream_t>(stream);
    Partial* p = static_cast<Partial*>(parts);
    if (grad_kind == kGradFP16) {
        if (nt)
            hipLaunchKernelGGL((scan_kernel<true, kGradFP16>), dim3(nblocks), dim3(kBlock), 0, s, g, begin, end, p);
        else
            hipLaunchKernelGGL((scan_kernel<false, kGradFP16>), dim3(nblocks), dim3(kBlock), 0, s, g, begin, end, p);
    } else {
        if (nt)
            hipLaunchKernelGGL((scan_kernel<true, kGradBF16>), dim3(nblocks), dim3(kBlock), 0, s, g, begin, end, p);
        else
            hipLaunchKernelGGL((scan_kernel<false, kGradBF16>), dim3(nblocks), dim3(kBlock), 0, s, g, begin, end, p);
    }
    return static_cast<int>(hipGetLastError());
}

Knobs default_knobs() {
    Knobs k;
    k.quads_per_thread = env_int("GOCKPT_QUADS", 1);
    k.ring_nt = env_int("GOCKPT_RING_NT", 1);
    k.prepass_nt = env_int("GOCKPT_PREPASS_NT", -1);
    k.fused_nt = env_int("GOCKPT_FUSED_NT", 1);
    k.fused_block = env_int("GOCKPT_FUSED_BLOCK", 0);
    k.step_again = env_int("GOCKPT_TEST_STEP_AGAIN", 0);
    k.defaults = k.quads_per_thread == 1 && k.ring_nt == 1 && k.prepass_nt != 0 && k.fused_nt == 1 &&
                 k.fused_block != kFusedWideBlock;
    return k;
}

int launch_prepass(const uint16_t* g, int64_t n, void* workspace, int nblocks, int nt, int grad_kind,
                   void* stream) {
    hipStream_t s = static_cast<hipStream_t>(stream);
    uint8_t* ws = static_cast<uint8_t*>(workspace);
    if (nblocks < 1 || nblocks > kPrepassMaxBlocks) return static_cast<int>(hipErrorInvalidValue);
    if (grad_kind == kGradFP16) {
        if (nt)
            hipLaunchKernelGGL((prepass_kernel<true, kGradFP16>), dim3(nblocks), dim3(kBlock), 0, s, g, n, ws);
        else
            hipLaunchKernelGGL((prepass_kernel<false, kGradFP16>), dim3(nblocks), dim3(kBlock), 0, s, g, n, ws);
    } else {
        if (nt)
            hipLaunchKernelGGL((prepass_kernel<true, kGradBF16>), dim3(nblocks), dim3(kBlock), 0, s, g, n, ws);
        else
            hipLaunchKernelGGL((prepass_kernel<false, kGradBF16>), dim3(nblocks), dim3(kBlock), 0, s, g, n, ws);
    }
    return static_cast<int>(hipGetLastError());
}

int launch_finalize(void* workspace, const void* parts, int nparts, const FinalizeArgs& fin, void* stream) {
    hipLaunchKernelGGL(finalize_kernel, dim3(1), dim3(kBlock), 0, static_cast<hipStream_t>(stream),
                       static_cast<uint8_t*>(workspace), static_cast<const Partial*>(parts), nparts, fin);
    return static_cast<int>(hipGetLastError());
}

int launch_gate(const uint64_t* released, uint64_t target, uint64_t max_ticks, uint32_t* timed_out, void* stream) {
    hipLaunchKernelGGL(gate_kernel, dim3(1), dim3(64), 0, static_cast<hipStream_t>(stream), released, target,
                       max_ticks, timed_out);
    return static_cast<int>(hipGetLastError());
}

int launch_init(void* workspace, int64_t t, int64_t tracker, float scale, void* stream) {
    hipLaunchKernelGGL(init_kernel, dim3(1), dim3(kBlock), 0, static_cast<hipStream_t>(stream),
                       static_cast<uint8_t*>(workspace), t, tracker, scale);
    return static_cast<int>(hipGetLastError());
}

int launch_gather(const GatherArgs& a, int nseg, void* stream) {
    if (nseg < 1 || nseg > kGatherSegs) return static_cast<int>(hipErrorInvalidValue);
    uint64_t most = 0;
    for (int k = 0; k < nseg; ++k) most = a.seg[k].bytes > most ? a.seg[k].bytes : most;
    uint64_t blocks = (most / 16 + 4 * kBlock - 1) / (4 * kBlock);
    blocks = blocks < 1 ? 1 : (blocks > kGatherBlocks ? kGatherBlocks : blocks);
    hipLaunchKernelGGL(gather_kernel, dim3(static_cast<unsigned>(blocks), static_cast<unsigned>(nseg)), dim3(kBlock),
                       0, static_cast<hipStream_t>(stream), a);
    return static_cast<int>(hipGetLastError());
}

template <int kQ, int kKind, bool kNT, int kB>
static int launch_fused_q(const FusedArgs& a, hipStream_t s) {
    // one tile of kB * kQ quads per block (at least one block for the ragged
    // tail); the launch holds at most 2^32 - 1 threads, i.e. n < 1.7e10 * kQ
    // elements, beyond what three fp32 arrays fit in HBM
    const int64_t per_block = static_cast<int64_t>(kB) * kQ * 4;
    int64_t tiles = (a.n + per_block - 1) / per_block;
    if (tiles < 1) tiles = 1;
    if (tiles > static_cast<int64_t>(0xFFFFFFFFu / kB)) return static_cast<int>(hipErrorInvalidValue);
    const unsigned grid = static_cast<unsigned>(tiles);
    // Residency.  A block asks for LDS it never touches so that 12 of them,
    // not 32, fit a compute unit: enough loads in flight for HBM's rate, and
    // fewer streams in its way.  Measured on packed arrays (us a step,
    // prepass included; 256-thread blocks without a limit | this block
    // without one | 16 | 13 | 12 | 11 | 10 | 8 a compute unit):
    //   1.63e9 elements   8454 | 7984 | 7710 | 7626 | 7710 | 7695 | 7862 | 8018
    //   1.24e8 elements    662 |  628 |  609 |  591 |  588 |  612 |  597 |  625
    //   1.68e7 elements   85.7 | 86.0 | 82.6 | 80.8 | 80.7 | 81.3 | 82.1 | 86.1
    // What it costs: blocks start at 0.21 ns each, so a skipped step, whose
    // blocks do nothing, takes 106 us for 1.24e8 elements and 1.08 ms for 1.3e9
    // against 43 and 0.40 with 256-thread blocks.  Fewer, larger ones lose more
    // on every step that is not skipped (1.3e9: 5.83 ms; two quads a lane at
    // its best residency 6.02; 128 threads, 6 blocks a compute unit 6.25; 256
    // threads, 3 blocks 6.45; four tiles a block in turn 6.48).
    // Two or four quads a lane (on request) were no better at any of them, and
    // take no limit.  Beside matrix products on another stream, whose blocks
    // want LDS too (ms for all steps | all products, this limit; no limit;
    // 256-thread blocks): 30 steps of 124e6 and 40 products of 4096^3 19.9 |
    // 12.4; 21.3 | 13.2; 23.1 | 14.0, and 6 of 8192^3 20.9 | 5.8; 22.0 | 5.9;
    // 24.3 | 6.0, and 300 of 2048^3 22.7 | 12.4; 23.6 | 17.2; 26.1 | 26.5.
    const unsigned lds = kB == kFusedBlock && kQ == 1 ? kFusedLds : 0u;
    if (a.w != nullptr)
        hipLaunchKernelGGL((fused_kernel<true, kQ, kKind, kNT, kB>), dim3(grid), dim3(kB), lds, s, a);
    else
        hipLaunchKernelGGL((fused_kernel<false, kQ, kKind, kNT, kB>), dim3(grid), dim3(kB), lds, s, a);
    return static_cast<int>(hipGetLastError());
}

// Blocks of 1024 threads (16 wavefronts) only with one quad per lane.
template <int kKind, bool kNT>
static int launch_fused_nt(const FusedArgs& a, hipStream_t s) {
    switch (a.quads_per_thread) {
        case 4: return launch_fused_q<4, kKind, kNT, kFusedBlock>(a, s);
        case 2: return launch_fused_q<2, kKind, kNT, kFusedBlock>(a, s);
        default:
            if (a.block == kFusedWideBlock) return launch_fused_q<1, kKind, kNT, kFusedWideBlock>(a, s);
            // up to two rounds of all wave slots (4.2e6 elements; steps that
            // step_kernel does not take) latency bounds the launch: four times
            // fewer blocks to start, and no residency limit (1.05e6 elements:
            // 8.8 us a step with 256 threads a block, 10.7 with 64; 8.4e6:
            // 44.2 against 40.7)
            return a.n <= 2 * kWaveSlots * int64_t{256} ? launch_fused_q<1, kKind, kNT, kBlock>(a, s)
                                                        : launch_fused_q<1, kKind, kNT, kFusedBlock>(a, s);
    }
}

template <int kB, int kQ, int kKind, int kMode>
static int launch_step_q(const FusedArgs& a, const FinalizeArgs& fa, uint8_t* ws, const Partial* parts, int nparts,
                         int again, hipStream_t s) {
    const int64_t per_block = static_cast<int64_t>(kB) * kQ * 4;
    int64_t tiles = (a.n / 4 * 4 + per_block - 1) / per_block;
    if (tiles < 1) tiles = 1;
    if (kMode == kStepJoint && tiles > kStepMaxTiles) return static_cast<int>(hipErrorInvalidValue);
    const unsigned grid = static_cast<unsigned>(tiles);
    if (a.w != nullptr)
        hipLaunchKernelGGL((step_kernel<true, kB, kQ, kKind, kMode>), dim3(grid), dim3(kB), 0, s, a, fa, ws, parts,
                           nparts, again);
    else
        hipLaunchKernelGGL((step_kernel<false, kB, kQ, kKind, kMode>), dim3(grid), dim3(kB), 0, s, a, fa, ws, parts,
                           nparts, again);
    return static_cast<int>(hipGetLastError());
}

template <int kKind, int kMode>
static int launch_step_n(const FusedArgs& a, const FinalizeArgs& fa, uint8_t* ws, const Partial* parts, int nparts,
                         int again, hipStream_t s) {
    const int64_t quads = a.n / 4, row = static_cast<int64_t>(kStepMaxTiles) * kBlock;
    // at most 256 tiles for the exchange, four partials a lane for the
    // wavefront that polls; beyond 256 tiles of one quad a lane, blocks of 512
    // threads (1.05e6 elements: two quads a lane 9% faster than 256 threads
    // and four).  Without the exchange one quad a lane again as long as three
    // blocks a compute unit hold all (us a step behind a prepass, one quad a
    // lane and two: 1.35e6 elements 12.5 and 13.2, 1.5e6 12.6 and 13.0, 1.65e6
    // 14.5 and 13.4).
    if (quads <= row) return launch_step_q<kBlock, 1, kKind, kMode>(a, fa, ws, parts, nparts, again, s);
    if (quads <= 2 * row || (kMode != kStepJoint && quads > 4 * row && quads <= 6 * row))
        return launch_step_q<2 * kBlock, 1, kKind, kMode>(a, fa, ws, parts, nparts, again, s);
    return launch_step_q<2 * kBlock, 2, kKind, kMode>(a, fa, ws, parts, nparts, again, s);
}

template <int kKind>
static int launch_step_kind(const FusedArgs& a, const FinalizeArgs& fa, int mode, uint8_t* ws, const Partial* parts,
                            int nparts, int again, hipStream_t s) {
    switch (mode) {
        case kStepJoint: return launch_step_n<kKind, kStepJoint>(a, fa, ws, parts, nparts, again, s);
        case kStepAfter: return launch_step_n<kKind, kStepAfter>(a, fa, ws, parts, nparts, again, s);
        default: return launch_step_n<kKind, kStepAlone>(a, fa, ws, parts, nparts, again, s);
    }
}

int launch_step(const FusedArgs& a, const FinalizeArgs& fin, int mode, void* workspace, const void* parts, int nparts,
                int again, void* stream) {
    hipStream_t s = static_cast<hipStream_t>(stream);
    uint8_t* ws = static_cast<uint8_t*>(workspace);
    const Partial* p = static_cast<const Partial*>(parts);
    if (a.n < 1 || a.n > (mode == kStepJoint ? kStepMaxElems : kAfterMaxElems))
        return static_cast<int>(hipErrorInvalidValue);
    return a.grad_kind == kGradFP16 ? launch_step_kind<kGradFP16>(a, fin, mode, ws, p, nparts, again, s)
                                    : launch_step_kind<kGradBF16>(a, fin, mode, ws, p, nparts, again, s);
}

template <int kKind>
static int launch_fused_kind(const FusedArgs& a, hipStream_t s) {
    return a.nt ? launch_fused_nt<kKind, true>(a, s) : launch_fused_nt<kKind, false>(a, s);
}

int launch_fused(const FusedArgs& a, void* stream) {
    hipStream_t s = static_cast<hipStream_t>(stream);
    return a.grad_kind == kGradFP16 ? launch_fused_kind<kGradFP16>(a, s) : launch_fused_kind<kGradBF16>(a, s);
}

}  // namespace gockpt
