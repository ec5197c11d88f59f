// gockpt_internal.h -- layouts shared by the runtime and the kernels.
#pragma once

#include <stdint.h>
#include <stddef.h>

#include "../../include/gockpt.h"
#include "gockpt_contract.h"

namespace gockpt {

constexpr int kBlock = 256;             // threads per block, 4 wavefronts
constexpr int kFusedBlock = 64;         // threads per block of the fused kernel, one wavefront
constexpr int kFusedWideBlock = 1024;   // the fused kernel's optional wide block, 16 wavefronts
constexpr int kWaveSlots = 256 * 32;     // wavefronts the device holds at once
constexpr unsigned kFusedLds = 13312;   // LDS of a fused block under the residency limit: 12 blocks a compute unit
constexpr int kVec = 8;                 // elements per thread per group
// Loads a lane of the prepass and of a bucket scan keeps in flight beside the
// current ones.  A scan beside the backward has one block a compute unit, so
// memory latency bounds it: with 8 buckets of 15.6e6 elements 632 us a step
// with one load, 617 with four, 618 with eight (350e6 elements: 1800, 1718,
// 1721).  The prepass fills the device: one, two, four or eight loads are
// within 1% from 8.4e6 elements on; below, two were 3% faster (2.1e6: 15.0,
// 14.5, 15.0, 16.4 us a step).
constexpr int kPrepassAhead = 2;
constexpr int kScanAhead = 4;
// Above this many gradient bytes the prepass and the scans read with the
// nontemporal hint (see create_ctx).
constexpr int64_t kCachedGradBytes = 512 << 20;
constexpr int kPrepassMaxBlocks = 2048; // partial sums slots
constexpr int kScanSlots = 8192;        // partials of the bucket scans of one step
constexpr int kScanMaxBlocks = 256;     // blocks of a bucket scan beside the backward (one per compute unit)

// Device-resident loss-scaler state (workspace offset 0).
struct alignas(64) DevScaler {
    int64_t t;
    int64_t tracker;
    float scale;
    int32_t pad0;
    int64_t pad1[5];
};
static_assert(sizeof(DevScaler) == 64, "DevScaler");

// Per-block partial of the prepass.
struct alignas(16) Partial {
    double sumsq;
    int32_t nonfinite;
    int32_t pad;
};
static_assert(sizeof(Partial) == 16, "Partial");

// One-launch steps (step_kernel): the tag of the next one's partials, and how
// many blocks of the running one have read the state (each in one of
// kStepArriveLanes counters, a line apart, and each full counter in `arrived`).
struct alignas(64) StepSync {
    uint32_t epoch;
    uint32_t arrived;
    uint32_t helped;  // partials computed again for want of their block's, over the context's life
    uint32_t pad[13];
};
static_assert(sizeof(StepSync) == 64, "StepSync");
struct alignas(256) StepArrive {
    uint32_t count;
};
constexpr int kStepArriveLanes = 16;
constexpr int kStepMaxTiles = 256;  // four partials a lane of the wavefront that reads them
static_assert(kStepMaxTiles % 64 == 0, "whole rows of a wavefront");
constexpr int64_t kStepMaxElems = int64_t{kStepMaxTiles} * 512 * 2 * 4 + 3;  // two quads a lane, and the tail
// Steps in one launch behind a prepass, or with nothing to sum: where the whole
// step could be one, and from kAfterMinElems to kAfterMaxElems.  Between them
// there are more blocks than compute units and too few to even that out, and
// the separate kernels' smaller ones are as fast or faster (us a step separate
// and in one launch, each at its best shape: behind a prepass 1.05e6 elements
// 10.6..12.1 and 11.9, 1.2e6 11.6..12.3 and 12.4, 1.35e6 13.2 and 12.5, 1.5e6
// 13.6 and 12.6; alone 8.1 and 8.7, 8.7 and 9.4, 10.3 and 9.5, 10.9 and 9.6).
// Behind bucket scans one launch is the faster one there too (13.0 and 11.8,
// 13.2 and 12.2 for 1.05e6 and 1.2e6).
constexpr int64_t kAfterMinElems = 5 << 18;
constexpr int64_t kAfterMaxElems = int64_t{1} << 22;
constexpr int kAfterMaxParts = 512;  // partials every block then reduces: 8 KiB from the L2
constexpr int kStepHelpSpins = 32;  // polls (0.5 to 1 us each) before a block computes the partials it misses

static_assert(sizeof(gockpt_step_record) == 64, "record size");

// Workspace layout: [DevScaler | pad to 256][records: (MAX_K+1) x 64]
// [prepass partials][bucket-scan partials: two banks, alternating by step,
// so the scans of the next step never overwrite what this step's finalize
// still has to read]
// The one-launch step keeps its sync words in the first pad, and its slots and
// counters in the second half of the prepass partials: a space of at most
// kAfterMaxElems, whatever form its steps take, has at most kAfterMaxParts
// prepass blocks (prepass_blocks_for).
constexpr size_t kWsScalerOff = 0;
constexpr size_t kWsSyncOff = 64;
constexpr size_t kWsRecordsOff = 256;
constexpr size_t kWsPartialsOff = kWsRecordsOff + (GOCKPT_MAX_K + 1) * sizeof(gockpt_step_record);
constexpr size_t kWsScanOff = kWsPartialsOff + kPrepassMaxBlocks * sizeof(Partial);
// 256-byte aligned, as the workspace is
constexpr size_t kWsSlotsOff = (kWsPartialsOff + kPrepassMaxBlocks / 2 * sizeof(Partial) + 255) / 256 * 256;
constexpr size_t kWsArriveOff = kWsSlotsOff + kStepMaxTiles * sizeof(uint64_t);
constexpr size_t kWsStepEnd = kWsArriveOff + kStepArriveLanes * sizeof(StepArrive);
static_assert(kWsSyncOff + sizeof(StepSync) <= kWsRecordsOff, "sync words");
static_assert(kWsArriveOff % 256 == 0 && kWsStepEnd <= kWsScanOff, "slots and counters");

// Blocks of the prepass, one group of a lane each as far as they go.  Up to
// kAfterMaxElems at most kAfterMaxParts, also where a finalize of its own
// reduces them (HOST_WAIT, timed windows): another step of the same context
// ends in one launch, and its counters lie behind these partials.
constexpr int prepass_blocks_for(int64_t n) {
    const int64_t most = n <= kAfterMaxElems ? kAfterMaxParts : kPrepassMaxBlocks;
    const int64_t b = (n / kVec + kBlock - 1) / kBlock;
    return static_cast<int>(b < 1 ? 1 : (b > most ? most : b));
}
static_assert(kWsPartialsOff + prepass_blocks_for(kAfterMaxElems) * sizeof(Partial) <= kWsSlotsOff &&
                  kStepMaxElems <= kAfterMaxElems,
              "slots and counters beside the partials");
constexpr size_t kWsBytes = kWsScanOff + 2 * kScanSlots * sizeof(Partial);

// Page-locked, host-coherent control page of a context (4 KiB).  The device
// writes each window step's skip decision there (finalize), and gate kernels
// on the copy stream read how many staged copies the host has moved out of
// their staging slots.
struct alignas(64) CtrlPage {
    uint64_t released;      // staged copies whose slot is free again, in copy order (host writes)
    uint64_t pad0[7];
    uint32_t gate_timeout;  // a gate kernel gave up waiting (device writes 1)
    uint32_t pad1[15];
    int32_t skip[GOCKPT_MAX_K + 1];  // finalize: skip decision of window step s (device writes)
};
static_assert(sizeof(CtrlPage) <= 4096, "control page");

// Loss-scaler settings the finalize needs.
struct ScalerCfg {
    int32_t check_overflow;
    int32_t dynamic_scale;
    float growth_factor;
    float backoff_factor;
    float min_scale;
    int32_t pad;
    int64_t growth_interval;
};

// Which elements one step packs into the ring, and where.  The step's pack
// list is [grads of elements 0..gb) | master, exp_avg, exp_avg_sq of the
// chunk [cb, ce)].  A prefix of that list goes to the ring; the rest is copied
// straight from the live buffers.  Elements [0, g_end) of the gradients and
// [cb, s_end[k]) of state array k go to the ring, at ring byte offsets
// (physical, < ring_bytes) off_g + 2*i and off_s[k] + 4*(i - cb), taken
// modulo ring_bytes.
struct PackPlan {
    int64_t g_end;
    int64_t cb;
    int64_t s_end[3];
    uint64_t off_g;
    uint64_t off_s[3];
    uint8_t* ring;
    uint64_t ring_bytes;
    int32_t ring_nt;      // 1: nontemporal ring stores
    int32_t any;          // 0: the step packs nothing (the ranges above are empty)
};

struct FusedArgs {
    float* p;
    float* m;
    float* v;
    uint16_t* w;
    const uint16_t* g;
    int64_t n;
    const gockpt_step_record* rec;  // this step's record (skip, scalars)
    float b1, b2, omb1, omb2, eps;  // step-independent scalars
    int32_t quads_per_thread;       // 1, 2 or 4 quads (4 elements) per thread
    int32_t grad_kind;              // kGradBF16 or kGradFP16
    int32_t nt;                     // nontemporal state loads and stores
    int32_t block;                  // kFusedWideBlock (one quad per lane), or kFusedBlock: kBlock threads a block up
                                    // to 4.2e6 elements, kFusedBlock above (launch_fused_nt)
    PackPlan pack;
};

// The copies of one window step of at most kGatherMaxBytes, queued as one
// kernel (gather_kernel) instead of one DMA transfer each.  The kernel was the
// faster one at every size measured (to the drain of a 4-step window with
// 2.4 MB a step 272 us against 453, 9.4 MB 742 against 881), but it runs on
// compute units and its stores to the link hold up what runs beside it (a
// matrix product by half while it lasts), so it gets at most 1 MiB: 18 us.
//
// The ranges: the record, four in the ring, one of which may wrap, and four of
// the live buffers.
constexpr uint64_t kGatherMaxBytes = 1 << 20;
constexpr int kGatherSegs = 12;
constexpr uint64_t kGatherBlocks = 16;  // blocks per range
struct GatherArgs {
    struct {
        const uint8_t* src;  // device, 16-byte aligned
        uint8_t* dst;        // device address of pinned host memory, 16-byte aligned
        uint64_t bytes;
    } seg[kGatherSegs];
};

// Launch-shape choices of a context (fixed at create).
struct Knobs {
    int quads_per_thread;  // fused kernel: quads of 4 elements per thread
    int ring_nt;      // nontemporal ring stores
    int prepass_nt;   // nontemporal gradient loads in the prepass and the scans; -1: by size
    int fused_nt;     // nontemporal loads and stores of the state in the fused kernel
    int fused_block;  // fused kernel threads per block: kFusedBlock (default) or kFusedWideBlock
    bool defaults;    // none of the above asked for otherwise
    int step_again;   // one-launch step: every block computes all partials again (GOCKPT_TEST_STEP_AGAIN)
};

// What the finalize of one step needs besides the partials.
struct FinalizeArgs {
    int32_t raw;        // partials hold squares of the scaled gradients (bucket scans)
    int32_t norm_off;
    const float* found_inf;
    int32_t slot;       // record slot (window step s, 0 outside a window)
    int32_t window_step;
    float lr;
    int32_t pad;
    HParams hp;
    ScalerCfg sc;
    int32_t* skip_out;  // host-coherent slot for this step's skip decision, or null
};

// Launchers (gockpt_kernels.hip).  All stream-ordered, no host sync.
// A new context's workspace: the loss-scaler state, and the words of the
// one-launch step cleared.
int launch_init(void* workspace, int64_t t, int64_t tracker, float scale, void* stream);
int launch_prepass(const uint16_t* g, int64_t n, void* workspace, int nblocks, int nt, int grad_kind, void* stream);
// parts: the partials to reduce (nparts of them, in order); raw: they hold
// squares of the scaled gradients (bucket scans), which the finalize unscales.
int launch_finalize(void* workspace, const void* parts, int nparts, const FinalizeArgs& fin, void* stream);
// Copies nseg ranges to pinned host memory in one launch.
int launch_gather(const GatherArgs& a, int nseg, void* stream);
// One wavefront on `stream` that waits until *released >= target (host-
// coherent memory the host advances), at most max_ticks of the 100 MHz
// constant clock; on giving up it sets *timed_out.
int launch_gate(const uint64_t* released, uint64_t target, uint64_t max_ticks, uint32_t* timed_out, void* stream);
int launch_scan(const uint16_t* g, int64_t begin, int64_t end, void* parts, int nblocks, int nt, int grad_kind,
                void* stream);
int scan_blocks_for(int64_t count, int max_blocks);
int launch_fused(const FusedArgs& a, void* stream);
// The step in one launch (see step_kernel).  kStepJoint: 1 <= n <=
// kStepMaxElems; the others: 1 <= n <= kAfterMaxElems, parts with kStepAfter.
enum StepMode : int { kStepAlone = 0, kStepJoint = 1, kStepAfter = 2 };
int launch_step(const FusedArgs& a, const FinalizeArgs& fin, int mode, void* workspace, const void* parts, int nparts,
                int again, void* stream);
Knobs default_knobs();

}  // namespace gockpt
