// Internal declarations shared by the host side (hop_api.cpp, hop_sim.cpp) and the
// kernels (hop_kernels.hip).  Nothing here is part of the public ABI.
#pragma once

#include <cstdint>
#include <string>
#include <vector>

#include "hop.h"

// ---- device-side job descriptors (plain data, uploaded once per schedule) ----------
struct alignas(16) HopMixJob {
    float* out;
    const float* g;            // null: no gradient term
    float* vel;                // null: no momentum; else v <- mu v + g in place, Apply uses v
    float eta;
    int32_t A;
    float mu;
    float lam_fold;            // with vel: v <- mu v + g + lam_fold * src[0] (the dense part of a sparse gradient)
    const float* src[HOP_MAX_A];
    float w[HOP_MAX_A];
};

constexpr int kMaxGradAhead = 16;
constexpr int HOP_PAIR_U = 12;   // most vectors in the union of a pair of records (the kernel unrolls up to this)

// One or two records of a wave whose source sets overlap, run by one workgroup per column chunk: the union of
// their sources (each loaded once), and per record a membership mask over the union with its weights.  A single
// record may have up to HOP_MAX_A sources; a pair at most 12 in the union.  Records with a velocity keep HopMixJob.
struct alignas(16) HopPairJob {
    int32_t U, G;              // vectors in the union, records (1 or 2)
    float eta;                 // of the records with a gradient
    int32_t reserved;
    float* out[2];
    const float* g[2];         // null: no gradient term
    uint32_t mask[2];          // bit u: the record averages src[u]
    const float* src[HOP_MAX_A];
    float w[2][HOP_MAX_A];     // weight of src[u] in record r (0 where the record does not read it)
};

// What a stand-alone call's kernel argument holds of a pair job: up to HOP_PAIR_U vectors.
struct alignas(8) HopPairArg {
    float* out[2];
    const float* g[2];
    const float* src[HOP_PAIR_U];
    float w[2][HOP_PAIR_U];
    uint32_t mask[2];
    uint8_t U, G;
    float eta;
};
constexpr int kPairArgs = 16;           // of them in the 4 KB of arguments a kernel can have, beside the sizes
static_assert(sizeof(HopPairArg) * kPairArgs <= 4096 - 64, "kernel arguments");

struct alignas(16) HopGradJob {
    // dense: X row-major rows x d; csr: rowptr/col/val
    const float* X;
    const int64_t* rowptr;
    const int32_t* col;
    const float* val;
    const float* y;
    const float* w;            // x_{k,i}: the version the gradient is taken at
    const int32_t* rows;       // B sample ids
    float* g;                  // dense gradient buffer of the worker (dense / synth modes)
    float* coef;               // B hinge coefficients of this record
    float* partial;            // dense: B x nseg partial dot products
    float* out;                // csr: the vector the sparse part is scattered into; dense: if set, the gradient is
                               // applied to it in place (out -= eta g) instead of being written to g
    float* vel;                // with momentum: csr, the velocity the sparse part is scattered into as well;
                               // dense with out set, v <- mu v + g in place and out -= eta v
    const HopMixJob* reduce;   // dense with out set: if set, out = sum_a w'_a x_a - eta g (the gradient kernel does the
                               // record's Reduce too); if null, out already holds the reduced vector
    float eta, mu;             // dense with out set
    uint32_t k0, k1, k2;       // synth: hash keys of (seed, worker, iteration); dense: k0 the loss, for the margins
    float scale;               // synth: fp32 factor
};

// ---- a whole pass as a program ------------------------------------------------------
// The records of a pass, for gradients that need no sum over the columns (none, synthetic, external): every column can then
// run the whole pass by itself.  What they read and where their values are kept, in words of 32 bits; hop_lower_sweep below
// writes it down for the kernel:
//   records  0 flags, 1 local slot of the result, 2 ring slot it is stored to, 3 local slot of the velocity, 4..6 key[]
//            (synthetic: hash keys, the first two folded; external: the worker, and the worker of
//            the next record with a gradient, whose load is issued ahead), 7 number of sources, then (local slot,
//            weight) of every source
//   loads    (ring slot, local slot) of the values read from the rings, then (worker, local slot) of the velocities
constexpr int kSweepHead = 8;
constexpr int kSweepInline = 12;        // most sources of the kernel's chain
constexpr int kSweepMaxLocal = 160;     // most local slots: 184 registers, 2 wavefronts per SIMD
enum : uint32_t { kSweepGrad = 1u, kSweepStore = 2u, kSweepKeep = 4u };
constexpr int hop_sweep_words(int A) { return kSweepHead + 2 * A; }

struct HopSweepOp {                     // one record, in ring-slot terms (host only)
    int out_slot = 0, worker = 0;
    bool grad = false, vel = false, external = false;
    uint32_t key[3] = {0, 0, 0};
    std::vector<std::pair<int, float>> terms;   // (ring slot, weight), in the order the sum is taken
};

struct HopSweepPlan {
    int n_local = 0, n_loads = 0, n_vel = 0;
    int first_load = 0;                         // word
    int first_external = 0;                     // worker of the first record with one
    std::vector<uint32_t> program;
};

// Ops come in an order that respects their dependences.
// False if the pass needs more than kSweepMaxLocal values at a time.  Host only.
bool hop_plan_sweep(const std::vector<HopSweepOp>& ops, int n_ring_slots, int n_workers, HopSweepPlan* plan);

// What sweep_kernel reads: the plan with its local slots as vector registers, in words of 32 bits.
//   records  of kSweepRecord words: 0 where the record enters the kernel's chains of sources (kSweepStep for every source
//            short of kSweepInline; kSweepLong unless it has the gradient of the pass, if there is any, and a result that
//            just goes to a local slot; kSweepOdd for every other record), 1 local slot of the result | flags, 2..4 hash
//            keys or 2..3 address of the external gradient that the next record with one takes, hop_sweep_source(k) and the
//            word behind it: (local slot, weight) of the first source (k = 0), then of the others from the last to the second,
//            15 local slot of the velocity, 30..31 address of the ring slot the result is stored to.  Short records of few
//            sources need the first half only.  More than kSweepInline sources become several records, whose sums go
//            through a local slot of their own.  Behind the last one: a record that enters nowhere, which ends the pass
//   lists    (address, address, local slot, 0) of the vectors loaded at the start, then of those stored back at the end,
//            both filled up to eights by zeros
constexpr int kSweepRecord = 32;
constexpr uint32_t kSweepStep = 8, kSweepLong = 256, kSweepOdd = 512;
constexpr int kSweepRegisters = 168;    // most local slots that the kernel is built for
enum : uint32_t { kSweepWithGrad = 0x200u, kSweepToLocal = 0x400u, kSweepToRing = 0x800u,
                  kSweepNextWhole = 0x1000u };          // flags; the last: the next record needs both halves of its words
constexpr int hop_sweep_source(int k) { return k < 5 ? 5 + 2 * k : 6 + 2 * k; }

struct HopSweepArgs {
    const uint32_t* program = nullptr;  // on the device
    uint64_t first_external = 0;        // address of the external gradient of the first record with one
    int32_t n_records = 0, n_local = 0, n_load_groups = 0, n_store_groups = 0, first_list = 0;
    int32_t mode = 0;                   // HOP_GRAD_ZERO, HOP_GRAD_SYNTH or HOP_GRAD_EXTERNAL
    int32_t velocities = 0;             // a context with velocities
    float eta = 0.f, mu = 0.f, scale = 0.f;
    int64_t d = 0;
};

// The vectors that a plan's numbers stand for.
struct HopSweepVectors {
    const float *ring = nullptr, *vel = nullptr, *external = nullptr;
    int64_t stride = 0, d = 0;
};
// Writes the plan down for the kernel; sets the counts of `args`.  Host only.
void hop_lower_sweep(const HopSweepPlan& plan, int n_ops, const HopSweepVectors& at, HopSweepArgs* args, std::vector<uint32_t>* words);

// Packs the Reduce jobs of one wave for pair_mix_kernel (appends to `out`; see its definition for the rule); returns the
// number of distinct vectors the jobs read.  Host only.
int hop_pack_pairs(const HopMixJob* jobs, int n, std::vector<HopPairJob>& out);

// ---- kernel launchers (hop_kernels.hip); all return a hipError_t as int ------------
int hopk_mix(const HopMixJob* jobs_dev, int n_jobs, int64_t d, void* stream);
int hopk_synth(const HopGradJob* jobs_dev, int n_jobs, int reverse, int64_t d, void* stream);
int hopk_dense_margin(const HopGradJob* jobs_dev, int n_jobs, int B, int64_t d, void* stream);
int hopk_csr_margin(const HopGradJob* jobs_dev, int n_jobs, int B, int loss, void* stream);
int hopk_mix_dense_margin(const HopMixJob* mix_dev, int n_mix, int64_t d, const HopGradJob* grad_dev, int n_grad, int B,
                          void* stream);
int hopk_mix_csr_margin(const HopMixJob* mix_dev, int n_mix, int64_t d, const HopGradJob* grad_dev, int n_grad, int B,
                        int loss, void* stream);
// n_sources: distinct vectors the jobs read (sizes the XCD runs); reverse: walk the vectors from their end
int hopk_pair(const HopPairJob* jobs_dev, int n_jobs, int n_sources, int reverse, int64_t d, void* stream);
int hopk_pair_dense_margin(const HopPairJob* mix_dev, int n_mix, int n_sources, int reverse, int64_t d,
                           const HopGradJob* grad_dev, int n_grad, int B, void* stream);
// out += factor c_m x_m over the active rows; into_velocity: vel -= c_m x_m too
int hopk_csr_scatter(const HopGradJob* jobs_dev, int n_jobs, int B, float factor, int into_velocity, void* stream);
int hopk_csr_check(const int64_t* rowptr, const int32_t* col, int64_t rows, int64_t first, int64_t nnz, int64_t d,
                   int* flag_dev, void* stream);
int hopk_copy(void* dst, const void* src, size_t bytes, void* stream);
// weak, so that the host files still link for checks that stub the launchers above and never reach a device
__attribute__((weak)) int hopk_pair_csr_margin(const HopPairJob* mix_dev, int n_mix, int n_results, int n_sources, int reverse, int64_t d,
                                               const HopGradJob* grad_dev, int n_grad, int B, int loss, void* stream);
__attribute__((weak)) int hopk_sweep(const HopSweepArgs& args, void* stream);
// one gradient written to job.g (HOP_GRAD_SVM_CSR: to job.out); the Reduce of a call's records in any number of jobs, and in up to
// kPairArgs jobs with descriptors on the host
__attribute__((weak)) int hopk_one_grad(const HopGradJob& job, int mode, int B, int64_t d, float lambda, int loss, void* stream);
__attribute__((weak)) int hopk_pair_alone(const HopPairJob* jobs_dev, int n_jobs, int n_results, int n_sources, int64_t d, void* stream);
__attribute__((weak)) int hopk_pair_args(const HopPairArg* jobs, int n_jobs, int n_sources, int64_t d, void* stream);
// rows_again: later waves read the same rows while a cache may still hold them (hop_rows_again)
__attribute__((weak)) int hopk_dense_grad(const HopGradJob* jobs_dev, int n_jobs, int B, int64_t d, float lambda, int loss, bool rows_again,
                                          void* stream);
int hopk_dense_nseg(int64_t d);                 // column segments per row in the margin pass

// ---- rules of a launch ---------------------------------------------------------------
// Vectors that the next launches find in the L2s: where the jobs of a launch come to no more than the 32 MB of all of them, results are
// stored like any other data (else non-temporally, so that they push nothing out), and a chunk of columns goes to the same XCD in
// every launch: runs of one chunk, always from the front.  us, without and with: a pass of 16 workers x 300 000 columns, sparse,
// 373 / 312; 16 x 2^20 (18 MB a wave) 2733 / 2500; wave by wave with external gradients 16 x 300 000 253 / 204, 32 x 150 000 322 / 257.
// Beyond, records that run singly: 16 x 4 M 1370 / 1440, 32 x 2 M (72 MB a wave) 1613 / 1665.  A pair counts once, so waves of pairs stay
// up to 64 MB: lock-step rings, tori and rings with chords of 4 to 64 workers that write 34 to 63 MB, 24 sizes each: external gradients
// 404 / 368 (4 workers, 34 MB) to 739 / 668 (64, 63 MB), sparse 404 / 309 (16, 34 MB) to 747 / 542 (64, 63 MB).
constexpr int64_t kNearBytes = 32ll << 20;
// `vectors` that go with a job: with a velocity its own share is written and read between, which counts as three (16 x 300 000,
// sparse, 419 / 402; 64 x 500 000 1357 / 1375).
inline bool hop_stays_near(int n_jobs, int64_t d, int vectors = 1) { return vectors * n_jobs * d * (int64_t)sizeof(float) <= kNearBytes; }

// A stand-alone average of uploaded jobs, past the L2s -> near, us a call: records of 13 sources, which run singly, 16 x 60 000 columns 47.7 ->
// 47.2, 16 x 240 000 (15 MB) 57.5 -> 56.4, 64 x 60 000 (15 MB) 89.9 -> 87.1, 16 x 350 000 (21 MB) 64.6 -> 69.7, 16 x 480 000 74.0 -> 80.5, 64 x 120 000
// 108.7 -> 111.8; 64 records in pairs, 60 000 columns (15 MB) 69.1 -> 70.8, 80 000 72.0 -> 73.5, 240 000 91.3 -> 90.5.  With velocities, which a
// call brings back into the L2s to write them, the rule of the waves: 17 sizes of 4 to 32 MB 1.4 % faster, the most 1.4 % slower.
inline bool hop_near_alone(int n_jobs, int n_results, int64_t d) { return n_jobs == n_results && hop_stays_near(n_jobs, d, 2); }

// Results that the gradient kernel of the same wave finishes in place stay near further: it reads them next.  Near against past the L2s by
// what the records with a gradient write, geometric means of 2 to 16 runs of 24 to 144 workers each: without velocities 30 to 50 MB 0.95, 70 to 90
// 0.96, 90 to 110 0.99, 127 to 160 1.03, 160 to 300 1.02 (64 workers x 200 000 columns 616 -> 615 us per pass, 64 x 330 000 1102 -> 1029, 144 x 524 288
// 4583 -> 4674); with velocities 30 to 50 MB 0.95, 70 to 110 1.00, 110 to 127 1.02, 127 to 160 1.04, 160 to 300 1.01 (32 x 330 000 684 -> 626, 100 x
// 400 000 2949 -> 3034).
constexpr int64_t kInPlaceNear = 96ll << 20;
inline bool hop_in_place_near(int n_records, int64_t d) { return n_records * d * (int64_t)sizeof(float) <= kInPlaceNear; }

constexpr int64_t kMemorySideCache = 256ll << 20;
constexpr int64_t kDenseInPlaceBytes = 2 << 20; // rows of a minibatch up to which its margins run beside the Reduce
// Whether the columns of a pass's dense minibatches may be dealt out to the 8 XCDs in slices.  The partial products, 8 a row, are in
// the worker's gradient buffer, which dense passes have no other use for.  us per pass of 4 / 16 / 64 workers without and with:
// B = 64, d = 12 000 211 / 699 / 1863 -> 179 / 585 / 1630; B = 64, d = 20 000 260 / 979 / 3132 -> 216 / 746 / 2421; B = 128, d = 65 536
// 556 / 2130 / 9528 -> 495 / 1964 / 9350.  Below, against margins beside the Reduce: B = 32, d = 10 000 143 / 412 / 938 -> 149 / 417 / 964,
// d = 7000 138 / 368 / 776 -> 140 / 384 / 862; against margins by themselves (over 2 MB): B = 100, d = 8000 193 / 574 / 1491 -> 162 / 510 /
// 1384, B = 128, d = 5000 163 / 484 / 1253 -> 161 / 498 / 1384.  Above, a slice would be more than a segment.
inline bool hop_dense_slices(int B, int64_t d) {
    return d <= 8 * 16384 && 8 * (int64_t)B <= d && d > ((int64_t)B * d * 4 > kDenseInPlaceBytes ? 7168 : 11264);
}

// Whether a wave of such minibatches is.  The more rows it has, the less of them the L2s hold until the gradient reads them again, and
// every workgroup of the gradient adds up 8 partial products a row, where rows of one segment have their coefficients worked out.
// us per pass, in slices -> in segments, log loss, rows of a wave = records x B: 7200 columns: 32 x 100 221 -> 239, 32 x 160 364 -> 339,
// 16 x 400 390 -> 337 (with a velocity); 8700: 8 x 400 391 -> 422, 64 x 64 383 -> 358, 32 x 800 2847 -> 2423; 10 000: 32 x 100 281 -> 304, 64 x 64
// 420 -> 405, 8 x 600 632 -> 601; 12 000: 16 x 300 388 -> 391, 32 x 300 1269 -> 1217; 13 000: 64 x 64 488 -> 496, 100 x 100 1154 -> 1124; 16 000: 64 x
// 100 807 -> 846, 32 x 200 1082 -> 1141, 32 x 600 3203 -> 3111; 24 000 (two segments): 32 x 600 4652 -> 4915.
inline bool hop_wave_slices(int n_jobs, int B, int64_t d) {
    const int64_t rows = (int64_t)n_jobs * B;
    return hop_dense_slices(B, d) && rows <= (d <= 11264 ? 3500 : d <= 14336 ? 6000 : INT64_MAX);
}

// Whether a wave's dense minibatches keep to one XCD each: up to kOneXcdBytes of rows of kOneXcdCols columns in launches of few column
// chunks.  us per pass of 4 / 16 / 64 workers, all XCDs -> one: B = 64, d = 1024 108 / 326 / 543 -> 101 / 301 / 485; B = 200,
// d = 1024 151 / 435 / 892 -> 145 / 401 / 781; B = 128, d = 4096 (2 MB, half of an L2) 142 / 436 / 1039 -> 141 / 427 / 999; B = 32, d = 8000
// 150 / 410 / 898 -> 153 / 402 / 863; but B = 32, d = 10 000 143 / 412 / 938 -> 147 / 423 / 914, d = 16 000 167 / 549 / 1231 -> 182 /
// 593 / 1236: an XCD is busy with some 32 chunks of 256 columns of a record.  Waves of up to five records at 7500 to 8192 columns: hinge
// loss 4 % slower on one, log loss 1 to 20 % faster.
// With one or two records most XCDs idle while one reads all rows.  12 iterations of 1 worker, hinge / log loss, 1000 columns: B = 100
// 78 / 87 -> 73 / 82, B = 200 89 / 107 -> 90 / 106, B = 240 94 / 115 -> 101 / 120, B = 400 119 / 154 -> 133 / 160; of 2 workers: B = 200 100 /
// 121 -> 99 / 112, B = 240, 2048 columns 112 / 133 -> 121 / 137, B = 400 136 / 166 -> 142 / 165; of 3: B = 400 142 / 171 -> 146 / 168, of 4:
// 157 / 184 -> 150 / 170.
constexpr int64_t kOneXcdBytes = 2 << 20, kOneXcdCols = 8192, kGradFew = 768;
constexpr int kOneXcdRows = 200;
inline bool hop_one_xcd(int n_jobs, int B, int64_t d) {
    return d <= kOneXcdCols && (int64_t)B * d * 4 <= kOneXcdBytes && n_jobs * ((d + 255) / 256) <= kGradFew && (n_jobs > 2 || B <= kOneXcdRows);
}
// A stand-alone call, whose margins have a launch of their own, takes one XCD with any number of rows.  us, all XCDs -> one, rows warm / cold:
// B = 64, d = 1024 8.6 / 7.7 -> 7.9 / 7.0, B = 128, d = 4096 8.5 / 7.6 -> 8.1 / 7.5, B = 64, d = 8192 8.6 / 7.4 -> 8.0 / 7.3, with synchronisation
// (B = 32, d = 8000) 18.1 / 19.3 -> 16.8 / 18.2; up to 512 columns B = 300 to 500 4 to 6 % faster, 600 to 1000 the same within 2 %.
inline bool hop_one_xcd_alone(int B, int64_t d) { return d <= kOneXcdCols && (int64_t)B * d * 4 <= kOneXcdBytes; }

// Whether the second and last reading of a record's rows, by its gradient kernel in slices, leaves them in the caches.  Non-temporal
// loads there keep more of what is yet to be read in the L2s (us per pass, log loss, 32 minibatches of data: 8 workers x 20 000 columns,
// B = 128, 262 -> 236; 16 x 65536, B = 64, 790 -> 745), but the next waves then find less of rows that come again: where all data sets
// fit the memory-side cache (160 rows: 8 x 20 000, B = 128, 176 -> 188; 16 x 12 000 294 -> 307), or each holds at most two minibatches
// (128 rows: 16 x 65536, B = 64, 628 -> 680).  With four: 16 x 65536, B = 64, 685 -> 702, 8 x 30 011, B = 100, 406 -> 389.  Waves whose rows
// the L2s hold find them there anyway (8 x 11 500, two and six minibatches: 18 MB 98 -> 97 and 108 -> 105, 22 MB 112 -> 110 and 121 -> 117, 30 MB
// 128 -> 133 and 140 -> 142; 76 sizes of 6 to 22 MB 0.3 % faster past the caches, 16 of 30 MB 1.6 % slower, 36 MB 4 %).
constexpr int64_t kRowsNear = 24ll << 20;       // bytes of rows of a wave
// Not in slices rows are always read by ordinary loads: 2 x 131 073, B = 64, 128 and 2048 rows 255 -> 220, 278 -> 278; 1 x 600,
// B = 1024, 32 768 rows 257 -> 201; 7 x 6283, B = 194, 1552 rows 238 -> 222.
inline bool hop_rows_again(int B, int64_t least_rows, int64_t all_bytes) {
    return least_rows <= 2 * (int64_t)B || all_bytes <= kMemorySideCache;
}

// ---- host-side random numbers (hop_sim.cpp) ---------------------------------------
namespace hoprng {
enum : uint64_t { STREAM_DELAY = 1, STREAM_BATCH = 2, STREAM_SYNTHGRAD = 6, STREAM_LATENCY = 7 };
uint64_t mix(uint64_t seed, uint64_t stream, uint64_t a, uint64_t b, uint64_t c);
void synth_keys(uint64_t seed, int worker, int iter, uint32_t* k0, uint32_t* k1, uint32_t* k2);
float synth_scale(float variance);
}  // namespace hoprng

// ---- schedule ----------------------------------------------------------------------
struct hop_schedule {
    int N = 0, D = 0, K = 0, batch = 0, stalled = 0, n_jumps = 0, n_waves = 0, late_sends = 0;   // D: slots per worker in memory
    std::vector<int32_t> kind, worker, iter, wave, out_slot, src_begin, src_worker, src_tag, src_slot;
    std::vector<uint64_t> time;
    std::vector<float> src_weight;
    std::vector<int32_t> batch_rows, final_iter, wave_begin, wave_order;
    std::vector<uint64_t> finish_time;
    std::vector<int64_t> rows_at_sim;   // data-set sizes the minibatch ids were drawn for

    // device side: descriptors laid out by hop_step, for the context's current gradient mode, inside the
    // workspace the caller lent with hop_schedule_bind (the library allocates no device memory for a schedule)
    hop_ctx* owner = nullptr;
    char* workspace = nullptr;
    size_t workspace_bytes = 0;
    int built_mode = -1;
    uint64_t built_epoch = 0;
    HopMixJob* mix_dev = nullptr;       // n_records, in wave order
    HopPairJob* pair_dev = nullptr;     // the same records packed in pairs, wave by wave (null with a velocity)
    HopGradJob* grad_dev = nullptr;     // STEP records only, in wave order
    HopSweepArgs sweep;                 // the whole pass as one launch (program null: not available for this schedule)
    int32_t* rows_dev = nullptr;        // n_records x batch
    float* coef_dev = nullptr;          // n_records x batch
    bool dense_in_place = false;        // dense SVM: margins beside the Reduce, gradient applied in place
    bool dense_rows_again = false;      // dense SVM: its minibatches come from few or small data, see hop_rows_again
    std::vector<int32_t> grad_begin;    // n_waves + 1 offsets into grad_dev
    std::vector<int32_t> pair_begin;    // n_waves + 1 offsets into pair_dev
    std::vector<int32_t> wave_sources;  // distinct vectors each wave reads
    std::vector<int32_t> wave_mix_jobs; // records in each wave's mix launch (its first descriptors; the rest, if any,
                                        // are reduced by their gradient kernel)
    std::vector<double> wave_mix_bytes; // algorithmic bytes of each wave's mix launch
    std::vector<double> wave_grad_bytes;
    void* graph_exec = nullptr;         // hipGraphExec_t of waves [0, n_waves), see hop_use_graph()
    uint64_t graph_epoch = 0;
    int graph_mode = -1;
};

// ---- context -----------------------------------------------------------------------
struct HopData {
    int64_t rows = 0;
    const float* X = nullptr;
    const int64_t* rowptr = nullptr;
    const int32_t* col = nullptr;
    const float* val = nullptr;
    const float* y = nullptr;
};

struct HopProfile {
    std::vector<void*> ev;              // pairs of hipEvent_t, recycled
    std::vector<int> pending_kernel;    // kernel id of each recorded pair
    std::vector<double> pending_bytes;
    double ms[HOP_KERNEL_COUNT] = {0, 0, 0};
    int64_t launches[HOP_KERNEL_COUNT] = {0, 0, 0};
    double bytes[HOP_KERNEL_COUNT] = {0, 0, 0};
};

struct hop_ctx {
    int N = 0, s = 0, b = 0, D = 0, max_ig = 0;
    int slots = 0;                      // slots per worker in memory: D, plus the current-parameter slot D when serial
    int64_t d = 0, stride = 0;
    hop_opts opts{};
    std::vector<std::vector<int>> in_nbrs, out_nbrs;
    std::vector<float> W;               // N x N, W[j*N+i]
    // device
    bool has_device = false;
    char* arena = nullptr;
    size_t arena_bytes = 0;
    void* stream = nullptr;
    float* ring = nullptr;              // N x D x stride
    float* gbuf = nullptr;              // N x grad_ahead x stride
    int grad_ahead = 1;                 // gradient buffers per worker (hop_opts.grad_ahead, at least 1)
    float* partial = nullptr;           // N x batch x nseg
    float* vel = nullptr;               // N x stride velocities, only with momentum
    std::vector<HopData> data;
    int grad_mode = HOP_GRAD_ZERO;
    float synth_variance = 0.f;
    const float* external = nullptr;
    uint64_t epoch = 0;                 // bumped whenever job descriptors would change
    std::vector<int32_t> version;       // newest iteration held per worker
    std::vector<hop_schedule*> schedules;   // live schedules of this context (hop_simulate .. hop_schedule_free)
    const hop_schedule* running = nullptr;
    int next_wave = 0;
    bool profiling = false;
    bool use_graph = false;
    void* capture_stream = nullptr;     // library-owned stream used only to record graphs
    HopProfile prof;
    std::string last_error;
};

int hop_run_protocol(const hop_ctx* ctx, const hop_delay_model* dm, int K, hop_schedule* out);
