// What a pass launches, on the CPU: hop_api.cpp with a HIP runtime of plain memory and launchers that print their arguments.
//   launch_driver dense|csr|skipping|external|complete WORKERS COLUMNS BATCH ROWS MOMENTUM
//   launch_driver rules RECORDS COLUMNS BATCH
//   launch_driver average RECORDS COLUMNS SOURCES MOMENTUM
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include <hip/hip_runtime_api.h>

#include "hop_internal.h"

extern "C" {
hipError_t hipMemcpy(void* to, const void* from, size_t n, hipMemcpyKind) { std::memcpy(to, from, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }   // parameters: not looked at
hipError_t hipMemset(void* p, int v, size_t n) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return ""; }
hipError_t hipEventCreate(hipEvent_t*) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float*, hipEvent_t, hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t*, unsigned) { return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
}

int hopk_mix(const HopMixJob*, int n, int64_t, void*) { std::printf("mix jobs=%d\n", n); return 0; }
int hopk_synth(const HopGradJob*, int n, int, int64_t, void*) { std::printf("synth jobs=%d\n", n); return 0; }
int hopk_dense_margin(const HopGradJob*, int n, int, int64_t, void*) { std::printf("dense_margin jobs=%d\n", n); return 0; }
int hopk_dense_grad(const HopGradJob*, int n, int, int64_t, float, int, bool again, void*) {
    std::printf("dense_grad jobs=%d rows_again=%d\n", n, (int)again);
    return 0;
}
int hopk_csr_margin(const HopGradJob*, int n, int, int, void*) { std::printf("csr_margin jobs=%d\n", n); return 0; }
int hopk_mix_dense_margin(const HopMixJob*, int n, int64_t, const HopGradJob*, int g, int, void*) {
    std::printf("mix_dense_margin jobs=%d gradients=%d\n", n, g);
    return 0;
}
int hopk_mix_csr_margin(const HopMixJob*, int n, int64_t, const HopGradJob*, int g, int, int, void*) {
    std::printf("mix_csr_margin jobs=%d gradients=%d\n", n, g);
    return 0;
}
int hopk_pair(const HopPairJob*, int n, int, int, int64_t, void*) { std::printf("pair jobs=%d\n", n); return 0; }
int hopk_pair_alone(const HopPairJob*, int n, int results, int, int64_t d, void*) {
    std::printf("pair_alone jobs=%d results=%d near=%d\n", n, results, hop_near_alone(n, results, d));
    return 0;
}
int hopk_pair_args(const HopPairArg*, int n, int, int64_t, void*) { std::printf("pair_args jobs=%d\n", n); return 0; }
int hopk_pair_csr_margin(const HopPairJob*, int n, int results, int, int, int64_t, const HopGradJob*, int g, int, int, void*) {
    std::printf("pair_csr_margin jobs=%d results=%d gradients=%d\n", n, results, g);
    return 0;
}
int hopk_pair_dense_margin(const HopPairJob*, int n, int, int, int64_t, const HopGradJob*, int g, int, void*) {
    std::printf("pair_dense_margin jobs=%d gradients=%d\n", n, g);
    return 0;
}
int hopk_csr_scatter(const HopGradJob*, int n, int, float, int, void*) { std::printf("csr_scatter jobs=%d\n", n); return 0; }
int hopk_csr_check(const int64_t*, const int32_t*, int64_t, int64_t, int64_t, int64_t, int*, void*) { return 0; }
int hopk_copy(void*, const void*, size_t, void*) { return 0; }
int hopk_sweep(const HopSweepArgs&, void*) { std::printf("sweep\n"); return 0; }
int hopk_dense_nseg(int64_t d) { return (int)((d + 16383) / 16384); }

static void* aligned(std::vector<char>& m, size_t n) {
    m.resize(n + 256);
    return m.data() + (256 - (uintptr_t)m.data() % 256) % 256;
}

int main(int argc, char** argv) {
    if (argc == 5) {
        const int n = std::atoi(argv[2]), B = std::atoi(argv[4]);
        const int64_t d = std::atoll(argv[3]);
        std::printf("rules one_xcd=%d one_xcd_alone=%d slices=%d wave_slices=%d near=%d near_velocity=%d in_place=%d\n", hop_one_xcd(n, B, d),
                    hop_one_xcd_alone(B, d), hop_dense_slices(B, d), hop_wave_slices(n, B, d), hop_stays_near(n, d), hop_stays_near(n, d, 3),
                    hop_in_place_near(n, d));
        return 0;
    }
    if (argc == 6) {                          // every record reads the same vectors
        const int n = std::atoi(argv[2]), A = std::atoi(argv[4]);
        std::vector<hop_mix_job> jobs((size_t)n);
        std::memset(jobs.data(), 0, jobs.size() * sizeof(hop_mix_job));
        for (hop_mix_job& j : jobs) {
            j.out = (float*)4096;             // never read here
            j.vel = std::atof(argv[5]) > 0 ? (float*)8192 : nullptr;
            j.A = A;
            for (int a = 0; a < A; ++a) j.src[a] = (const float*)(uintptr_t)(16384 + 4096 * a);
        }
        return hop_mix(jobs.data(), n, std::atoll(argv[3]), nullptr);
    }
    if (argc != 7) return 2;
    const std::string model = argv[1];
    const int N = std::atoi(argv[2]), B = std::atoi(argv[4]);
    const int64_t d = std::atoll(argv[3]), rows = std::atoll(argv[5]);
    std::vector<int32_t> row_ptr{0}, col;
    std::vector<float> W((size_t)N * N, 0.f);
    for (int i = 0; i < N; ++i) {
        for (int j = 0; j < N && model == "complete"; ++j)       // external gradients, a whole pass of 15 iterations
            if (j != i) col.push_back(j);
        if (model != "complete") for (int j : {(i + N - 1) % N < (i + 1) % N ? (i + N - 1) % N : (i + 1) % N, (i + N - 1) % N < (i + 1) % N ? (i + 1) % N : (i + N - 1) % N})
            if (j != i && (col.size() == (size_t)row_ptr.back() || col.back() != j)) col.push_back(j);
        const int deg = (int)col.size() - row_ptr.back();
        for (size_t p = (size_t)row_ptr.back(); p < col.size(); ++p) W[(size_t)col[p] * N + i] = 1.0f / (float)(deg + 1);
        W[(size_t)i * N + i] = 1.0f / (float)(deg + 1);
        row_ptr.push_back((int32_t)col.size());
    }
    hop_opts o;
    hop_opts_default(&o);
    o.batch = B;
    o.momentum = (float)std::atof(argv[6]);
    o.skip_on = model == "skipping";          // csr, Exp(1) delays, every second worker four times as slow
    const int bound = o.skip_on ? 2 : 1;
    const hop_graph g{N, row_ptr.data(), col.data()};
    hop_device dev;
    std::vector<char> arena, workspace;
    dev.arena_bytes = hop_arena_bytes(N, d, bound, 0, &o);
    dev.arena = aligned(arena, dev.arena_bytes);
    dev.hip_stream = nullptr;
    hop_ctx* c = nullptr;
    if (hop_init(&c, &g, W.data(), N, d, bound, 0, &o, &dev)) return 3;
    // never read here: the launchers only print
    std::vector<int64_t> rowptr((size_t)rows + 1, 0);
    float* some = (float*)dev.arena;
    for (int i = 0; i < N; ++i) {
        const int rc = model == "dense" ? hop_set_data_dense(c, i, some, some, rows)
                       : model == "csr" || model == "skipping" ? hop_set_data_csr(c, i, rowptr.data(), (const int32_t*)some, some, some, rows)
                                        : HOP_OK;
        if (rc) return 4;
    }
    if (hop_set_grad_source(c, model == "dense" ? HOP_GRAD_SVM_DENSE : model == "csr" || model == "skipping" ? HOP_GRAD_SVM_CSR : HOP_GRAD_EXTERNAL, 0.f, some)) return 5;
    if (hop_set_params(c, some, 0, 1)) return 6;
    hop_schedule* s = nullptr;
    std::vector<double> slow((size_t)N, 1.0);
    for (int i = 1; i < N; i += 2) slow[(size_t)i] = 4.0;
    hop_delay_model delays;
    std::memset(&delays, 0, sizeof delays);
    delays.kind = HOP_DELAY_EXP1;
    delays.mult = slow.data();
    if (hop_simulate(c, o.skip_on ? &delays : nullptr, o.skip_on ? 30 : model == "complete" ? 15 : 2, &s)) return 7;
    const size_t need = hop_schedule_bytes(s);
    if (hop_schedule_bind(c, s, aligned(workspace, need), need)) return 8;
    hop_schedule_arrays v;
    hop_schedule_view(s, &v);
    if (model == "complete" && hop_step(c, s, 0, -1)) return 9;
    for (int w = 0; w < v.n_waves && model != "complete"; ++w)
        if (hop_step(c, s, w, w + 1)) return 9;
    hop_schedule_free(s);
    return hop_destroy(c);
}
