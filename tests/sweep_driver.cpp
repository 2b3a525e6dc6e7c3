// The program of a whole pass (hop_plan_sweep) run on the CPU against its records run one by one on the rings:
// random schedules of waves, ring depths, source counts past what the kernel takes in one part, vectors listed twice, jumps into
// their own slot, velocities, every kind of gradient.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <random>

#include "hop_internal.h"

// launchers that hop_api.cpp names; nothing here reaches a device
int hopk_mix(const HopMixJob*, int, int64_t, void*) { return 1; }
int hopk_synth(const HopGradJob*, int, int, int64_t, void*) { return 1; }
int hopk_dense_margin(const HopGradJob*, int, int, int64_t, void*) { return 1; }
int hopk_dense_grad(const HopGradJob*, int, int, int64_t, float, int, void*) { return 1; }
int hopk_csr_margin(const HopGradJob*, int, int, int, void*) { return 1; }
int hopk_mix_dense_margin(const HopMixJob*, int, int64_t, const HopGradJob*, int, int, void*) { return 1; }
int hopk_mix_csr_margin(const HopMixJob*, int, int64_t, const HopGradJob*, int, int, int, void*) { return 1; }
int hopk_pair(const HopPairJob*, int, int, int, int64_t, void*) { return 1; }
int hopk_pair_csr_margin(const HopPairJob*, int, int, int, int64_t, const HopGradJob*, int, int, int, void*) { return 1; }
int hopk_pair_dense_margin(const HopPairJob*, int, int, int, int64_t, const HopGradJob*, int, int, void*) { return 1; }
int hopk_csr_scatter(const HopGradJob*, int, int, float, int, void*) { return 1; }
int hopk_csr_dense_grad(const HopGradJob*, int, int, int64_t, float, void*) { return 1; }
int hopk_csr_check(const int64_t*, const int32_t*, int64_t, int64_t, int64_t, int64_t, int*, void*) { return 1; }
int hopk_copy(void*, const void*, size_t, void*) { return 1; }
int hopk_dense_nseg(int64_t d) { return (int)((d + 16383) / 16384); }

static float as_float(uint32_t u) {
    float f;
    std::memcpy(&f, &u, sizeof(f));
    return f;
}
// any function of the keys stands in for the gradient's values
static float grad_of(const uint32_t* key) { return (float)((key[0] * 2654435761u ^ key[1] ^ key[2]) >> 20) / 4096.f - 0.5f; }

#define EXPECT(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)

int main() {
    std::mt19937 gen(3);
    auto below = [&](int n) { return (int)(gen() % (unsigned)n); };
    int wide = 0, refused = 0, kinds[4] = {0, 0, 0, 0};
    for (int run = 0; run < 400; ++run) {
        const int N = 1 + below(run % 7 == 0 ? 90 : 12), depth = 1 + below(5), slots = N * depth, waves = 1 + below(12);
        const int mode = below(3);                                   // 0 none, 1 keys, 2 external
        const bool mom = below(3) == 0;
        const int uniform = run % 4 == 0 ? 1 + below(9) : 0;           // long runs: the same number of sources everywhere
        const float eta = 0.125f, mu = 0.9f;
        std::vector<HopSweepOp> ops;
        for (int w = 0; w < waves; ++w) {
            // no record of a wave writes a slot that another one of it reads or writes
            const size_t wave_begin = ops.size();
            std::vector<int> read_by((size_t)slots, -1), written_by((size_t)slots, -1);
            for (int n = 1 + below(2 * N); n > 0; --n) {
                HopSweepOp op;
                op.worker = below(N);
                op.out_slot = op.worker * depth + below(depth);
                bool seen = false;
                for (size_t o = wave_begin; o < ops.size(); ++o) seen = seen || ops[o].worker == op.worker;
                const int me = (int)ops.size();
                if (seen || written_by[op.out_slot] >= 0 || read_by[op.out_slot] >= 0) continue;
                const int A = uniform ? uniform : 1 + below(below(6) == 0 ? 20 : 8);
                for (int t = 0; t < A; ++t) {
                    const int src = below(slots);
                    if (written_by[src] >= 0) { t -= uniform && below(8) ? 1 : 0; continue; }
                    op.terms.emplace_back(src, 0.0625f * (1 + below(9)));
                    if (!uniform && below(12) == 0) op.terms.push_back(op.terms.back());       // listed twice
                }
                if (op.terms.empty()) continue;
                for (auto& t : op.terms) if (t.first != op.out_slot) read_by[t.first] = me;
                written_by[op.out_slot] = me;
                op.grad = mode != 0 && (uniform || below(5) != 0);
                op.vel = mom && op.grad;
                op.external = op.grad && mode == 2;
                if (op.grad && mode == 1) for (uint32_t& k : op.key) k = gen();
                if (op.external) op.key[0] = (uint32_t)op.worker;
                wide += op.terms.size() > (size_t)kSweepInline;
                ops.push_back(op);
            }
        }
        // record by record
        std::vector<float> ring((size_t)slots), vel((size_t)N), ext((size_t)N);
        for (float& v : ring) v = (float)below(2000) / 1000.f - 1.f;
        for (float& v : vel) v = (float)below(2000) / 1000.f - 1.f;
        for (float& v : ext) v = (float)below(2000) / 1000.f - 1.f;
        const std::vector<float> ring0 = ring, vel0 = vel;
        for (const HopSweepOp& op : ops) {
            float acc = 0.f;
            for (const auto& t : op.terms) acc = std::fmaf(t.second, ring[t.first], acc);
            if (op.grad) {
                float g = op.external ? ext[op.worker] : grad_of(op.key);
                if (op.vel) g = vel[op.worker] = std::fmaf(mu, vel[op.worker], g);
                acc = std::fmaf(-eta, g, acc);
            }
            ring[op.out_slot] = acc;
        }
        // the program, as the kernel reads it
        HopSweepPlan plan;
        if (!hop_plan_sweep(ops, slots, N, &plan)) { ++refused; continue; }
        EXPECT(plan.n_local <= kSweepMaxLocal);
        std::vector<float> got = ring0, gvel = vel0, local((size_t)plan.n_local, NAN);
        const std::vector<uint32_t>& P = plan.program;
        std::vector<char> used((size_t)plan.n_local, 0);
        auto at = [&](uint32_t slot) -> float& { used.at(slot) = 1; return local[slot]; };
        size_t list = (size_t)plan.first_load;
        for (int k = 0; k < plan.n_loads; ++k, list += 2) at(P.at(list + 1)) = ring0.at(P.at(list));
        const size_t vels = list;
        for (int k = 0; k < plan.n_vel; ++k, list += 2) at(P.at(list + 1)) = vel0.at(P.at(list));
        EXPECT(list == P.size());
        std::vector<char> stored((size_t)slots, 0);
        size_t rec = 0;
        int done = 0;
        float ahead = ext.at(plan.first_external);
        for (; rec < (size_t)plan.first_load; ++done) {
            const uint32_t* h = &P.at(rec);
            const int A = (int)h[7];
            EXPECT(rec + hop_sweep_words(A) <= (size_t)plan.first_load);
            kinds[(h[0] & kSweepGrad) + ((h[0] & kSweepKeep) && !(h[0] & kSweepStore) ? 0 : 2)]++;
            float acc = 0.f;
            for (int t = 0; t < A; ++t) {
                EXPECT(!std::isnan(at(h[kSweepHead + 2 * t])));
                acc = std::fmaf(as_float(h[kSweepHead + 2 * t + 1]), at(h[kSweepHead + 2 * t]), acc);
            }
            if (h[0] & kSweepGrad) {
                float g;
                if (mode == 2) {
                    g = ahead;
                    EXPECT(g == ext.at(h[4]));
                    ahead = ext.at(h[5]);
                } else {
                    g = grad_of(h + 4);
                }
                if (mom) g = at(h[3]) = std::fmaf(mu, at(h[3]), g);
                acc = std::fmaf(-eta, g, acc);
            }
            if (h[0] & kSweepKeep) at(h[1]) = acc;
            if (h[0] & kSweepStore) {
                EXPECT(!stored.at(h[2]));                        // once per ring slot
                stored[h[2]] = 1;
                got[h[2]] = acc;
            }
            rec += hop_sweep_words(A);
        }
        EXPECT(done == (int)ops.size());
        EXPECT(ops.empty() || std::find(used.begin(), used.end(), 0) == used.end());    // no local slot is counted in vain
        for (int k = 0; k < plan.n_vel; ++k) gvel.at(P.at(vels + 2 * k)) = at(P.at(vels + 2 * k + 1));
        for (int q = 0; q < slots; ++q) EXPECT(got[q] == ring[q]);
        for (int q = 0; q < N; ++q) EXPECT(gvel[q] == vel[q]);
    }
    EXPECT(wide > 50 && refused > 0 && kinds[0] && kinds[1] && kinds[2] && kinds[3]);
    // as many values at a time as there are local slots, and one more
    for (int n = kSweepMaxLocal; n <= kSweepMaxLocal + 1; ++n) {
        std::vector<HopSweepOp> ops((size_t)n);
        for (int q = 0; q < n; ++q) {
            ops[q].out_slot = ops[q].worker = q;
            ops[q].terms.emplace_back(q, 1.f);
        }
        HopSweepPlan plan;
        EXPECT(hop_plan_sweep(ops, n, n, &plan) == (n == kSweepMaxLocal) && (n > kSweepMaxLocal || plan.n_local == n));
    }
    std::printf("ok wide=%d refused=%d\n", wide, refused);
    return 0;
}
