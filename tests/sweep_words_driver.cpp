// What sweep_kernel reads (hop_lower_sweep) run on the CPU against the records one by one on the rings: random schedules,
// up to 32 sources per record (12 go through the kernel's chain), every kind of gradient, with and without velocities.
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
int hopk_csr_check(const int64_t*, const int32_t*, int64_t, int64_t, int64_t, int64_t, int*, void*) { return 1; }
int hopk_copy(void*, const void*, size_t, void*) { return 1; }
int hopk_dense_nseg(int64_t d) { return (int)((d + 16383) / 16384); }

static float as_float(uint32_t u) {
    float f;
    std::memcpy(&f, &u, sizeof(f));
    return f;
}
static float* address(const uint32_t* w) { return (float*)(uintptr_t)((uint64_t)w[1] << 32 | w[0]); }
static float grad_of(const uint32_t* key) { return (float)((key[0] * 2654435761u ^ key[1] ^ key[2]) >> 20) / 4096.f - 0.5f; }

#define EXPECT(c) do { if (!(c)) { std::printf("run %d, line %d: %s\n", run, __LINE__, #c); return 1; } } while (0)

int main() {
    std::mt19937 gen(11);
    auto below = [&](int n) { return (int)(gen() % (unsigned)n); };
    int run = 0, parts = 0, shorts = 0, rest = 0, most = 0;
    for (; run < 300; ++run) {
        const int N = 1 + below(run % 9 == 0 ? 60 : 12), depth = 1 + below(4), slots = N * depth;
        const int mode = run % 3 == 0 ? HOP_GRAD_ZERO : run % 3 == 1 ? HOP_GRAD_SYNTH : HOP_GRAD_EXTERNAL;
        const bool mom = below(3) == 0;
        const float eta = 0.125f, mu = 0.9f;
        std::vector<HopSweepOp> ops;
        for (int w = 0, waves = 1 + below(10); w < waves; ++w) {
            std::vector<char> read((size_t)slots, 0), written((size_t)slots, 0), used((size_t)N, 0);
            for (int n = 1 + below(2 * N); n > 0; --n) {
                HopSweepOp op;
                op.worker = below(N);
                op.out_slot = op.worker * depth + below(depth);
                if (used[op.worker] || written[op.out_slot] || read[op.out_slot]) continue;
                for (int t = 1 + below(below(4) == 0 ? 32 : 8); t > 0; --t)
                    if (const int src = below(slots); !written[src]) op.terms.emplace_back(src, 0.0625f * (float)(1 + below(9)));
                if (op.terms.empty()) continue;
                for (auto& t : op.terms) if (t.first != op.out_slot) read[t.first] = 1;
                used[op.worker] = written[op.out_slot] = 1;
                op.grad = mode != HOP_GRAD_ZERO && below(5) != 0;
                op.vel = mom && op.grad;
                op.external = op.grad && mode == HOP_GRAD_EXTERNAL;
                if (op.grad && mode == HOP_GRAD_SYNTH) for (uint32_t& k : op.key) k = gen();
                if (op.external) op.key[0] = (uint32_t)op.worker;
                ops.push_back(op);
            }
        }
        std::vector<float> ring((size_t)slots), vel((size_t)N), ext((size_t)N);
        for (auto* v : {&ring, &vel, &ext}) for (float& x : *v) x = (float)below(2000) / 1000.f - 1.f;
        std::vector<float> want = ring, wvel = vel;
        for (const HopSweepOp& op : ops) {
            float acc = 0.f;
            for (const auto& t : op.terms) acc = std::fmaf(t.second, want[t.first], acc);
            if (op.grad) {
                float g = op.external ? ext[op.worker] : grad_of(op.key);
                if (op.vel) g = wvel[op.worker] = std::fmaf(mu, wvel[op.worker], g);
                acc = std::fmaf(-eta, g, acc);
            }
            want[op.out_slot] = acc;
        }
        HopSweepPlan plan;
        if (!hop_plan_sweep(ops, slots, N, &plan)) continue;
        HopSweepArgs a;
        a.mode = mode;
        HopSweepVectors at;
        at.ring = ring.data(); at.vel = vel.data(); at.external = ext.data();
        at.stride = at.d = 1;
        std::vector<uint32_t> P;
        hop_lower_sweep(plan, (int)ops.size(), at, &a, &P);
        // as the kernel reads it: a record is loaded while the one before is at work, so the words behind the end are read too
        EXPECT(a.n_local <= kSweepRegisters && a.first_list == (a.n_records + 1) * kSweepRecord);
        EXPECT(P[(size_t)a.n_records * kSweepRecord] == (a.n_records % 2 ? kSweepOdd : 0u));
        EXPECT(P.size() == (size_t)a.first_list + 32 * (size_t)(a.n_load_groups + a.n_store_groups) && a.n_load_groups >= 1);
        most = std::max(most, a.n_local);
        std::vector<float> local((size_t)a.n_local, NAN);
        for (int k = 0; k < 8 * a.n_load_groups && address(&P.at(a.first_list + 4 * k)); ++k)
            local.at(P.at(a.first_list + 4 * k + 2)) = *address(&P.at(a.first_list + 4 * k));
        const float* ahead = (const float*)(uintptr_t)a.first_external;
        int finished = 0;
        for (int r = 0; r < a.n_records; ++r) {
            const uint32_t *w = &P.at((size_t)r * kSweepRecord), flags = w[1] & ~255u, whole = r == 0 || (w[1 - kSweepRecord] & kSweepNextWhole);
            const uint32_t entry = w[0] % kSweepLong;
            const bool through = w[0] & kSweepLong;
            EXPECT(!(w[0] & kSweepOdd) == !(r & 1) && w[0] < 2 * kSweepOdd && entry % kSweepStep == 0 && entry >= kSweepStep);
            EXPECT(entry <= kSweepInline * kSweepStep && (w[1] & 255u) < (uint32_t)a.n_local && flags < 2 * kSweepNextWhole);
            EXPECT(whole || (!through && entry >= 8 * kSweepStep));                 // not read: words 16 to 31
            EXPECT(!std::isnan(local.at(w[5])));
            float acc = std::fmaf(as_float(w[6]), local.at(w[5]), 0.f);
            const int chain[11] = {28, 26, 24, 22, 20, 18, 16, 13, 11, 9, 7};      // the words that the kernel's chain reads
            for (uint32_t k = entry / kSweepStep - 1; k < 11; ++k) {
                EXPECT(!std::isnan(local.at(w[chain[k]])));
                acc = std::fmaf(as_float(w[chain[k] + 1]), local.at(w[chain[k]]), acc);
            }
            EXPECT(through || ((flags & kSweepToLocal) && !(flags & kSweepToRing) && (mode == HOP_GRAD_ZERO || (flags & kSweepWithGrad))));
            (through ? rest : shorts)++;
            if (flags & kSweepWithGrad) {
                float g = mode == HOP_GRAD_SYNTH ? grad_of(w + 2) : 0.f;
                if (mode == HOP_GRAD_EXTERNAL) { g = *ahead; ahead = address(w + 2); }
                if (mom) g = local.at(w[15]) = std::fmaf(mu, local.at(w[15]), g);
                acc = std::fmaf(-eta, g, acc);
            }
            if (flags & kSweepToLocal) local.at(w[1] & 255u) = acc;
            if (flags & kSweepToRing) *address(w + 30) = acc;
            finished += (flags & kSweepToLocal) == 0 || (w[1] & 255u) != (uint32_t)plan.n_local;
        }
        EXPECT(finished == (int)ops.size());
        parts += a.n_records - finished;
        for (int k = 8 * a.n_load_groups; k < 8 * (a.n_load_groups + a.n_store_groups) && address(&P.at(a.first_list + 4 * k)); ++k)
            *address(&P.at(a.first_list + 4 * k)) = local.at(P.at(a.first_list + 4 * k + 2));
        for (int q = 0; q < slots; ++q) EXPECT(ring[q] == want[q]);
        for (int q = 0; q < N; ++q) EXPECT(vel[q] == wvel[q]);
    }
    EXPECT(parts > 50 && shorts > 500 && rest > 500 && most > 112);
    std::printf("ok parts=%d short=%d rest=%d locals=%d\n", parts, shorts, rest, most);
    return 0;
}
