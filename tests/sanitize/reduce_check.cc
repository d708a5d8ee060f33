// CPU run of the small-tile GEMM kernels' reduction (gemm_reduce.h), one thread per lane of a block: LDS accesses are recorded with the
// barriers and fences passed before them.  Checked: all waves of the block meet at one barrier instruction; no two lanes
// use the same 16 bytes, one of them writing, without a barrier between (or, in one wave, a fence); the sums; and that the area handed to
// each wave is then its own in any lane layout.
#include <pthread.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <map>
#include <thread>
#include <vector>

#define __device__
#define __forceinline__ inline

typedef float floatx16 __attribute__((vector_size(64)));

struct Access { int thread, block_epoch, wave_epoch; bool write; };
struct LaneState {
    int thread = 0, block_epoch = 0, wave_epoch = 0;
    std::vector<std::pair<uintptr_t, Access>> log;
};
static thread_local LaneState *me;
static uint8_t *lds, *lds_end;
static pthread_barrier_t block_barrier, wave_barriers[8];
static std::vector<void *> barrier_sites[1024];   // per thread, in order

static void record(const void *p, bool write)
{
    const uint8_t *b = (const uint8_t *)p;
    if (b < lds || b >= lds_end) return;
    if ((b - lds) % 16) { printf("misaligned LDS access\n"); exit(1); }
    me->log.push_back({(uintptr_t)(b - lds) / 16, {me->thread, me->block_epoch, me->wave_epoch, write}});
}

struct float4 {
    float x, y, z, w;
    float4(float a, float b, float c, float d) : x(a), y(b), z(c), w(d) {}
    float4(const float4 &o) { record(&o, false); x = o.x; y = o.y; z = o.z; w = o.w; }
    float4 &operator=(const float4 &o) { record(this, true); x = o.x; y = o.y; z = o.z; w = o.w; return *this; }
};
static float4 make_float4(float a, float b, float c, float d) { return float4(a, b, c, d); }

__attribute__((noinline)) static void __syncthreads()
{
    barrier_sites[me->thread].push_back(__builtin_return_address(0));
    pthread_barrier_wait(&block_barrier);
    ++me->block_epoch;
}

namespace qii {
namespace {
__attribute__((noinline)) void wave_lds_fence()
{
    pthread_barrier_wait(&wave_barriers[me->thread / 64]);
    ++me->wave_epoch;
}
}  // namespace
}  // namespace qii

#include "../../paper_2601_22813_amd/csrc/gemm_reduce.h"

// (whole numbers: every order of the sum gives the same)
static float value(int thread, int unit, int entry) { return (float)((thread * 7 + unit * 131 + entry * 17) % 1009); }

template <int WM, int KG, int N>
static int check(const char *name)
{
    constexpr int kArea = (N / 2) * 4096 + 512, kThreads = 64 * WM * KG, kOut = N / KG;
    std::vector<uint8_t> memory(WM * KG * kArea + 64);
    lds = (uint8_t *)(((uintptr_t)memory.data() + 15) & ~(uintptr_t)15);
    lds_end = lds + WM * KG * kArea;
    pthread_barrier_init(&block_barrier, nullptr, kThreads);
    for (int i = 0; i < WM * KG; ++i) pthread_barrier_init(&wave_barriers[i], nullptr, 64);
    std::vector<LaneState> lanes(kThreads);
    std::vector<float> sums((size_t)kThreads * kOut * 16);
    std::vector<uint8_t *> areas(kThreads);
    std::vector<std::thread> threads;
    for (int t = 0; t < kThreads; ++t) {
        barrier_sites[t].clear();
        threads.emplace_back([&, t] {
            me = &lanes[t];
            me->thread = t;
            const int lane = t & 63, wave = t >> 6, wm = wave % WM, kg = wave / WM;
            floatx16 acc[N], out[kOut];
            for (int u = 0; u < N; ++u)
                for (int e = 0; e < 16; ++e) acc[u][e] = value(t, u ^ qii::reduce_flip<KG, N>(kg), e);
            uint8_t *area = qii::reduce_groups<WM, KG, kArea>(acc, out, lds, kg, wm, lane);
            areas[t] = area;
            for (int u = 0; u < kOut; ++u)
                for (int e = 0; e < 16; ++e) sums[((size_t)t * kOut + u) * 16 + e] = out[u][e];
            // the epilogue: this lane writes where other lanes of its wave wrote and read
            float4 *cells = reinterpret_cast<float4 *>(area);
            for (int i = lane * (kArea / 16 / 64); i < (lane + 1) * (kArea / 16 / 64); ++i) cells[i] = make_float4(1, 2, 3, 4);
        });
    }
    for (auto &t : threads) t.join();
    pthread_barrier_destroy(&block_barrier);
    for (int i = 0; i < WM * KG; ++i) pthread_barrier_destroy(&wave_barriers[i]);

    int bad = 0;
    for (int t = 1; t < kThreads; ++t)
        if (barrier_sites[t] != barrier_sites[0]) { printf("%s: thread %d waits at another barrier than thread 0\n", name, t); ++bad; break; }
    for (int w = 0; w < WM * KG; ++w)
        for (int v = 0; v < w; ++v)
            if (areas[64 * w] == areas[64 * v]) { printf("%s: waves %d and %d have one area\n", name, v, w); ++bad; }
    int wrong = 0;
    for (int t = 0; t < kThreads; ++t) {
        const int wave = t >> 6, wm = wave % WM, kg = wave / WM;
        for (int u = 0; u < kOut; ++u)
            for (int e = 0; e < 16; ++e) {
                float want = 0;
                for (int k = 0; k < KG; ++k) want += value((k * WM + wm) * 64 + (t & 63), kg * kOut + u, e);
                wrong += sums[((size_t)t * kOut + u) * 16 + e] != want;
            }
    }
    if (wrong) { printf("%s: %d wrong sums\n", name, wrong); ++bad; }
    std::map<uintptr_t, std::vector<Access>> cells;
    for (auto &l : lanes)
        for (auto &a : l.log) cells[a.first].push_back(a.second);
    int races = 0;
    for (auto &c : cells)
        for (auto &a : c.second)
            for (auto &b : c.second)
                if (a.write && a.thread != b.thread && a.block_epoch == b.block_epoch &&
                    (a.thread / 64 != b.thread / 64 || a.wave_epoch == b.wave_epoch))
                    ++races;
    if (races) { printf("%s: %d pairs of unordered accesses to one place of LDS\n", name, races); ++bad; }
    return bad;
}

int main()
{
    const int bad = check<2, 2, 8>("128 x 128, two groups") + check<1, 4, 16>("128 x 128, four groups") + check<1, 4, 4>("64 x 64");
    if (bad == 0) printf("reduce check: ok\n");
    return bad != 0;
}
