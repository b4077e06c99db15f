// Runs the device code that shares out a batch's attention on the CPU: one workgroup of 256 threads as coroutines that
// take turns at every barrier.  Reads batches from stdin, one line of numbers each:
//   n_wgs n_kv group max_pages rows_per_wg max_items n_seq  new_len[n_seq]  prefix_len[n_seq]
// and prints, a line per batch: tile_start[n_seq + 1], item_seq[items], then three numbers per bound.
#include <ucontext.h>

#include <cstdio>
#include <vector>

#include <hip/hip_runtime.h>

namespace {
struct Dim {
    unsigned x;
};
Dim threadIdx;
constexpr int kThreads = 256;
ucontext_t scheduler, fiber[kThreads];
int lane_value[kThreads];
bool done[kThreads];

void barrier() {
    const unsigned me = threadIdx.x;
    swapcontext(&fiber[me], &scheduler);
}
int exchange(int v, int from, bool valid) {   // every thread writes, then every thread reads
    lane_value[threadIdx.x] = v;
    barrier();
    const int r = valid ? lane_value[from] : v;
    barrier();
    return r;
}
int shfl_up(int v, int o) { return exchange(v, (int)threadIdx.x - o, (int)(threadIdx.x & 63) >= o); }
int shfl_xor(int v, int o) { return exchange(v, (int)threadIdx.x ^ o, true); }
float as_float(unsigned u) {
    float f;
    __builtin_memcpy(&f, &u, 4);
    return f;
}
}  // namespace

#define __syncthreads() barrier()
#define __shfl_up(v, o, w) shfl_up(v, o)
#define __shfl_xor(v, o, w) shfl_xor(v, o)
#define __uint_as_float(u) as_float(u)
#include "../paper_2601_11589_amd/csrc/laps_internal.h"

namespace {
struct Batch {
    int n_wgs, n_kv, group, max_pages, rows_per_wg, max_items, n_seq;
    std::vector<int> new_len, prefix_len, tile_start, item_seq, pre;
    std::vector<int4> bounds;
} b;
int sums[4];

void thread_main() {
    laps_dev_attn_sched(b.new_len.data(), b.n_seq, b.group, b.rows_per_wg, b.tile_start.data(), b.item_seq.data(), b.max_items, sums);
    laps_dev_attn_bounds(b.new_len.data(), b.prefix_len.data(), b.n_seq, b.group, b.n_kv, b.max_pages, b.tile_start.data(),
                         b.item_seq.data(), b.max_items, b.n_wgs, b.pre.data(), b.bounds.data(), sums);
    done[threadIdx.x] = true;
    barrier();
}
}  // namespace

int main() {
    std::vector<std::vector<char>> stack(kThreads, std::vector<char>(64 << 10));
    while (std::scanf("%d %d %d %d %d %d %d", &b.n_wgs, &b.n_kv, &b.group, &b.max_pages, &b.rows_per_wg, &b.max_items, &b.n_seq) == 7) {
        b.new_len.resize(b.n_seq);
        b.prefix_len.resize(b.n_seq);
        for (int& v : b.new_len)
            if (std::scanf("%d", &v) != 1) return 1;
        for (int& v : b.prefix_len)
            if (std::scanf("%d", &v) != 1) return 1;
        b.tile_start.assign(b.n_seq + 1, -1);
        b.item_seq.assign(b.max_items, -1);
        b.pre.assign(b.max_items + 1, -1);
        b.bounds.assign(b.n_wgs + 1, int4{-1, -1, -1, -1});
        for (int t = 0; t < kThreads; ++t) {
            done[t] = false;
            getcontext(&fiber[t]);
            fiber[t].uc_stack.ss_sp = stack[t].data();
            fiber[t].uc_stack.ss_size = stack[t].size();
            fiber[t].uc_link = nullptr;
            makecontext(&fiber[t], thread_main, 0);
        }
        for (int left = kThreads; left > 0;)
            for (int t = 0; t < kThreads; ++t) {
                if (done[t]) continue;
                threadIdx.x = t;
                swapcontext(&scheduler, &fiber[t]);
                left -= done[t];
            }
        for (int v : b.tile_start) std::printf("%d ", v);
        for (int v : b.item_seq) std::printf("%d ", v);
        for (const int4& v : b.bounds) std::printf("%d %d %d ", v.x, v.y, v.z);
        std::printf("\n");
    }
    return 0;
}
