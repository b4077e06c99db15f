// Runs the device code that describes a batch's attention work items, and cuts their key ranges into parts, on the CPU, with the
// coroutines of the driver next to it.  Reads batches from stdin, one line of numbers each:
//   n_split min_tiles group max_pages rows_per_wg max_items n_seq  new_len[n_seq]  prefix_len[n_seq]
// and prints, a line per batch, eight numbers per item of the table and a guard entry behind.
#define main shares_main
#include "attn_shares_driver.cpp"
#undef main

namespace {
int n_split, min_tiles;
std::vector<int> row_start;
std::vector<int4> desc;

void split_main() {
    laps_dev_attn_sched(b.new_len.data(), b.n_seq, b.group, b.rows_per_wg, b.tile_start.data(), b.item_seq.data(), b.max_items, sums);
    laps_dev_attn_desc(b.new_len.data(), b.prefix_len.data(), row_start.data(), b.n_seq, b.group, b.rows_per_wg, b.max_pages,
                       b.tile_start.data(), b.item_seq.data(), b.max_items, n_split, min_tiles, desc.data());
    done[threadIdx.x] = true;
    barrier();
}
}  // namespace

int main() {
    std::vector<std::vector<char>> stack(kThreads, std::vector<char>(64 << 10));
    while (std::scanf("%d %d %d %d %d %d %d", &n_split, &min_tiles, &b.group, &b.max_pages, &b.rows_per_wg, &b.max_items,
                      &b.n_seq) == 7) {
        b.new_len.resize(b.n_seq);
        b.prefix_len.resize(b.n_seq);
        for (int& v : b.new_len)
            if (std::scanf("%d", &v) != 1) return 1;
        for (int& v : b.prefix_len)
            if (std::scanf("%d", &v) != 1) return 1;
        row_start.assign(1, 0);
        for (int v : b.new_len) row_start.push_back(row_start.back() + v);
        b.tile_start.assign(b.n_seq + 1, -1);
        b.item_seq.assign(b.max_items, -1);
        desc.assign(2 * (b.max_items + 1), int4{-7, -7, -7, -7});
        for (int t = 0; t < kThreads; ++t) {
            done[t] = false;
            getcontext(&fiber[t]);
            fiber[t].uc_stack.ss_sp = stack[t].data();
            fiber[t].uc_stack.ss_size = stack[t].size();
            fiber[t].uc_link = nullptr;
            makecontext(&fiber[t], split_main, 0);
        }
        for (int left = kThreads; left > 0;)
            for (int t = 0; t < kThreads; ++t) {
                if (done[t]) continue;
                threadIdx.x = t;
                swapcontext(&scheduler, &fiber[t]);
                left -= done[t];
            }
        for (const int4& v : desc) std::printf("%d %d %d %d ", v.x, v.y, v.z, v.w);
        std::printf("\n");
    }
    return 0;
}
