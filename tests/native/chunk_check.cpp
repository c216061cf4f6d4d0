// Host-only check of the pieces of cut extend blocks: reads a pool shape and
// a batch as plan_driver.cpp does, builds the plan and checks that the pieces
// of every block tile its steps in order, that the first two steps' page ids
// are the plan's, and that states have slots of their own, consecutive per
// block.  Prints "cut <blocks cut> of <blocks>, <pieces> pieces, <slots>
// slots" per case, or what is wrong.
#include <cstdio>
#include <cstring>
#include <set>
#include <vector>

#include "../../paper_2608_25523_amd/csrc/pfx_internal.h"

static bool read_vec(FILE* f, std::vector<int32_t>& v, long n) {
  v.assign(n, 0);
  for (long i = 0; i < n; ++i)
    if (fscanf(f, "%d", &v[i]) != 1) return false;
  return true;
}

#define CHECK(x)                                         \
  do {                                                   \
    if (!(x)) {                                          \
      printf("case %d line %d: %s\n", n, __LINE__, #x);  \
      return 1;                                          \
    }                                                    \
  } while (0)

int main(int argc, char** argv) {
  if (argc != 2) return 2;
  FILE* f = fopen(argv[1], "r");
  if (!f) return 2;
  pfx_pool pool{};
  int hq, mode, piece_steps, workers;
  for (int n = 0; fscanf(f, "%d %d %d %d %d %d %d", &pool.num_pages, &pool.num_kv_heads, &pool.head_dim, &hq, &mode,
                         &piece_steps, &workers) == 7; ++n) {
    pool.page_size = PFX_PAGE_SIZE;
    int A = 0, R = 0;
    std::vector<int32_t> plen, pind, pids, agent, sind, sids, slen, qind;
    CHECK(fscanf(f, "%d", &A) == 1 && read_vec(f, plen, A) && read_vec(f, pind, A + 1) && read_vec(f, pids, pind[A]));
    CHECK(fscanf(f, "%d", &R) == 1 && read_vec(f, agent, R) && read_vec(f, sind, R + 1) && read_vec(f, sids, sind[R]) &&
          read_vec(f, slen, R) && read_vec(f, qind, R + 1));
    pfx_prefix_table pt = {A, pind.data(), pids.data(), plen.data()};
    pfx_batch b = {R, agent.data(), sind.data(), sids.data(), slen.data(), qind.data()};
    pfx_plan* p = nullptr;
    CHECK(pfx_plan_create(&pool, &pt, &b, hq, mode, nullptr, &p) == PFX_OK);
    const auto* chunks = reinterpret_cast<const pfx::Chunk*>(p->blob.data() + p->off_chunks);
    const auto* merges = reinterpret_cast<const pfx::ChunkMerge*>(p->blob.data() + p->off_chunk_merge);
    std::vector<std::vector<pfx::Chunk>> of(p->num_items);
    for (int i = 0; i < p->num_chunks; ++i) {
      CHECK(chunks[i].item >= 0 && chunks[i].item < p->num_items);
      CHECK(i % pool.num_kv_heads == p->host_items()[chunks[i].item].kv_head);  // one XCD per KV head
      of[chunks[i].item].push_back(chunks[i]);
    }
    std::set<int> slots;
    int cut = 0;
    for (int k = 0; p->num_chunks && k < p->num_items; ++k) {
      const pfx::Item& it = p->host_items()[k];
      const int s0 = (it.s0_kend + 31) / 32, steps = s0 + (it.s1_kend + 31) / 32;
      CHECK(!of[k].empty() && of[k].front().st0 == 0 && of[k].back().st1 == steps);
      for (size_t i = 0; i < of[k].size(); ++i) {
        const pfx::Chunk& c = of[k][i];
        CHECK(c.st0 < c.st1 && c.st0 % 2 == 0 && (i == 0 || c.st0 == of[k][i - 1].st1));
        for (int e = 0; e < 2 && c.st0 + e < c.st1; ++e) {
          const int st = c.st0 + e;
          const int32_t* list = p->page_list.data() + (st < s0 ? it.s0_page_off : it.s1_page_off);
          const int kend = st < s0 ? it.s0_kend : it.s1_kend, pg = 2 * (st < s0 ? st : st - s0);
          CHECK(c.pages[2 * e] == list[pg]);
          CHECK(c.pages[2 * e + 1] == list[16 * (pg + 1) < kend ? pg + 1 : pg]);
        }
        if (of[k].size() == 1) CHECK(c.slot == -1);
        else CHECK(c.slot >= 0 && slots.insert(c.slot).second && (i == 0 || c.slot == of[k][i - 1].slot + 1));
      }
      if (of[k].size() > 1) {
        bool found = false;
        for (int i = 0; i < p->num_chunk_merges; ++i)
          if (merges[i].item == k) {
            CHECK(!found && merges[i].base == of[k][0].slot && merges[i].nparts == int(of[k].size()));
            found = true;
          }
        CHECK(found);
        ++cut;
      }
    }
    CHECK(cut == p->num_chunk_merges && (slots.empty() || *slots.rbegin() == int(slots.size()) - 1));
    CHECK(p->off_xlpart + slots.size() * 128 * 8 <= p->total_bytes &&
          p->off_xopart + slots.size() * 128 * 4 * pool.head_dim <= p->off_xlpart);
    printf("cut %d of %d, %d pieces, %zu slots\n", cut, p->num_items, p->num_chunks, slots.size());
    pfx_plan_destroy(p);
  }
  fclose(f);
  return 0;
}
