// Host-side checks of libbrsvd for a build whose host code is instrumented with the address and undefined-
// behaviour sanitizers (python -m paper_1706_07191_amd.build --host-asan).  Everything here runs without a
// GPU: argument validation, working-set sizing and block resolution, the launch planners of the two thin
// products over many shapes, and the failure paths of the calls that would touch a device -- on a machine
// without one they fail inside the runtime, and the library has to hand back a status and free what it took.
// The sanitizers turn an out-of-bounds access, a signed overflow or a leak on any of these paths into a
// non-zero exit status.
#include <cinttypes>
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include <vector>

#include "brsvd.h"
#include "brsvd_steps.h"
#include "common.h"
#include "split.h"

static int g_checks = 0, g_failed = 0;
#define CHECK(cond)                                                             \
  do {                                                                          \
    ++g_checks;                                                                 \
    if (!(cond)) { ++g_failed; std::printf("FAILED line %d: %s\n", __LINE__, #cond); } \
  } while (0)

static brsvd_params base_params() {
  brsvd_params p;
  std::memset(&p, 0, sizeof(p));
  p.m = 2000; p.n = 1000; p.k = 20; p.p = 10; p.q = 2; p.row_block = 512;
  return p;
}

// small deterministic generator (no library state)
static uint64_t g_state = 0x1706071910ull;
static uint64_t next_u64() {
  g_state ^= g_state << 13; g_state ^= g_state >> 7; g_state ^= g_state << 17;
  return g_state;
}
static int64_t uniform(int64_t lo, int64_t hi) { return lo + (int64_t)(next_u64() % (uint64_t)(hi - lo + 1)); }

int main() {
  uint64_t bytes = 0;
  brsvd_handle h = nullptr;

  // ---- blocks of a split contraction: read inside the range, every index covered once, the first of any two whole ----
  for (int i = 0; i < 4000; ++i) {
    using namespace brsvd;
    const int64_t K = i < 1500 ? 3 * kSplitB + i : uniform(512, 200000), chunks = split_chunks(K);
    std::vector<unsigned char> covered((size_t)K, 0);
    int64_t next = 0;                                    // the first index that the chunks before do not cover
    bool good = true;
    for (int64_t c = 0; c < chunks; ++c) {
      good &= next == std::min(K, block_index(2 * c, K) * kSplitB) && block_first(2 * c, K) == block_start(2 * c, K);
      if (c < whole_steps(K)) good &= block_first(2 * c + 1, K) == block_start(2 * c, K) + kSplitB;
      for (int64_t b = 2 * c; b < 2 * c + 2; ++b) {
        const int64_t k0 = block_start(b, K), first = block_first(b, K);
        good &= k0 >= 0 && k0 + kSplitB <= K && k0 == block_start((int)b, (int)empty_block(K), (int)K);
        for (int64_t k = std::max(k0, first); k < k0 + kSplitB; ++k) { good &= covered[k]++ == 0; ++next; }
      }
    }
    CHECK(good && next == K);
  }

  // ---- argument validation ----
  CHECK(brsvd_workspace_bytes(nullptr, &bytes) == BRSVD_ERR_ARG);
  CHECK(brsvd_create(nullptr, &h) == BRSVD_ERR_ARG && h == nullptr);
  {
    brsvd_params p = base_params();
    CHECK(brsvd_workspace_bytes(&p, nullptr) == BRSVD_ERR_ARG);
    CHECK(brsvd_create(&p, nullptr) == BRSVD_ERR_ARG);
    struct { int field; int64_t value; } bad[] = {{0, 0}, {1, -1}, {2, 0}, {3, -1}, {4, -1}, {2, 600}, {0, 20}, {5, -5},
                                                  {6, 7}, {7, 5}, {8, 3}, {9, 9}, {10, 4}};
    for (auto& b : bad) {
      brsvd_params q = base_params();
      switch (b.field) {
        case 0: q.m = b.value; break;
        case 1: q.n = b.value; break;
        case 2: q.k = (int32_t)b.value; break;
        case 3: q.p = (int32_t)b.value; break;
        case 4: q.q = (int32_t)b.value; break;
        case 5: q.row_block = b.value; break;
        case 6: q.pass_mode = (int32_t)b.value; break;
        case 7: q.dtype = (int32_t)b.value; break;
        case 8: q.timing_level = (int32_t)b.value; break;
        case 9: q.a_location = (int32_t)b.value; break;
        case 10: q.orth_method = (int32_t)b.value; break;
      }
      CHECK(brsvd_workspace_bytes(&q, &bytes) == BRSVD_ERR_ARG);
      h = (brsvd_handle)0x1;
      CHECK(brsvd_create(&q, &h) == BRSVD_ERR_ARG && h == nullptr);
    }
    brsvd_params w = base_params();
    w.workspace = (void*)0x1004;          // misaligned
    w.workspace_bytes = 1ull << 30;
    CHECK(brsvd_create(&w, &h) == BRSVD_ERR_ARG && h == nullptr);
  }
  CHECK(brsvd_run(nullptr, nullptr, 0, nullptr, nullptr, nullptr, nullptr, nullptr) == BRSVD_ERR_ARG);
  CHECK(brsvd_run_f64(nullptr, nullptr, 0, nullptr, nullptr, nullptr, nullptr, nullptr) == BRSVD_ERR_ARG);
  CHECK(brsvd_run_alg2(nullptr, nullptr, 0, 1, nullptr, nullptr, nullptr, nullptr, nullptr) == BRSVD_ERR_ARG);
  CHECK(brsvd_rpca_ialm(nullptr, nullptr, nullptr, 1, 0.1f, 1.f, 1.5f, 0.0, nullptr, nullptr, nullptr, nullptr, nullptr) ==
        BRSVD_ERR_ARG);
  CHECK(brsvd_norm2_power(nullptr, nullptr, 0, nullptr, 1, nullptr) == BRSVD_ERR_ARG);
  CHECK(brsvd_destroy(nullptr) == BRSVD_OK);
  CHECK(std::strcmp(brsvd_status_string(BRSVD_OK), "ok") == 0);
  for (int s = -6; s < 0; ++s) CHECK(std::strlen(brsvd_status_string(s)) > 2);
  CHECK(std::strcmp(brsvd_status_string(-99), "unknown status") == 0);

  // ---- working-set sizing and block resolution over many parameter sets ----
  for (int it = 0; it < 400; ++it) {
    brsvd_params p = base_params();
    p.m = uniform(1, 3) == 1 ? uniform(1, 400) : uniform(400, 300000);
    p.n = uniform(1, 3) == 1 ? uniform(1, 400) : uniform(400, 120000);
    const int64_t lmax = p.m < p.n ? p.m : p.n;
    const int64_t l = uniform(1, lmax < 512 ? lmax : 512);
    p.p = (int32_t)uniform(0, l - 1);
    p.k = (int32_t)(l - p.p);
    p.q = (int32_t)uniform(0, 3);
    p.dtype = (int32_t)uniform(0, 1);
    p.pass_mode = (int32_t)uniform(0, 1);
    p.a_location = (int32_t)uniform(0, 1);
    p.row_block = uniform(0, 3) == 0 ? 0 : uniform(1, p.m);
    if (p.a_location == BRSVD_A_HOST_PINNED && p.row_block == 0) p.device_budget_bytes = (uint64_t)uniform(1, 64) << 28;
    const int st = brsvd_workspace_bytes(&p, &bytes);
    CHECK(st == BRSVD_OK || st == BRSVD_ERR_BUDGET);
    if (st == BRSVD_OK) {
      const uint64_t esz = p.dtype == BRSVD_DTYPE_F64 ? 8 : 4;
      const uint64_t Lp = (uint64_t)(l + 15) / 16 * 16;
      CHECK(bytes >= 2 * (uint64_t)(p.m + p.n) * Lp * esz);              // the four thin panels
      if (p.device_budget_bytes) CHECK(bytes <= p.device_budget_bytes);
      brsvd_params tight = p;
      tight.device_budget_bytes = bytes - 1;
      if (p.row_block != 0) CHECK(brsvd_workspace_bytes(&tight, &bytes) == BRSVD_ERR_BUDGET);
    }
  }

  // ---- launch planners: every shape must give a plan with positive sizes and no overflow ----
  for (int it = 0; it < 3000; ++it) {
    const int64_t rows = uniform(1, 3) == 1 ? uniform(1, 300) : uniform(1, 2500000);
    const int64_t n = uniform(1, 3) == 1 ? uniform(1, 300) : uniform(1, 150000);
    const int32_t l = (int32_t)uniform(1, 512);
    const int32_t dtype = (int32_t)uniform(0, 1);
    int32_t out[12];
    CHECK(brsvd_gemm_plan(0, rows, n, l, 0, dtype, out) == BRSVD_OK);
    CHECK(out[0] > 0 && out[1] > 0 && out[2] > 0 && out[3] + out[4] == out[1] && out[9] > 0);
    const int64_t b = uniform(0, 1) ? 0 : uniform(1, rows);
    CHECK(brsvd_gemm_plan(1, rows, n, l, b, dtype, out) == BRSVD_OK);
    CHECK(out[2] > 0 && out[3] > 0 && out[4] > 0 && out[5] > 0 && out[6] == out[3] * out[4]);
    CHECK(brsvd_gemm_plan(2, rows, n, l, b, dtype, out) == BRSVD_OK);
    CHECK(out[0] >= 0 && out[1] >= 0 && out[2] >= 0 && out[3] >= 0);
  }
  {
    int32_t out[12];
    CHECK(brsvd_gemm_plan(0, 0, 10, 4, 0, 0, out) == BRSVD_ERR_ARG);
    CHECK(brsvd_gemm_plan(3, 10, 10, 4, 0, 0, out) == BRSVD_ERR_ARG);
    CHECK(brsvd_gemm_plan(0, 10, 10, 4, 0, 0, nullptr) == BRSVD_ERR_ARG);
    CHECK(brsvd_gemm_scratch_bytes(0, 10, 4) == 0 && brsvd_gemm_scratch_bytes(512, 1000, 30) > 0);
    CHECK(brsvd_orth_scratch_bytes(100, 600) == 0 && brsvd_small_svd_scratch_bytes(0) == 0);
    CHECK(brsvd_small_svd_scratch_bytes(512) >= 2ull * 512 * 512 * 8);
  }

  // ---- plans of the split products: every unit of work covered once, partial panels inside whatever scratch there is ----
  for (int it = 0; it < 400; ++it) {
    const int64_t rows = uniform(1, 3) == 1 ? uniform(64, 3000) : uniform(64, 700000);
    const int64_t n = uniform(1, 3) == 1 ? uniform(64, 3000) : uniform(64, 100000);
    const int Lp = 16 * (int)uniform(3, 32);
    const uint64_t an = brsvd::gemm_an_scratch_bytes(rows, n, Lp), at = brsvd::gemm_at_scratch_bytes(rows, n, Lp, rows);
    const uint64_t scratch = uniform(1, 4) == 1 ? (uint64_t)uniform(0, 1 << 24) : (an > at ? an : at);
    const brsvd::SplitPlan p = brsvd::split_an_plan(rows, n, Lp, scratch);
    CHECK((uint64_t)p.nsplit * p.partial_rows * Lp * 4 <= scratch && p.groups * p.nt * 16 >= Lp && p.nt <= 17);
    CHECK((int64_t)(p.sh.whole + p.sh.lt) * p.tile >= rows && (int64_t)(p.sh.whole + p.sh.lt - 1) * p.tile < rows);
    CHECK((int64_t)p.sh.C * 64 >= n && p.partial_rows == (p.nsplit ? rows - (int64_t)p.sh.whole * p.tile : 0));
    std::vector<int> chunks(p.sh.whole + p.sh.lt, 0);
    for (int b = 0; b < p.wgs; ++b) {
      const brsvd::AnWork w = brsvd::an_work(p.sh, b);
      CHECK(w.c0 < w.c1 && w.c1 <= p.sh.C && w.partial == (w.first_tile >= p.sh.whole) && (!w.partial || w.slot < p.nsplit));
      for (int t = 0; t < w.nseg; ++t) chunks[w.first_tile + t] += w.c1 - w.c0;
    }
    for (int c : chunks) CHECK(c == p.sh.C);
    const brsvd::SplitPlan q = brsvd::split_at_plan(rows, n, Lp, scratch);
    CHECK((uint64_t)q.nsplit * n * Lp * 4 <= scratch);
    if (q.nsplit > 0) {
      CHECK(q.blocks % 2 == 0 && q.blocks_per_sub % 2 == 0 && q.blocks_per_sub >= 2 && (int64_t)q.blocks * 32 >= rows);
      CHECK((int64_t)q.nsplit * q.blocks_per_sub >= q.blocks && (int64_t)(q.nsplit - 1) * q.blocks_per_sub < q.blocks);
      CHECK((int64_t)q.col_tiles * q.tile >= n && (int64_t)(q.col_tiles - 1) * q.tile < n);
    }
    // the packed panel fits where the driver and the step calls put it: the TSQR work area, two padded fp32 panels
    if (rows * n >= brsvd::kSplitMinA && n >= brsvd::kSplitMinK) {
      const int64_t most = rows > n ? rows : n;
      CHECK(brsvd::split_fits(false, (const float*)0x4, rows, n, Lp, n, brsvd::tsqr_work_bytes(most, Lp)));
      CHECK(brsvd::split_fits(true, (const float*)0x4, rows, n, Lp, n, 2ull * most * Lp * 4));
      CHECK(brsvd_gemm_is_split(0, (const void*)0x4, n, rows, n, Lp, BRSVD_DTYPE_F32) == 1);
    }
  }

  // ---- tickets of the block Jacobi iteration: with any number of resident workgroups, in any order of their steps, every pair of
  // blocks is rotated once per sweep, no round starts before the one before has ended, and all workgroups come to an end ----
  for (int it = 0; it < 600; ++it) {
    const int nblk2 = 2 * (int)uniform(2, 16), P = nblk2 / 2, rounds = nblk2 - 1, max_sweeps = 5;
    const int sweeps = (int)uniform(1, max_sweeps), resident = (int)uniform(1, P);
    const bool settles = sweeps < max_sweeps || uniform(0, 1) == 1;
    struct Group { int ticket, next, stage; };           // stage 0: no ticket, 1: waits, 2: at work with the next ticket drawn, 3: left
    std::vector<Group> wg(P, Group{0, 0, 0});
    std::vector<int> turned(max_sweeps * rounds * P, 0), ended(4, 0);
    int taken = 0, done = 0, last = 0, left = 0;
    bool stuck = false;
    // the workgroups from `resident` on only start when one before them has left
    while (left < P && !stuck) {
      std::vector<int> ready;
      for (int g = 0; g < P && g < resident + left; ++g) {
        if (wg[g].stage == 1 && done < brsvd::jacobi_ticket(wg[g].ticket, nblk2).before) continue;
        if (wg[g].stage != 3) ready.push_back(g);
      }
      if (ready.empty()) { stuck = true; break; }
      Group& g = wg[ready[uniform(0, (int)ready.size() - 1)]];
      const brsvd::JacobiTicket k = brsvd::jacobi_ticket(g.ticket, nblk2);
      if (g.stage == 0) {
        g = Group{taken++, 0, 1};
      } else if (g.stage == 1) {
        const int what = brsvd::jacobi_work(k, last, max_sweeps);
        ++ended[what];
        g.stage = what == brsvd::JACOBI_END ? 3 : 2;
        left += g.stage == 3;
        if (g.stage == 2) g.next = taken++;
        if (what == brsvd::JACOBI_ROTATE) {
          CHECK(k.sweep < sweeps && done >= (k.sweep * rounds + k.round) * P && done < (k.sweep * rounds + k.round + 1) * P);
          ++turned[(k.sweep * rounds + k.round) * P + k.pair];
          if ((k.sweep + 1 < sweeps || !settles) && k.pair == P - 1 && k.round == (k.sweep % rounds)) last = k.sweep + 1;
        } else if (what == brsvd::JACOBI_RANKS) {
          CHECK(ended[brsvd::JACOBI_NORMS] == P && k.sweep == sweeps && (last < k.sweep) == settles);
        }
      } else {
        ++done;
        g = Group{g.next, 0, 1};
      }
    }
    CHECK(!stuck && left == P && ended[brsvd::JACOBI_RANKS] == P);
    for (int x = 0; x < sweeps * rounds * P; ++x) CHECK(turned[x] == 1);
  }

  // ---- step calls: scratch that is missing, misaligned or too short is refused before any device call ----
  {
    void* one = (void*)0x100;
    CHECK(brsvd_gemm_an(nullptr, 0, 0, 0, nullptr, 0, nullptr, nullptr, 0, nullptr) == BRSVD_ERR_ARG);
    CHECK(brsvd_gemm_an((const float*)one, 64, 64, 64, (const float*)one, 8, (float*)one, one, 16, nullptr) == BRSVD_ERR_BUDGET);
    CHECK(brsvd_gemm_at((const float*)one, 64, 64, 64, (const float*)one, 8, (float*)one, 0, nullptr, 0, nullptr) ==
          BRSVD_ERR_BUDGET);
    CHECK(brsvd_orth(nullptr, 0, 0, 0, nullptr, nullptr, nullptr, 0, nullptr) == BRSVD_ERR_ARG);
    CHECK(brsvd_orth((float*)one, 100, 8, 0, nullptr, nullptr, one, 16, nullptr) == BRSVD_ERR_BUDGET);
    CHECK(brsvd_orth((float*)one, 100, 8, 0, nullptr, nullptr, (void*)0x108, 1 << 20, nullptr) == BRSVD_ERR_ARG);
    CHECK(brsvd_small_svd((const double*)one, 8, (double*)one, (double*)one, (double*)one, nullptr, nullptr, 1 << 20, nullptr) ==
          BRSVD_ERR_ARG);
    CHECK(brsvd_small_svd((const double*)one, 8, (double*)one, (double*)one, (double*)one, nullptr, one, 16, nullptr) ==
          BRSVD_ERR_BUDGET);
    CHECK(brsvd_small_svd_static((const double*)one, 513, (double*)one, (double*)one, (double*)one, nullptr, nullptr) ==
          BRSVD_ERR_BUDGET);
    CHECK(brsvd_small_svd_static(nullptr, 8, (double*)one, (double*)one, (double*)one, nullptr, nullptr) == BRSVD_ERR_ARG);
    CHECK(brsvd_philox_normal(1, 0, 0, 4, (float*)one, nullptr) == BRSVD_ERR_ARG);
    CHECK(brsvd_probe(0, nullptr, 16, nullptr, nullptr, nullptr) == BRSVD_ERR_ARG);
  }

  // ---- calls that reach the device: without one they must fail with a status and free everything ----
  {
    brsvd_params p = base_params();
    h = (brsvd_handle)0x1;
    const int st = brsvd_create(&p, &h);
    if (st == BRSVD_OK) {
      // a GPU is present: the handle is real; exercise destroy and stop here
      CHECK(h != nullptr && brsvd_destroy(h) == BRSVD_OK);
      std::printf("device present: failure paths of the runtime calls not exercised\n");
    } else {
      CHECK((st == BRSVD_ERR_ALLOC || st == BRSVD_ERR_HIP) && h == nullptr);
      brsvd_params hp = base_params();
      hp.a_location = BRSVD_A_HOST_PINNED;
      h = (brsvd_handle)0x1;
      const int st2 = brsvd_create(&hp, &h);
      CHECK((st2 == BRSVD_ERR_ALLOC || st2 == BRSVD_ERR_HIP) && h == nullptr);
      // caller-owned workspace: the failing create must not free it (it is not even a real allocation here)
      brsvd_params wp = base_params();
      CHECK(brsvd_workspace_bytes(&wp, &bytes) == BRSVD_OK);
      wp.workspace = (void*)0x10000;
      wp.workspace_bytes = bytes;
      h = (brsvd_handle)0x1;
      const int st3 = brsvd_create(&wp, &h);
      CHECK((st3 == BRSVD_ERR_ALLOC || st3 == BRSVD_ERR_HIP) && h == nullptr);
      wp.workspace_bytes = bytes - 1;
      CHECK(brsvd_create(&wp, &h) == BRSVD_ERR_BUDGET && h == nullptr);
      double sec = 0, work = 0;
      CHECK(brsvd_probe(0, (void*)0x10000, 1024, &sec, &work, nullptr) != BRSVD_OK);
    }
  }

  std::printf("host checks: %d run, %d failed\n", g_checks, g_failed);
  std::fflush(stdout);
  return g_failed ? 1 : 0;
}
