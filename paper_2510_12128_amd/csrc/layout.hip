// Host-side planning: argument validation, workspace layout, strip work tables.
#include <algorithm>
#include <cstring>

#include "nugpr_internal.h"

namespace nugpr {

static thread_local std::string g_last_error = "";

void set_error(const std::string& msg) { g_last_error = msg; }

const char* last_error_cstr() { return g_last_error.c_str(); }

int hip_fail(hipError_t e, const char* what) {
  set_error(std::string(what) + ": " + hipGetErrorString(e));
  (void)hipGetLastError();
  return NUGPR_ERR_HIP;
}

static size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

static size_t take(size_t& cursor, size_t bytes) {
  size_t at = align_up(cursor, 256);
  cursor = at + bytes;
  return at;
}

// Work lists of the factorisation (factor.hip).  A cluster of nt tiles has ceil(nt / 2) block columns.  A node of the tree
// inverse with children of `half` tiles takes (half / 2) x (block rows of its second child) workgroups in either product; in
// the first one a workgroup's contraction is as long as the first child on average half over, in the second one as the second.
static void plan_factor(Layout& L) {
  L.blocks_by_rank.clear();
  L.tree.clear();
  L.rows_before.assign(1, 0u);
  for (int i = 0; i < L.nc; ++i) {
    const uint32_t nb = (L.cl[L.cl[i].by_size].nt + 1) / 2;
    L.blocks_by_rank.push_back(nb);
    L.rows_before.push_back(L.rows_before.back() + nb);
  }
  for (int half = 2; half < L.ntmax; half *= 2) {
    TreeLevel t;
    t.half = half;
    t.at = (uint32_t)L.rows_before.size();
    const uint32_t hb = (uint32_t)half / 2;
    std::vector<double> work1(1, 0.0), work2(1, 0.0);
    uint32_t before = 0;
    L.rows_before.push_back(0u);
    for (int i = 0; i < L.nc; ++i) {
      const uint32_t nt = L.cl[L.cl[i].by_size].nt;
      if (nt <= (uint32_t)half) break;
      uint32_t count = 0;
      double w1 = 0.0, w2 = 0.0;
      for (uint32_t mid = (uint32_t)half; mid < nt; mid += 2 * (uint32_t)half) {
        const uint32_t rows = std::min(hb, (nt - mid + 1) / 2);
        count += hb * rows;
        w1 += (double)hb * rows * (half + 2);
        w2 += (double)hb * rows * (2 * rows + 2);
      }
      before += count;
      L.rows_before.push_back(before);
      work1.push_back(work1.back() + w1);
      work2.push_back(work2.back() + w2);
      t.ranks += 1;
    }
    // cut the list where the work of both products is an eighth each, a cluster's work spread evenly over its workgroups
    auto cut = [&](const std::vector<double>& work, uint32_t (&from)[9]) {
      for (int d = 0; d <= 8; ++d) {
        const double goal = work.back() * d / 8;
        int i = 0;
        while (i + 1 < t.ranks && work[i + 1] <= goal) ++i;
        const double part = (goal - work[i]) / (work[i + 1] - work[i]);
        const uint32_t lo = L.rows_before[t.at + i], hi = L.rows_before[t.at + i + 1];
        from[d] = d == 8 ? before : lo + (uint32_t)(std::min(1.0, part) * (hi - lo));
      }
    };
    cut(work1, t.from1);
    cut(work2, t.from2);
    L.tree.push_back(t);
  }
}

int plan_layout(const nugpr_problem* pb, uint32_t flags, Layout& L, int one_system_iter) {
  if (!pb || !pb->cluster_offsets) { set_error("null problem or cluster_offsets"); return NUGPR_ERR_INVALID; }
  if (pb->n <= 0 || pb->n > (int64_t)0x7fff0000) { set_error("n out of range"); return NUGPR_ERR_INVALID; }
  if (pb->d < 1 || pb->d > MAX_D) { set_error("d must be 1..64"); return NUGPR_ERR_INVALID; }
  if (pb->n_clusters < 1 || pb->n_clusters > 65535) { set_error("n_clusters out of range"); return NUGPR_ERR_INVALID; }
  if (pb->rank < 1) { set_error("rank must be >= 1"); return NUGPR_ERR_INVALID; }
  if (pb->n_probes < 0 || pb->n_probes > MAX_COLS - 1) { set_error("n_probes must be 0..32"); return NUGPR_ERR_INVALID; }
  const int64_t* off = pb->cluster_offsets;
  if (off[0] != 0 || off[pb->n_clusters] != pb->n) { set_error("cluster_offsets must start at 0 and end at n"); return NUGPR_ERR_INVALID; }
  L = Layout();
  L.n = pb->n; L.d = pb->d; L.nc = pb->n_clusters; L.r = pb->rank; L.t = pb->n_probes;
  L.T = L.t + 1;
  L.p = (flags & NUGPR_ISOTROPIC) ? 3 : L.d + 2;
  L.max_iter = one_system_iter > 0 ? one_system_iter : MAX_ITER_CAP;          // rows of the coefficient logs
  L.compensate = (flags & NUGPR_COMPENSATE) != 0;
  if ((int64_t)L.nc * L.r > (int64_t)1 << 24) { set_error("n_clusters*rank too large"); return NUGPR_ERR_INVALID; }
  L.ncr = L.nc * L.r;
  L.ldc = (int)align_up(L.ncr, TILE);
  L.ldw = (int)align_up(L.r, TILE);
  L.cl.resize(L.nc);
  uint64_t koff = 0, wtoff = 0, prow = 0;
  for (int i = 0; i < L.nc; ++i) {
    int64_t b = off[i + 1] - off[i];
    if (b < L.r) { set_error("a cluster is smaller than rank (or offsets not ascending)"); return NUGPR_ERR_INVALID; }
    if (b > 64 * 4096) { set_error("cluster too large"); return NUGPR_ERR_INVALID; }
    ClusterInfo& c = L.cl[i];
    c.row0 = (uint32_t)off[i];
    c.b = (uint32_t)b;
    c.ld = (uint32_t)align_up((size_t)b, TILE);
    c.nt = c.ld / TILE;
    c.koff = koff;
    c.wtoff = wtoff;
    c.prow = (uint32_t)prow;
    prow += c.ld;
    koff += (uint64_t)c.ld * c.ld;
    wtoff += (uint64_t)L.r * c.ld;
    L.ntmax = std::max<int>(L.ntmax, (int)c.nt);
    L.n_diag_tiles += (uint64_t)c.nt * (c.nt + 1) / 2;
  }
  {
    std::vector<uint32_t> order(L.nc);
    for (int i = 0; i < L.nc; ++i) order[i] = (uint32_t)i;
    std::stable_sort(order.begin(), order.end(), [&](uint32_t a, uint32_t b) { return L.cl[a].b > L.cl[b].b; });
    for (int i = 0; i < L.nc; ++i) L.cl[i].by_size = order[i];
    plan_factor(L);
  }
  L.kd_elems = koff;
  L.rows_pad = prow;
  if (prow > 0xffffffffull) { set_error("padded row count out of range"); return NUGPR_ERR_INVALID; }
  L.wt_elems = wtoff;
  {
    uint64_t ct = (uint64_t)L.ldc / TILE;
    L.n_c_tiles = ct * (ct + 1) / 2;
  }
  // how many column slabs the two reductions over long rows are split into
  {
    int strips_S = L.nc * ((L.r + TILE - 1) / TILE);
    int want = (1024 + strips_S - 1) / strips_S;
    int min_chunks = 1 << 30;
    for (auto& c : L.cl) min_chunks = std::min<int>(min_chunks, (int)c.nt);
    L.nsS = std::max(1, std::min({want, 8, min_chunks}));
    int strips_P = L.ldc / TILE;
    want = (2048 + strips_P - 1) / strips_P;
    L.nsP = std::max(1, std::min({want, 16, L.ldc / TILE}));
  }
  // workgroups (= partial sums per column) of the kernels with dot products: 64 rows each up to 8192 points (a loss at
  // 4096 points 161 us, with 128 rows 169; at 8192 points 260 / 281), 128 beyond (training step at 32768 points 5821 us,
  // 6408 with 256: half of the chip idle).  The line could lie higher: with 64 rows a loss at 12288 points takes 275 us in
  // place of 295, at 16384 298 / 318, and that training step 5566, though its sums are then too many for FUSE_BLOCKS.
  L.n_dot_blocks = L.n <= 8192 ? (int)((L.n + 63) / 64) : (int)std::min<int64_t>(1024, (L.n + 127) / 128);

  size_t cur = 0;
  const size_t f = sizeof(float);
  const size_t vec = (size_t)L.n * L.T * sizeof(double);      // fp64 vector blocks (fp32 mode uses half)
  L.o_cl = take(cur, sizeof(ClusterInfo) * L.nc);
  L.o_rows_before = take(cur, L.rows_before.size() * sizeof(uint32_t));        // (right behind: one upload)
  L.o_Kd = take(cur, L.kd_elems * f);
  L.o_G = take(cur, L.kd_elems * f);
  L.o_C = take(cur, (size_t)L.ldc * L.ldc * f);
  L.o_Kd2 = take(cur, L.kd_elems * f);
  L.o_C2 = take(cur, (size_t)L.ldc * L.ldc * f);
  L.o_Wd = take(cur, (size_t)L.n * L.ldw * f);
  L.o_Wt = take(cur, L.wt_elems * f);
  L.o_reps = take(cur, (size_t)L.ncr * L.d * f);
  {
    const size_t kd = (size_t)((L.d + 3) & ~3);
    L.o_Xs = take(cur, (size_t)L.rows_pad * kd * sizeof(double));
    L.o_Xn = take(cur, (size_t)L.rows_pad * sizeof(double));
    L.o_Rs = take(cur, (size_t)L.ldc * kd * sizeof(double));
    L.o_Rn = take(cur, (size_t)L.ldc * sizeof(double));
  }
  // residual matrix of the compensated coupling; reserved whenever the problem is small enough for the
  // compensation, so that the workspace size does not depend on the flags
  // (larger couplings keep it in the spare coupling matrix, which only the pair assembly uses and the
  // compensation does without)
  if (L.ncr <= COMPENSATE_HOST_MAX) L.o_Clo = take(cur, (size_t)L.ldc * L.ldc * sizeof(float));
  if (L.ncr > COMPENSATE_HOST_MAX) L.o_dav = take(cur, eigmin_workspace_doubles((size_t)L.ldc, (size_t)L.ncr) * sizeof(double));
  L.o_assign = take(cur, (size_t)L.n * sizeof(int32_t));
  L.o_rep_ptr = take(cur, ((size_t)L.ncr + 1) * sizeof(int32_t));
  L.o_rep_pts = take(cur, (size_t)L.n * sizeof(int32_t));
  L.o_B = take(cur, vec);
  L.o_x0 = take(cur, (size_t)L.n * sizeof(double));
  L.o_Z0 = take(cur, vec);
  L.o_P = take(cur, vec);
  L.o_Q0 = take(cur, vec);
  L.o_S0 = take(cur, (size_t)L.ncr * L.T * sizeof(double));
  // The blocks of a solve, once per system that can be taken side by side.  Up to 32768 points (256 partial sums a dot product):
  // there a launch of one system leaves most of the chip idle.
  L.slots = L.n_dot_blocks <= 256 && one_system_iter <= 0 ? MAX_SLOTS : 1;
  // Their logs share the rows of one solve at the cap between them: a context that allows a solve more than its share takes one
  // system at a time.
  L.slot_iter = L.max_iter / L.slots;
  cur = align_up(cur, 256);
  const size_t slot0 = cur;
  L.o_X = take(cur, vec);
  L.o_R = take(cur, vec);
  L.o_Z = take(cur, vec);
  L.o_D = take(cur, vec);
  L.o_Q = take(cur, vec);
  L.o_V = take(cur, vec);
  L.o_U = take(cur, vec);
  // (the slabs, or one and behind it a byte for every few rows: odd_offset)
  L.o_Spart = take(cur, std::max((size_t)L.nsS * L.ncr * L.T * sizeof(double),
                                 align_up((size_t)L.ncr * L.T * sizeof(double), 256) + (size_t)L.ncr));
  L.o_Ppart = take(cur, (size_t)L.nsP * L.ncr * L.T * sizeof(double));
  L.o_dot = take(cur, (size_t)4 * L.n_dot_blocks * MAX_COLS * sizeof(double));
  L.o_state = take(cur, sizeof(PcgState));
  L.o_alog = take(cur, (size_t)L.slot_iter * MAX_COLS * sizeof(double));
  L.o_blog = take(cur, (size_t)L.slot_iter * MAX_COLS * sizeof(double));
  cur = align_up(cur, 256);
  L.slot_bytes = cur - slot0;
  cur = slot0 + L.slots * L.slot_bytes;
  L.o_logdet = take(cur, (size_t)L.nc * sizeof(double));
  // tile list of the diagonal blocks (mirroring) + row-panel work items of the two assembly launches
  // tile list of the diagonal blocks + the assembly work items (32 bytes each, at most one per tile)
  L.o_tiles = take(cur, (5 * L.n_diag_tiles + 4 * L.n_c_tiles) * sizeof(uint64_t));
  // strip tables: exact item counts
  size_t items = 0;
  for (auto& c : L.cl) {
    items += (size_t)((L.r + TILE - 1) / TILE) * L.nsS;  // Wt * D
    items += c.nt;                                       // K_ii * D
    items += c.nt;                                       // W * P
    items += 3 * (size_t)c.nt;                           // tril(G), triu(G), tril(L)
  }
  items += 2 * (size_t)(L.ldc / TILE) * L.nsP;           // C * S, in the joint table and on its own
  L.items_bytes = items * sizeof(StripItem);
  L.o_items = take(cur, L.items_bytes);
  // Behind all the rest: a size that is no multiple of a page in front of the vector blocks costs their accesses.  Product of 9 / 17
  // columns, 128 clusters of 256 points, 8 representatives each, behind C2 / here: 28.6 / 27.6 us, 31.5 / 30.9.
  L.o_c_live = take(cur, 2 * L.n_c_tiles * sizeof(uint32_t));
  L.total = align_up(cur, 256);
  return NUGPR_OK;
}

}  // namespace nugpr
