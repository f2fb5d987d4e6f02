// kb_launch.hpp -- the kernel sequence of one build, enqueued on the caller's stream.
//
// Templates over the element and the precision; kb_f64.hip, kb_f32.hip and kb_f32fb.hip
// each instantiate one precision (compiled side by side), kb_api.hip calls them.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "kb_assemble.hpp"
#include "kb_kernels.hpp"
#include "kbuild.h"

namespace kb {

constexpr size_t kAlign = 256;
constexpr float kDefaultTau = 16.0f;
constexpr int kDefaultBlock = 256;
// pairs per pass-2 segment: the short one keeps three scatter workgroups per CU, the long
// one (one per CU) is taken for tetrahedra when a segment would otherwise give runs of
// fewer than kMinRun pairs per sub-bucket (measured: 18% faster scatter on the 20M-tet
// mesh, 35% slower on brick meshes with the same sub-bucket counts)
constexpr int kSeg = 4096, kSegLong = 8192, kMinRun = 16;
constexpr int kSegThreads = 512;   // threads per pass-2 scatter workgroup
constexpr int kTargetBuckets = 256;  // first-level buckets (pass-1 run length)
constexpr double kSubEntries = 300;   // target distinct entries per sub-bucket
constexpr double kDirectLoad = 0.46;  // of pass 3's table, at most, on the direct way
// (and only where there are more sub-buckets than the device takes at once: fewer, larger ones
// are then one round of longer workgroups.  64 small boxes of tetrahedra, 1755 sub-buckets: 109 us
// against 120, in random order, where rows are of unlike length, 112 against 161; 128 boxes of
// bricks, 27,449: 299 against 278, in random order 362 against 344)
constexpr int64_t kWideSubs = 4096;
constexpr int kHTMin = 512, kHTMax = 4096;
// the direct way for small meshes: at most kDirectRuns runs (tiles x sub-buckets), each of
// which may take a global atomic when counted and when written (72,000 tets in random order,
// 481,000 runs: counting and pass 1 82 us against 22 on two levels, whose other kernels and
// launches cost 48), and tiles small enough to give every compute unit one
constexpr int64_t kDirectRuns = 1 << 18;
constexpr int64_t kDirectTiles = 256;
// elements that a workgroup of k_count takes (in whole tiles), as long as kCountGroups
// workgroups per CU are left
constexpr int64_t kCountElems = 1024;
constexpr int64_t kCountGroups = 16;
constexpr int64_t kPadGroups = 16;  // workgroups per CU that pad the coordinates beside it
constexpr int64_t kPadFirst = 1 << 20;  // nodes padded beside the sampling
constexpr int kSmallTile = 64;
constexpr double kHalfTileRatio = 16;   // pairs per tile x bucket histogram entry
constexpr size_t kWideStage = 112640;  // staged pair bytes per pass-1 tile, elements of > 8 rows

inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }
inline int64_t div_up(int64_t a, int64_t b) { return (a + b - 1) / b; }

struct Plan {
  int nen = 0, te = 0, prec = 0, block = kDefaultBlock;
  int op = KB_OP_STIFFNESS;            // element integrand
  int dof = 1;                         // degrees of freedom per node (assembly only)
  float tau = kDefaultTau;
  int64_t nel = 0, nn = 0, T = 0;
  size_t vbytes = 8;
  // assembly geometry
  int s1 = 0, s2 = 0, p2 = 1, nb = 0;  // bucket / sub-bucket shifts, sub-buckets per bucket, buckets
  int s2d = 0;                         // sub-bucket shift of the direct way
  int colbits = 1;                     // bits of a column index
  int ht = 2048;                       // pass-3 hash slots
  int seg = kSeg;                      // pairs per pass-2 segment
  int tile = 0;                        // elements (= threads) per pass-1 workgroup
  int mode = kTwoLevel;                // where pass 1 sends its pairs
  int cus = 256;                       // compute units of the current device (launch time)
  int64_t ntiles = 0, nsub = 0, nsub_d = 0, nhist = 0, nseg_max = 0;
  int64_t csr_cap = 0, ntiles_csr = 0;  // running sums read back as pairs (grouped builds)
  size_t lds1 = 0, lds2 = 0, lds_csr = 0;
  // workspace offsets
  size_t o_coords4 = 0, o_hist = 0, o_csum = 0, o_tot = 0, o_part = 0, o_bstart = 0, o_segbase = 0, o_hist2 = 0,
         o_seg2b = 0, o_head = 0, o_dconn = 0, o_ovl = 0, o_hvy = 0, o_tres = 0, o_row1 = 0, o_col1 = 0, o_val1 = 0,
         o_key2 = 0, o_val2 = 0, o_sbb = 0, o_rowoff = 0, o_usub = 0, o_ubase = 0, total = 0;
};

struct Events {
  void** ev;
  hipStream_t s;
  int rec(int i) {
    if (!ev) return KB_OK;
    return hipEventRecord((hipEvent_t)ev[i], s) == hipSuccess ? KB_OK : KB_EHIP;
  }
};

#define KB_LAUNCH_CHECK()                                   \
  do {                                                      \
    if (hipGetLastError() != hipSuccess) return KB_EHIP;    \
  } while (0)
#define KB_TRY(x)                  \
  do {                             \
    int _r = (x);                  \
    if (_r != KB_OK) return _r;    \
  } while (0)

inline unsigned grid_for(int64_t n, int block) { return (unsigned)div_up(n, block); }

template <typename K>
bool set_lds(K kernel, size_t bytes) {
  return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) ==
         hipSuccess;
}

// (with as many sub-buckets either way, nothing has to know which was taken)
inline SubBuckets sub_buckets(const Plan& p, unsigned char* ws) {
  return SubBuckets{{p.s2, p.s2d},
                    {(int)p.nsub, (int)p.nsub_d},
                    p.nsub == p.nsub_d ? (int)kTwoLevel : p.mode,
                    (const uint32_t*)(ws + p.o_head) + kHeadWay};
}

template <typename V>
PairOut<V> pair_out(const Plan& p, unsigned char* ws) {
  return PairOut<V>{(uint16_t*)(ws + p.o_row1),
                    (uint32_t*)(ws + p.o_col1),
                    (V*)(ws + p.o_val1),
                    (const uint32_t*)(ws + p.o_hist),
                    (uint32_t*)(ws + p.o_key2),
                    (V*)(ws + p.o_val2),
                    (uint32_t*)(ws + p.o_hist2),
                    (const uint32_t*)(ws + p.o_head) + kHeadWay,
                    p.mode,
                    p.s1,
                    p.nb,
                    p.s2d,
                    (int)p.nsub_d,
                    p.colbits};
}

// persistent workgroups of pass 1: those that fit on the device at once (LDS-bound), at
// least one per XCD slot (b % 8) that owns tiles
inline unsigned persistent_grid(const Plan& p, int threads, int64_t ntiles) {
  const int per_cu = std::max(1, (int)(163840 / std::max<size_t>(p.lds1, 1)));
  return (unsigned)std::min<int64_t>(ntiles,
                                     std::max<int64_t>(8, (int64_t)p.cus * std::min(per_cu, 2048 / threads)));
}

// their grid where a workgroup per tile may be the better choice (TileWalk): the others
// return, about 0.4 ns each, so only with so many buckets that a random tile's runs are short
inline unsigned walk_grid(const Plan& p, unsigned persist, int64_t ntiles) {
  return p.mode == kAsk && p.nb > 2 * kTargetBuckets ? (unsigned)std::max<int64_t>(persist, ntiles) : persist;
}

template <int NEN, Prec P, bool FROM_VALUES, int BLOCK, Op OP>
int launch_pass1_block(const Plan& p, const kb_mesh* m, const void* klow, unsigned char* ws, uint32_t* status,
                       hipStream_t s) {
  using V = typename PrecTraits<P>::V;
  const PairOut<V> o = pair_out<V>(p, ws);
  auto* emax = (uint32_t*)(ws + p.o_head);
  auto* coords4 = (const double4*)(ws + p.o_coords4);
  if constexpr (NEN == 8 && !FROM_VALUES && OP == Op::Stiffness && P != Prec::F64) {
    // bricks in FP32: a lane pair per element, 2 * BLOCK lanes for a tile of BLOCK elements
    // (in FP64 the pair kernel sits at the register limit and was slower on 1M bricks)
    auto kern = k_pass1_pair<P, 2 * BLOCK>;
    if (!set_lds(kern, p.lds1)) return KB_EHIP;
    const unsigned persist = persistent_grid(p, 2 * BLOCK, p.ntiles);
    kern<<<walk_grid(p, persist, p.ntiles), 2 * BLOCK, p.lds1, s>>>(m->conn, m->coords, coords4, m->coef, p.nel, p.nn,
                                                                    p.tau, p.ntiles, o, emax, status, persist);
    KB_LAUNCH_CHECK();
    return KB_OK;
  }
  if constexpr (NEN == 8 && !FROM_VALUES && P == Prec::F64 && BLOCK > kSmallTile) {
    // bricks in FP64: two tiles per workgroup (two waves per SIMD while integrating)
    auto kern = k_pass1_two<NEN, P, BLOCK, OP>;
    if (!set_lds(kern, p.lds1)) return KB_EHIP;
    const int64_t n2 = div_up(p.ntiles, 2);
    const unsigned persist = persistent_grid(p, 2 * BLOCK, n2);
    kern<<<walk_grid(p, persist, n2), 2 * BLOCK, p.lds1, s>>>(m->conn, m->coords, coords4, m->coef, p.nel, p.nn, p.tau,
                                                              p.ntiles, o, emax, status, persist);
    KB_LAUNCH_CHECK();
    return KB_OK;
  }
  if constexpr (NEN == 8) {
    auto kern = k_pass1<NEN, P, FROM_VALUES, BLOCK, OP>;
    if (!set_lds(kern, p.lds1)) return KB_EHIP;
    kern<<<(unsigned)p.ntiles, BLOCK, p.lds1, s>>>(m->conn, m->coords, coords4, m->coef, (const V*)klow, p.nel, p.nn,
                                                   p.tau, o, emax, status);
  } else {
    // tetrahedra: persistent
    auto kern = k_pass1_tet<P, FROM_VALUES, BLOCK, OP>;
    if (!set_lds(kern, p.lds1)) return KB_EHIP;
    kern<<<persistent_grid(p, BLOCK, p.ntiles), BLOCK, p.lds1, s>>>(m->conn, m->coords, coords4, m->coef,
                                                                    (const V*)klow, p.nel, p.nn, p.tau, p.ntiles, o,
                                                                    emax, status);
  }
  KB_LAUNCH_CHECK();
  return KB_OK;
}

// pass-1 tile sizes (elements = lanes per workgroup): {small, default} per element and
// value size, and kSmallTile; the staging LDS is tile * pairs * (8 + value bytes)
template <int NEN, Prec P>
struct TileSizes {
  static constexpr int big = NEN == 4 ? (P == Prec::F64 ? 768 : 1024) : 256;
  static constexpr int mid = NEN == 8 && P == Prec::F64 ? 192 : 0;  // FP64, many buckets
  static constexpr int small = big / 2 >= 64 && (big / 2) % 64 == 0 ? big / 2 : 64 * ((big / 2 + 63) / 64);
};

// elements of more than 8 rows: `tile` elements on kWideThreads threads, one tile per workgroup
template <int NEN, typename V>
int launch_pass1_wide(const Plan& p, const kb_mesh* m, const void* klow, unsigned char* ws, uint32_t* status,
                      hipStream_t s) {
  auto kern = k_pass1_wide<NEN, V>;
  if (!set_lds(kern, p.lds1)) return KB_EHIP;
  kern<<<(unsigned)p.ntiles, kWideThreads, p.lds1, s>>>(m->conn, (const V*)klow, p.nel, p.nn, p.tile,
                                                        pair_out<V>(p, ws), (uint32_t*)(ws + p.o_head), status);
  KB_LAUNCH_CHECK();
  return KB_OK;
}

// OP: the integrand of pass 1 when the values are not given
template <int NEN, Prec P, bool FROM_VALUES, Op OP = Op::Stiffness>
int launch_pass1(const Plan& p, const kb_mesh* m, const void* klow, unsigned char* ws, uint32_t* status,
                 hipStream_t s) {
  if constexpr (NEN > 8) {
    static_assert(FROM_VALUES, "elements of more than 8 rows are assembled from given values");
    return launch_pass1_wide<NEN, typename PrecTraits<P>::V>(p, m, klow, ws, status, s);
  } else {
    if (p.tile == TileSizes<NEN, P>::big)
      return launch_pass1_block<NEN, P, FROM_VALUES, TileSizes<NEN, P>::big, OP>(p, m, klow, ws, status, s);
    if (p.tile == TileSizes<NEN, P>::small)
      return launch_pass1_block<NEN, P, FROM_VALUES, TileSizes<NEN, P>::small, OP>(p, m, klow, ws, status, s);
    if (p.tile == kSmallTile)
      return launch_pass1_block<NEN, P, FROM_VALUES, kSmallTile, OP>(p, m, klow, ws, status, s);
    if constexpr (TileSizes<NEN, P>::mid > 0) {
      if (p.tile == TileSizes<NEN, P>::mid)
        return launch_pass1_block<NEN, P, FROM_VALUES, TileSizes<NEN, P>::mid, OP>(p, m, klow, ws, status, s);
    }
    return KB_EINVAL;
  }
}

// Running sums of a grouped build: read back as a second source of pairs (in), and the
// pass's entries written with their residuals and rows (out).
struct Carry {
  bool first = true;              // first pass: the status words are initialised
  const int32_t* rows = nullptr;  // in: rows, columns, values, residuals of the entries
  const int32_t* cols = nullptr;
  const void* vals = nullptr;
  const void* res = nullptr;
  const int64_t* nnz = nullptr;   // in: number of entries (device); nullptr: no input
  void* res_out = nullptr;        // out: residuals and rows of the pass's entries
  int32_t* rows_out = nullptr;
};

// a build so small that its heavy sub-buckets are reduced by teams of one launch
inline bool heavy_teams(const Plan& p) { return p.T <= kHeavySplitPairs; }

// pass 3, then the sub-buckets it could not hold (in parts; k_heavy, which returns at once when there
// are none; its last launch scans the entry counts of few sub-buckets into ubase and nnz)
template <typename V, bool RES>
int launch_pass3(const Plan& p, unsigned char* ws, V* tres, int64_t* nnz_dev, hipStream_t s) {
  auto* key2 = (uint32_t*)(ws + p.o_key2);
  auto* val2 = (V*)(ws + p.o_val2);
  auto* sbb = (uint32_t*)(ws + p.o_sbb);
  auto* head = (uint32_t*)(ws + p.o_head);
  auto* tcol = (int32_t*)(ws + p.o_col1);
  auto* tval = (V*)(ws + p.o_val1);
  auto* rowoff = (uint32_t*)(ws + p.o_rowoff);
  auto* usub = (uint32_t*)(ws + p.o_usub);
  auto* ov_list = (uint32_t*)(ws + p.o_ovl);
  const SubBuckets sub = sub_buckets(p, ws);
  const size_t lds3 = (size_t)8 << std::max(p.s2, p.s2d);
  const bool parts = p.mode == kAsk && p.s2d > p.s2;
  // (the list of k_pass3_parts lies where the scan of the entry counts goes later)
  auto* list = parts ? (uint32_t*)(ws + p.o_ubase) : ov_list;
  uint32_t* const count = head + (parts ? 4 : 1);
  const auto reduce = [&](auto slots) {
    constexpr int HT = decltype(slots)::value;
    k_pass3<V, HT, RES><<<(unsigned)p.nsub, kPass3Threads, lds3, s>>>(
        key2, val2, sbb, sub, p.colbits, p.nn, head, tcol, tval, tres, rowoff, usub, list, count);
    KB_LAUNCH_CHECK();
    if (parts) {
      k_pass3_parts<V, HT, RES><<<(unsigned)std::min<int64_t>(p.nsub, (int64_t)kPartsGroups * std::max(1, p.cus)),
                                  kPass3Threads, lds3, s>>>(key2, val2, sbb, sub, p.colbits, p.nn, head, tcol, tval,
                                                            tres, rowoff, usub, list, count, ov_list, head + 1);
      KB_LAUNCH_CHECK();
    }
    return (int)KB_OK;
  };
  switch (p.ht) {
    case 512: KB_TRY(reduce(std::integral_constant<int, 512>{})); break;
    case 1024: KB_TRY(reduce(std::integral_constant<int, 1024>{})); break;
    case 2048: KB_TRY(reduce(std::integral_constant<int, 2048>{})); break;
    default: KB_TRY(reduce(std::integral_constant<int, 4096>{}));
  }
  const HeavyArgs<V> A{key2, val2, (uint32_t*)tcol, tval, tres, sbb, sub, p.s2, p.colbits, p.nn, 0, rowoff, usub,
                       ov_list, 0, 0, (uint32_t*)(ws + p.o_hvy)};
  uint32_t* const ubase = p.nsub <= kScanHere ? (uint32_t*)(ws + p.o_ubase) : nullptr;
  const unsigned cus = (unsigned)std::max(1, p.cus);
  auto phase = [&](auto kern, unsigned grid, size_t lds) {
    if (!set_lds(kern, lds)) return (int)KB_EHIP;
    kern<<<grid, kHeavyThreads, lds, s>>>(A, head, head + 1, (uint32_t)kHeavyPar, head + 2, ubase, nnz_dev);
    return hipGetLastError() == hipSuccess ? (int)KB_OK : (int)KB_EHIP;
  };
  constexpr size_t kTabLds = 4 * (size_t)(kHvyDigits + 2 * kHvyRows + 1 + kHeavyThreads / 64 + 1);
  if (heavy_teams(p))  // (at least a workgroup for each of the sub-buckets that a team may take)
    return phase(k_heavy<V, RES, kHeavyTeamPhase, true>,
                 std::max<unsigned>(kHeavyPar, (unsigned)std::min<int64_t>(p.nsub, cus)), HeavySmem::bytes());
  KB_TRY(phase(k_heavy<V, RES, kHeavyRowsPhase>, 2 * cus, kTabLds));
  KB_TRY(phase(k_heavy<V, RES, kHeavyHistPhase>, 2 * cus, kTabLds));
  KB_TRY(phase(k_heavy<V, RES, kHeavyScatterPhase>, 2 * cus, kTabLds));
  KB_TRY(phase(k_heavy<V, RES, kHeavyBigPhase>, cus, HeavySmem::bytes()));
  KB_TRY(phase(k_heavy<V, RES, kHeavyRangesPhase>, cus, HeavySmem::bytes()));
  return phase(k_heavy<V, RES, kHeavyFinishPhase, true>, kHeavyPar, kTabLds);
}

template <typename V>
int assemble_tail(const Plan& p, unsigned char* ws, int32_t* row_ptr, int32_t* col_idx, V* vals, int64_t cap,
                  int64_t* nnz_dev, uint32_t* status, Events& ev, hipStream_t s, const Carry* cr, const BatchRows* br) {
  auto* bstart = (uint32_t*)(ws + p.o_bstart);
  auto* segbase = (uint32_t*)(ws + p.o_segbase);
  auto* hist2 = (uint32_t*)(ws + p.o_hist2);
  auto* seg2b = (uint32_t*)(ws + p.o_seg2b);
  auto* head = (uint32_t*)(ws + p.o_head);
  auto* row1 = (uint16_t*)(ws + p.o_row1);
  auto* col1 = (uint32_t*)(ws + p.o_col1);
  auto* val1 = (V*)(ws + p.o_val1);
  auto* key2 = (uint32_t*)(ws + p.o_key2);
  auto* val2 = (V*)(ws + p.o_val2);
  auto* sbb = (uint32_t*)(ws + p.o_sbb);
  auto* usub = (int32_t*)(ws + p.o_usub);
  auto* ubase = (uint32_t*)(ws + p.o_ubase);
  auto* part = (int32_t*)(ws + p.o_part);
  const uint32_t* way = head + kHeadWay;
  const bool two = p.nb > 0 && p.mode != kDirect;
  KB_TRY(ev.rec(KB_STAGE_HISTOGRAM));
  if (two) {
    const unsigned gs = (unsigned)p.nseg_max;
    if (p.seg == kSegLong)
      k_hist2<kSegLong><<<gs, 256, 4 * (size_t)p.p2, s>>>(row1, bstart, segbase, seg2b, p.nb, p.s2, p.p2, hist2, p.mode,
                                                          way);
    else
      k_hist2<kSeg><<<gs, 256, 4 * (size_t)p.p2, s>>>(row1, bstart, segbase, seg2b, p.nb, p.s2, p.p2, hist2, p.mode,
                                                      way);
    KB_LAUNCH_CHECK();
    k_colscan<<<(unsigned)p.nb, 256, 0, s>>>(hist2, bstart, segbase, p.nb, p.p2, sbb, p.mode, way);
    KB_LAUNCH_CHECK();
  }
  KB_TRY(ev.rec(KB_STAGE_PARTITION));
  if (two) {
    const unsigned gs = (unsigned)p.nseg_max;
    auto k2 = p.seg == kSegLong ? k_scatter2<V, kSegLong, kSegThreads> : k_scatter2<V, kSeg, kSegThreads>;
    if (!set_lds(k2, p.lds2)) return KB_EHIP;
    k2<<<gs, kSegThreads, p.lds2, s>>>(row1, col1, val1, bstart, segbase, seg2b, hist2, sbb, p.nb, p.s2, p.p2,
                                      p.colbits, key2, val2, p.mode, way);
    KB_LAUNCH_CHECK();
  }
  // pass-3 output reuses the pass-1 buffers (dead after pass 2)
  auto* tres = (V*)(ws + p.o_tres);
  KB_TRY(ev.rec(KB_STAGE_REDUCE));
  if (p.nsub > 0) {
    if (cr)
      KB_TRY((launch_pass3<V, true>(p, ws, tres, nnz_dev, s)));
    else
      KB_TRY((launch_pass3<V, false>(p, ws, nullptr, nnz_dev, s)));
  }
  KB_TRY(ev.rec(KB_STAGE_COMPRESS));
  if (p.nsub > 0) {
    const SubBuckets sub = sub_buckets(p, ws);
    if (p.nsub > kScanHere) {
      const unsigned g = grid_for(p.nsub, kScanChunk);
      k_scan_partials<<<g, kScanThreads, 0, s>>>(usub, sub, part);
      KB_LAUNCH_CHECK();
      k_scan_down<<<g, kScanThreads, 0, s>>>(usub, sub, part, (int32_t*)ubase, nnz_dev);
      KB_LAUNCH_CHECK();
    }
    const unsigned gf = (unsigned)div_up(p.nsub, 4) + kFinalHeavyGrid;
    auto* tcol = (const int32_t*)col1;
    auto* tval = (const V*)val1;
    auto* rowoff = (const uint32_t*)(ws + p.o_rowoff);
    auto* ov_list = (const uint32_t*)(ws + p.o_ovl);
    auto* hvy = (const uint32_t*)(ws + p.o_hvy);
    const uint32_t par = kHeavyPar;
    if (br)
      k_final<V, false, true><<<gf, 256, 0, s>>>(sbb, ubase, tcol, tval, nullptr, rowoff, sub, p.nn, row_ptr, col_idx,
                                                 vals, nullptr, nullptr, cap, status, ov_list, head + 1, hvy, par, *br);
    else if (cr)
      k_final<V, true><<<gf, 256, 0, s>>>(sbb, ubase, tcol, tval, tres, rowoff, sub, p.nn, row_ptr, col_idx,
                                          vals, (V*)cr->res_out, cr->rows_out, cap, status, ov_list, head + 1, hvy, par,
                                          BatchRows{});
    else
      k_final<V><<<gf, 256, 0, s>>>(sbb, ubase, tcol, tval, nullptr, rowoff, sub, p.nn, row_ptr, col_idx,
                                    vals, nullptr, nullptr, cap, status, ov_list, head + 1, hvy, par, BatchRows{});
    KB_LAUNCH_CHECK();
  } else {
    k_scan_empty<<<1, 1, 0, s>>>(br ? nullptr : row_ptr, nnz_dev);
    KB_LAUNCH_CHECK();
  }
  KB_TRY(ev.rec(KB_N_STAGES));
  return KB_OK;
}

template <int NEN, Prec P>
int build_impl(const Plan& p, const kb_mesh* m, const void* klow, unsigned char* ws, int32_t* row_ptr,
               int32_t* col_idx, void* vals, int64_t cap, int64_t* nnz_dev, uint32_t* status, Events& ev,
               hipStream_t s, const Carry* cr = nullptr, const BatchRows* br = nullptr) {
  using V = typename PrecTraits<P>::V;
  auto* hist = (uint32_t*)(ws + p.o_hist);
  auto* csum = (uint32_t*)(ws + p.o_csum);
  auto* tot = (uint32_t*)(ws + p.o_tot);
  auto* part = (int32_t*)(ws + p.o_part);
  auto* bstart = (uint32_t*)(ws + p.o_bstart);
  auto* segbase = (uint32_t*)(ws + p.o_segbase);
  auto* seg2b = (uint32_t*)(ws + p.o_seg2b);
  auto* subcnt = (uint32_t*)(ws + p.o_hist2);
  auto* sbb = (uint32_t*)(ws + p.o_sbb);
  auto* head = (uint32_t*)(ws + p.o_head);
  const uint32_t* way = head + kHeadWay;

  // tiles of running sums read back (grouped builds) follow the element tiles
  const int64_t ntc = (cr && cr->nnz && p.nb > 0) ? p.ntiles_csr : 0;
  const int64_t nt_all = p.ntiles + ntc;
  // coordinates padded: the first of them by k_begin, the others by k_count
  const int64_t n_pad = p.ntiles > 0 && p.mode != kDirect && p.nb > 0 && !klow ? p.nn : 0;
  const int64_t pad0 = std::min<int64_t>(n_pad, kPadFirst);
  KB_TRY(ev.rec(KB_STAGE_INIT));
  {
    const bool first = !cr || cr->first;
    auto* hvy = (uint32_t*)(ws + p.o_hvy);
    const int n_zero = heavy_teams(p) ? 1 : kHvyRows;
    const int64_t n = std::max<int64_t>({pad0, p.mode != kTwoLevel ? p.nsub_d : 0, (int64_t)n_zero * kHeavyPar});
    k_begin<NEN><<<(unsigned)(kSamples + std::min<int64_t>(div_up(n, 256), 8192)), 256, 0, s>>>(
        m->conn, p.nel, p.nn, p.tile, p.ntiles, p.s2d, p.mode, first ? status : nullptr, first ? nnz_dev : nullptr,
        head, subcnt, p.nsub_d, m->coords, (double4*)(ws + p.o_coords4), pad0,
        hvy + (heavy_teams(p) ? HeavyTable::kTeamAt : HeavyTable::kRpairAt), kHeavyPar, kHvyWords, n_zero);
    KB_LAUNCH_CHECK();
  }

  KB_TRY(ev.rec(KB_STAGE_COUNT));
  // LDS words of the counting kernels' slots
  const size_t slots = p.mode == kDirect ? (size_t)p.nsub_d
                       : p.mode == kAsk  ? std::max<size_t>(2 * kSlotsHash, (size_t)p.nb)
                                         : (size_t)std::max(p.nb, 1);
  if (p.ntiles > 0) {
    // with no nodes every element has an index error: flagged, nothing counted
    const int per = (int)std::max<int64_t>(
        1, std::min<int64_t>(kCountElems / p.tile, p.ntiles / (kCountGroups * (int64_t)p.cus)));
    const size_t ids = NEN > 8 ? (size_t)p.tile * (NEN + 1) : 0;
    const int64_t n_count = div_up(p.ntiles, per);
    const int64_t pad_groups = std::min<int64_t>(div_up(n_pad - pad0, 256), kPadGroups * (int64_t)p.cus);
    k_count<NEN><<<(unsigned)(pad_groups + n_count), 256, 4 * (slots + ids), s>>>(
        m->conn, p.nel, p.nn, p.tile, p.ntiles, per, (int)slots, p.nb > 0 ? p.s1 : 30, p.nb, p.s2d, (int)p.nsub_d,
        p.mode, head, hist, subcnt, sbb, status, (uint32_t)pad_groups, m->coords, (double4*)(ws + p.o_coords4), pad0);
    KB_LAUNCH_CHECK();
  }
  if (ntc > 0) {
    k_hist_csr<<<(unsigned)ntc, kCsrThreads, 4 * slots, s>>>(cr->rows, cr->nnz, p.csr_cap, p.nn, p.s1, p.nb, p.s2d,
                                                             (int)p.nsub_d, p.mode, way, hist + p.ntiles * p.nb,
                                                             subcnt);
    KB_LAUNCH_CHECK();
  }
  KB_TRY(ev.rec(KB_STAGE_OFFSETS));
  if (p.nb > 0 && p.mode != kDirect) {
    const int64_t nchunk = div_up(nt_all, kColChunk), nsc = p.mode == kAsk ? div_up(p.nsub_d, kScanChunk) : 0;
    const int64_t gc = nchunk * div_up(p.nb, 256);
    if (std::max(gc, nsc) > 0) {
      k_offsets_sums<<<(unsigned)std::max(gc, nsc), kScanThreads, 0, s>>>(hist, nt_all, p.nb, nchunk, csum, subcnt,
                                                                         p.nsub_d, part, p.mode, way);
      KB_LAUNCH_CHECK();
    }
    k_offsets_scan<<<(unsigned)std::max<int64_t>(p.nb, nsc), kScanThreads, 0, s>>>(csum, nchunk, p.nb, tot, subcnt,
                                                                                  p.nsub_d, part, sbb, p.mode, way);
    KB_LAUNCH_CHECK();
    k_bucket_starts<<<1, 1024, 0, s>>>(tot, p.nb, p.seg, bstart, segbase, p.mode, way);
    KB_LAUNCH_CHECK();
    k_offsets_down<<<(unsigned)(gc + p.nb), 256, 0, s>>>(hist, csum, bstart, nt_all, p.nb, nchunk, segbase, seg2b,
                                                         p.mode, way);
    KB_LAUNCH_CHECK();
  }
  // the integrate stage is exactly one kernel (pass 1), for either integrand
  KB_TRY(ev.rec(KB_STAGE_INTEGRATE));
  if (p.ntiles > 0 && p.nb > 0) {
    if (klow) {
      KB_TRY((launch_pass1<NEN, P, true>(p, m, klow, ws, status, s)));
    } else if constexpr (NEN <= 8) {
      if (p.op == KB_OP_MASS)
        KB_TRY((launch_pass1<NEN, P, false, Op::Mass>(p, m, nullptr, ws, status, s)));
      else
        KB_TRY((launch_pass1<NEN, P, false>(p, m, nullptr, ws, status, s)));
    } else {
      return KB_EINVAL;  // several DOFs per node: values are always given
    }
  }
  if (ntc > 0) {
    if (!set_lds(k_pass1_csr<V>, p.lds_csr)) return KB_EHIP;
    PairOut<V> o = pair_out<V>(p, ws);
    o.off1 = hist + p.ntiles * p.nb;
    k_pass1_csr<V><<<(unsigned)ntc, kCsrThreads, p.lds_csr, s>>>(cr->rows, cr->cols, (const V*)cr->vals,
                                                                 (const V*)cr->res, cr->nnz, p.csr_cap, p.nn, o, head);
    KB_LAUNCH_CHECK();
  }
  return assemble_tail<V>(p, ws, row_ptr, col_idx, (V*)vals, cap, nnz_dev, status, ev, s, cr, br);
}

template <int NEN, Prec P>
int integrate_impl(const Plan& p, const kb_mesh* m, void* vals, uint32_t* status, Events& ev, hipStream_t s) {
  using V = typename PrecTraits<P>::V;
  KB_TRY(ev.rec(KB_STAGE_INIT));
  k_init_status<<<1, 64, 0, s>>>(status, nullptr);
  KB_LAUNCH_CHECK();
  for (int i = KB_STAGE_COUNT; i <= KB_STAGE_INTEGRATE; ++i) KB_TRY(ev.rec(i));
  if (p.nel > 0) {
    const int blk = std::min(p.block, 256);  // the kernel is built for at most 256 lanes
    if (p.op == KB_OP_MASS)
      k_integrate_store<NEN, P, Op::Mass><<<grid_for(p.nel, blk), blk, 0, s>>>(m->conn, m->coords, m->coef, p.nel,
                                                                              p.nn, p.tau, (V*)vals, status);
    else
      k_integrate_store<NEN, P><<<grid_for(p.nel, blk), blk, 0, s>>>(m->conn, m->coords, m->coef, p.nel, p.nn, p.tau,
                                                                    (V*)vals, status);
    KB_LAUNCH_CHECK();
  }
  for (int i = KB_STAGE_HISTOGRAM; i <= KB_N_STAGES; ++i) KB_TRY(ev.rec(i));
  return KB_OK;
}

// the instantiations of one precision
#define KB_BUILD_INSTANCE(X, NEN, P)                                                                                 \
  X template int build_impl<NEN, P>(const Plan&, const kb_mesh*, const void*, unsigned char*, int32_t*, int32_t*, void*, \
                                    int64_t, int64_t*, uint32_t*, Events&, hipStream_t, const Carry*, const BatchRows*);
#define KB_INSTANCES(X, P)                                                                                         \
  KB_BUILD_INSTANCE(X, 4, P)                                                                                       \
  KB_BUILD_INSTANCE(X, 8, P)                                                                                       \
  KB_BUILD_INSTANCE(X, 12, P)                                                                                      \
  KB_BUILD_INSTANCE(X, 16, P)                                                                                      \
  KB_BUILD_INSTANCE(X, 24, P)                                                                                      \
  X template int integrate_impl<4, P>(const Plan&, const kb_mesh*, void*, uint32_t*, Events&, hipStream_t);          \
  X template int integrate_impl<8, P>(const Plan&, const kb_mesh*, void*, uint32_t*, Events&, hipStream_t);

}  // namespace kb
