// Host side of libmkv: argument validation, arena layout, call-order state machine, kernel
// launches, state export and kernel timing.  See include/mkv.h for the contract.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "mkv.h"
#include "mkv_internal.h"

using namespace mkv;

namespace {

thread_local std::string g_err;

mkv_status fail(mkv_status s, const char *fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return s;
}

}  // namespace

namespace mkv {
mkv_status report_error(mkv_status s, const char *msg) { return fail(s, "%s", msg); }
}  // namespace mkv

namespace {

mkv_status hip_fail(hipError_t e, const char *what) {
  return fail(MKV_EHIP, "%s: %s", what, hipGetErrorString(e));
}

enum Phase { PH_CREATED, PH_PROMPT, PH_READY, PH_APPENDED, PH_SELECTED, PH_ATTENDED };

constexpr int kProfKinds = 5;

struct Layout {
  std::vector<SeqDesc> seqs;  // offsets (relative to the arena) in the pointer fields
  // [off_tables, tables_end) holds everything that the host writes at creation, in one copy: the
  // descriptors, the state words (zero), the lists below and the codebook region
  size_t off_tables = 0, tables_end = 0, off_partials = 0, total = 0;
  size_t off_seqs = 0, off_state = 0, off_tiles = 0, off_prep = 0, off_comb = 0, off_rk_pairs = 0, off_lists = 0,
         off_cbtab = 0;
  int n_tiles = 0, n_tiles_uq = 0, n_tiles_rk = 0;
  std::vector<int4> tiles;     // attention tiles in launch order
  std::vector<int4> prep;      // decode-step append / scoring work list
  std::vector<int2> rk_pairs;  // RocketKV (seq, kv head) pairs
  std::vector<int4> comb;      // combine work list
  std::vector<int32_t> lists;    // the groups' sequences, one group after another
  std::vector<SeqGroup> groups;  // `list` not set (the place in `lists` follows from the counts)
};

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// Every region pointer of a descriptor (arena offsets in the layout, device addresses once the
// arena is known); the descriptor is its integer fields followed by exactly these.
constexpr uint64_t SeqDesc::*kRegionFields[] = {
    &SeqDesc::k,      &SeqDesc::v,      &SeqDesc::kc,      &SeqDesc::vc,      &SeqDesc::kmeta, &SeqDesc::vmeta,
    &SeqDesc::kres,   &SeqDesc::krow,   &SeqDesc::kout,    &SeqDesc::vout,    &SeqDesc::vdel,  &SeqDesc::pos,
    &SeqDesc::score,  &SeqDesc::logits, &SeqDesc::vbest,   &SeqDesc::stage_k, &SeqDesc::stage_v,
    &SeqDesc::kcm,    &SeqDesc::sel,    &SeqDesc::akeys,   &SeqDesc::aux0,    &SeqDesc::aux1,  &SeqDesc::colpart};
static_assert(offsetof(SeqDesc, k) + sizeof(kRegionFields) / sizeof(kRegionFields[0]) * sizeof(uint64_t) ==
                  sizeof(SeqDesc),
              "every region pointer of SeqDesc is relocated");

constexpr int kMaxTiles = 32;  // per (sequence, kv head); the combine kernel holds up to 64

// Bytes each token costs the attention pass.
double token_bytes(const SeqDesc &s, int D) {
  switch (s.method) {
    case UQ: return D + D / 64.0 * 8 + 8;
    case KVQ: return D * s.bits / 4.0 + 4 + 8 + 4;
    default: return 4.0 * D;
  }
}

// What a token of a quantized sequence costs a wave, in the same unit (KVQ at 4 bits: its bytes): tiles
// of a short launch all start together, so equal times balance it, not equal bytes (clock stamps per
// 32-token batch: uniform 4-bit 2.0 us, KVQ at 2, 3 and 4 bits 2.3, 3.0 and 3.5).
double token_cost(const SeqDesc &s, int D) {
  const double c = s.method == UQ ? 80 : s.bits == 2 ? 92 : s.bits == 3 ? 120 : 140;
  return c * D / 128;
}

// Tile size: large tiles amortise each workgroup's set-up, but a launch needs several
// workgroups per slot (256 CUs x 3 resident workgroups) to balance: about 4 rounds, within
// 64 to 192 KiB (measured best for batches of ~40 MB and ~600 MB per step); then adjusted to
// whole rounds (below).
constexpr int kTileSlots = kCus * 3;  // resident attention workgroups (3 per CU)
double tile_bytes_for(double total_bytes) {
  constexpr double kRounds = 4;
  return std::min(196608.0, std::max(65536.0, total_bytes / (kTileSlots * kRounds)));
}

mkv_status check_shape(const mkv_shape *sh) {
  if (!sh) return fail(MKV_EINVAL, "shape is NULL");
  if (sh->n_seqs < 1 || sh->n_kv_heads < 1 || sh->n_q_heads < 1 || sh->max_new_tokens < 0)
    return fail(MKV_EINVAL, "shape fields must be positive (max_new_tokens >= 0)");
  if (sh->n_q_heads % sh->n_kv_heads != 0) return fail(MKV_EINVAL, "n_q_heads %% n_kv_heads != 0");
  const int G = sh->n_q_heads / sh->n_kv_heads;
  if (G != 1 && G != 2 && G != 4 && G != 8)
    return fail(MKV_EUNSUPPORTED, "query heads per kv head must be 1, 2, 4 or 8 (got %d)", G);
  if (sh->head_dim != 64 && sh->head_dim != 128)
    return fail(MKV_EUNSUPPORTED, "head_dim must be 64 or 128 (got %d)", sh->head_dim);
  return MKV_OK;
}

// RocketKV's SnapKV budget: keep_tokens, or in ratio mode max(floor(n0 / keep_ratio), window).
int rocket_keep(const mkv_config &c, int n0) {
  return c.keep_ratio > 0 ? std::max(n0 / c.keep_ratio, c.window) : c.keep_tokens;
}

mkv_status check_config(const mkv_config &c, int n0, int D, int s) {
  if (n0 < 1) return fail(MKV_EINVAL, "seq %d: prompt_len must be >= 1", s);
  switch (c.method) {
    case MKV_FP16: return MKV_OK;
    case MKV_UQ:
      if (c.bits != 4) return fail(MKV_EUNSUPPORTED, "seq %d: uniform quantization supports bits=4", s);
      if (c.group != 64) return fail(MKV_EUNSUPPORTED, "seq %d: uniform quantization supports group=64", s);
      return MKV_OK;
    case MKV_KVQ:
      if (c.bits < 2 || c.bits > 4) return fail(MKV_EINVAL, "seq %d: KVQ bits must be 2, 3 or 4", s);
      if (c.outlier_bp < 0 || c.outlier_bp > 5000) return fail(MKV_EINVAL, "seq %d: outlier_bp in 0..5000", s);
      if (n0 > 65535) return fail(MKV_EUNSUPPORTED, "seq %d: KVQ prompt longer than 65535", s);
      return MKV_OK;
    case MKV_H2O: {
      if (c.budget_pct < 1 || c.budget_pct > 10000) return fail(MKV_EINVAL, "seq %d: budget_pct in 1..10000", s);
      const long long B = (long long)c.budget_pct * n0 / 100;
      if (B < 1) return fail(MKV_EINVAL, "seq %d: H2O budget is 0 tokens for prompt_len %d", s, n0);
      return MKV_OK;
    }
    case MKV_ROCKET:
      if (c.window < 1) return fail(MKV_EINVAL, "seq %d: window must be >= 1", s);
      if (c.keep_ratio < 0) return fail(MKV_EINVAL, "seq %d: keep_ratio must be >= 0", s);
      if (c.keep_ratio == 0 && c.keep_tokens < c.window) return fail(MKV_EINVAL, "seq %d: keep_tokens must be >= window", s);
      if (c.pool < 1 || (c.pool & 1) == 0) return fail(MKV_EINVAL, "seq %d: pool must be odd and >= 1", s);
      if (c.n_channels < 1 || c.n_channels > D) return fail(MKV_EINVAL, "seq %d: n_channels in 1..head_dim", s);
      if (c.topk < 0) return fail(MKV_EINVAL, "seq %d: topk must be >= 0", s);
      if (c.topk == 0 && rocket_keep(c, n0) / 2 < 1) return fail(MKV_EINVAL, "seq %d: the keep budget / 2 is 0", s);
      return MKV_OK;
    default:
      return fail(MKV_EINVAL, "seq %d: unknown method %d", s, c.method);
  }
}

// RocketKV scoring workgroups of a decode step per kv head.
int score_parts(const SeqDesc &d) { return (d.cap + kScoreTokensPerPart - 1) / kScoreTokensPerPart; }

// The work lists of a layout whose sizes are set.
void fill_lists(Layout *L, int Hkv) {
  const int S = (int)L->seqs.size();
  // Attention tiles in launch order (a tile's partial slot is tile_first + h tile_count + z / chunk,
  // whatever its place): the quantized tiles, the longest-running per byte, spread evenly over the
  // first 3/4 of the fp16-row and quantized tiles, the fp16-row tiles evenly over all of them, RocketKV
  // tiles last.  Long tiles then start early enough to end with the rest, while issue-bound and
  // bandwidth-bound tiles still share the chip throughout (measured on the mixed batch: 136-137
  // against 140-141 us per partial launch for the sequence order; spreading the quantized tiles
  // over 60 %, 90 % or all of the list, or putting them all first, did less or worse).
  {
    constexpr double kQuantSpan = 0.75;
    std::vector<int4> of[2];  // fp16-row and quantized tiles in sequence order
    std::vector<int> at[2];   // their places in the sequence order
    std::vector<int4> rocket;
    int place = 0;
    for (int s = 0; s < S; ++s) {
      const SeqDesc &d = L->seqs[s];
      const int amax = d.method == ROCKET ? d.topk : d.cap, q = d.method == KVQ || d.method == UQ;
      for (int h = 0; h < Hkv; ++h)
        for (int t = 0; t < d.tile_count; ++t) {
          const int4 tile = make_int4(s, h, t * d.chunk, std::min(amax, (t + 1) * d.chunk));
          if (d.method == ROCKET) {
            rocket.push_back(tile);
          } else {
            of[q].push_back(tile);
            at[q].push_back(place++);
          }
        }
    }
    // the two in the order of their places in the list, in units of its length, the earlier one in the
    // sequence order where they coincide
    const double nr = (double)of[0].size(), nq = (double)of[1].size();
    size_t ir = 0, iq = 0;
    L->tiles.reserve(L->n_tiles);
    while (ir < of[0].size() || iq < of[1].size()) {
      const double r = ir < of[0].size() ? (ir + 0.5) / nr : 2.0, q = iq < of[1].size() ? (iq + 0.5) / nq * kQuantSpan : 2.0;
      if (q < r || (q == r && at[1][iq] < at[0][ir])) L->tiles.push_back(of[1][iq++]);
      else L->tiles.push_back(of[0][ir++]);
    }
    L->tiles.insert(L->tiles.end(), rocket.begin(), rocket.end());
  }
  // a decode step's append and scoring work: RocketKV scoring parts (one per kScoreTokens tokens
  // of the largest retained set) first, then the plain appends
  for (int s = 0; s < S; ++s) {
    const SeqDesc &d = L->seqs[s];
    if (d.method != ROCKET) continue;
    const int parts = score_parts(d);
    for (int h = 0; h < Hkv; ++h) {
      L->rk_pairs.push_back(make_int2(s, h));
      for (int p = 0; p < parts; ++p) L->prep.push_back(make_int4(s, h, p, parts));
    }
  }
  for (int s = 0; s < S; ++s)
    if (L->seqs[s].method != ROCKET)
      for (int h = 0; h < Hkv; ++h) L->prep.push_back(make_int4(s, h, -1, 0));
  // the combine: H2O kv heads' parts (one per kCombineSlots slots) first, then one item per pair
  for (int pass = 0; pass < 2; ++pass)
    for (int s = 0; s < S; ++s) {
      const SeqDesc &d = L->seqs[s];
      if ((d.method == H2O) != (pass == 0)) continue;
      const int parts = d.method == H2O ? d.vparts : 1;
      for (int h = 0; h < Hkv; ++h)
        for (int p = 0; p < parts; ++p) L->comb.push_back(make_int4(s, h, p, parts));
    }
  // Prefill groups.  A launch has workgroups for every sequence up to the longest's length, and those
  // past a shorter one's end leave at once, 4-5 a nanosecond (1 where they hold the H2O scores' LDS); a
  // launch of its own costs a few microseconds.  A group ends where its idle tokens would pass twice its
  // own plus 2^20 / Hkv.  (One fp16 prompt of 131072 tokens with 127 of 300: 704 us with launches per
  // sequence, 1885 in one group, 227 in two; uniform 4-bit 3416, 1187, 313; one of 32768 with 31 of 300
  // under KVQuant at 3 bits 3258, 394, 370.)
  const double spare = double(1 << 20) / Hkv;
  for (int m = 0; m < kMethods; ++m) {
    const size_t first = L->lists.size();
    for (int s = 0; s < S; ++s)
      if (L->seqs[s].method == m) L->lists.push_back(s);
    std::stable_sort(L->lists.begin() + first, L->lists.end(),
                     [&](int32_t a, int32_t b) { return L->seqs[a].n0 > L->seqs[b].n0; });
    double own = 0.0, idle = 0.0;
    for (size_t i = first; i < L->lists.size(); ++i) {
      const SeqDesc &d = L->seqs[L->lists[i]];
      if (i > first) idle += L->groups.back().longest - d.n0;
      if (i == first || idle > 2 * own + spare || L->groups.back().n == kMaxGridY) {
        L->groups.push_back(SeqGroup{nullptr, m, 0, d.n0, 0, 0});
        own = idle = 0.0;
      }
      SeqGroup &sg = L->groups.back();
      ++sg.n;
      own += d.n0;
      if (m == ROCKET && d.T < d.n0) sg.max_vote_rows = std::max(sg.max_vote_rows, d.w_eff);
      sg.max_kept = std::max(sg.max_kept, m == H2O ? std::min(d.B, d.n0) : m == ROCKET ? std::min(d.T, d.n0) : d.n0);
    }
  }
}

// `lists`: fill the lists too (the sizes and offsets do not need them).
mkv_status make_layout(const mkv_shape *shp, const mkv_config *cfg, const int32_t *plen, Layout *L, bool lists) {
  mkv_status st = check_shape(shp);
  if (st != MKV_OK) return st;
  if (!cfg || !plen) return fail(MKV_EINVAL, "cfg and prompt_len must be non-NULL");
  const int S = shp->n_seqs, Hkv = shp->n_kv_heads, D = shp->head_dim, G = shp->n_q_heads / Hkv;
  const int mn = shp->max_new_tokens;
  for (int s = 0; s < S; ++s)
    if ((st = check_config(cfg[s], plen[s], D, s)) != MKV_OK) return st;

  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off = align256(off + std::max<size_t>(bytes, 1));
    return (uint64_t)o;
  };
  take(1);  // no region at offset 0: a zero offset marks one the method lacks
  L->seqs.assign(S, SeqDesc{});
  int q_h2o = 0, q_rk = 0, row0 = 0;
  for (int s = 0; s < S; ++s) {
    SeqDesc &d = L->seqs[s];
    const mkv_config &c = cfg[s];
    const int n0 = plen[s];
    d.method = c.method;
    d.n0 = n0;
    d.bits = c.bits;
    d.bp = c.outlier_bp;
    d.row0 = row0;
    row0 += n0;
    const size_t H = Hkv;
    switch (c.method) {
      case FP16:
        d.cap = n0 + mn;
        d.k = take(H * d.cap * D * 2);
        d.v = take(H * d.cap * D * 2);
        break;
      case UQ:
        d.cap = (n0 + mn + 3) & ~3;  // value codes are stored in 4-token blocks
        d.rowbytes = D / 2;
        d.nblk = d.cap / 64;
        d.kc = take(H * d.cap * d.rowbytes);
        d.vc = take(H * d.cap * d.rowbytes);
        d.kmeta = take(H * std::max(d.nblk, 1) * D * 8);
        d.vmeta = take(H * d.cap * (D / 64) * 8);
        d.kres = take(H * 64 * D * 2);
        break;
      case KVQ: {
        d.cap = (n0 + mn + 3) & ~3;  // value codes are stored in 4-token blocks
        d.rowbytes = D * c.bits / 8;
        d.n_o = (int)(((long long)n0 * c.outlier_bp + 5000) / 10000);
        d.n_ov = (int)(((long long)D * c.outlier_bp + 5000) / 10000);
        d.nov_slots = c.outlier_bp > 0 ? std::max(1, d.n_ov) : 1;
        d.pool_cap = c.outlier_bp > 0 ? (std::min(d.n_o, n0) + mn) * D : 1;
        d.kc = take(H * d.cap * d.rowbytes);
        d.vc = take(H * d.cap * d.rowbytes);
        d.kmeta = take(H * D * 8);
        d.vmeta = take(H * d.cap * 4);
        d.krow = take(H * (d.cap + 1) * 4);
        d.kout = take(H * d.pool_cap * 4);
        d.vout = take(H * d.cap * d.nov_slots * 4);
        d.vdel = take(H * d.cap * d.nov_slots * 4);
        break;
      }
      case H2O: {
        d.B = (int)((long long)c.budget_pct * n0 / 100);
        d.R = d.B / 2;
        d.cap = (int)std::min<long long>((long long)d.B + 1, (long long)n0 + mn);
        d.k = take(H * d.cap * D * 2);
        d.v = take(H * d.cap * D * 2);
        d.pos = take(H * d.cap * 4);
        d.score = take(H * d.cap * 4);
        d.logits = take(H * d.cap * G * 4);
        d.vparts = (d.cap + kCombineSlots - 1) / kCombineSlots;
        d.vbest = take(H * d.vparts * 16);
        d.stage_k = take(H * n0 * D * 2);
        d.stage_v = take(H * n0 * D * 2);
        d.aux0 = take(H * n0 * 4);
        d.aux1 = take(H * G * n0 * 8);
        {
          // row segments of the column sums: whole streamed tiles, at least 512 virtual rows each
          const long long rows = (long long)n0 * G;
          d.seg_rows = (int)std::max<long long>(512, ((rows + kScoreSegs - 1) / kScoreSegs + 255) / 256 * 256);
          d.nseg = (int)((rows + d.seg_rows - 1) / d.seg_rows);
          d.colpart = take(H * d.nseg * n0 * 4);
        }
        d.q_off = q_h2o;
        q_h2o += n0;
        break;
      }
      case ROCKET: {
        d.T = rocket_keep(c, n0);
        d.window = c.window;
        d.w_eff = std::min(c.window, n0);
        d.pool = c.pool;
        d.nch = c.n_channels;
        d.topk = c.topk > 0 ? c.topk : d.T / 2;
        const int kept = std::min(d.T, n0);
        d.cap = kept + mn;
        const int nchunk = (n0 + 255) / 256;
        d.k = take(H * d.cap * D * 2);
        d.v = take(H * d.cap * D * 2);
        d.cstride = (d.cap + 7) & ~7;
        d.kcm = take(H * d.cstride * D * 2);
        d.pos = take(H * d.cap * 4);
        d.sel = take(H * d.topk * 4);
        d.akeys = take(H * d.cap * 4);
        d.stage_k = take(H * n0 * D * 2);
        d.stage_v = take(H * n0 * D * 2);
        d.aux0 = take(H * n0 * 4);
        d.aux1 = take(std::max({H * d.w_eff * G * nchunk * 8, H * D * 4, H * n0 * 4}));
        d.q_off = q_rk;
        q_rk += c.window;
        break;
      }
    }
  }
  // attention tiles: per sequence and kv head, ranges of `chunk` tokens over its largest active set;
  // one launch covers them all, RocketKV sequences last (their gathered tiles are the shortest)
  double total = 0.0;
  for (int s = 0; s < S; ++s) {
    const SeqDesc &d = L->seqs[s];
    total += (double)Hkv * (d.method == ROCKET ? d.topk : d.cap) * token_bytes(d, D);
  }
  int n_quant = 0;
  for (const SeqDesc &d : L->seqs) n_quant += d.method == UQ || d.method == KVQ;
  // a sequence's tokens per tile (a multiple of `gran`) and tile count for tiles of `unit` tokens
  auto split = [&](const SeqDesc &d, double unit, int gran, int *chunk) {
    const int amax = d.method == ROCKET ? d.topk : d.cap;
    int c = std::max(gran, std::min((int)unit & -gran, 4096)), n = std::max(1, (amax + c - 1) / c);
    if (n > kMaxTiles) {  // long sequences: fewer, larger tiles keep the combine short
      c = (((amax + kMaxTiles - 1) / kMaxTiles) + 63) & ~63;
      n = (amax + c - 1) / c;
    }
    *chunk = c;
    return n;
  };
  // Tiles are multiples of 64 tokens (of 32, which filled the slots of small launches more finely,
  // measured slower), quantized ones of 128 in short launches: the 4 waves of a workgroup take 32-token
  // batches, so other sizes leave waves idle for the last one (a 320-token tile takes as long as a
  // 384-token one).  In launches of three or more rounds of workgroups, fp16-row tiles (FP16, H2O)
  // take twice the bytes: they are bandwidth-bound, and each tile a CU starts costs a dispatch gap (a
  // median 2 us from one tile's end to the next one's start on that CU, measured with clock stamps), so
  // fewer, longer row tiles leave the slots busier (mixed batch: 134.0-135.1 against 135.8-136.3
  // us per partial launch; 1.5x and 2.5-3x no better, 0.75x 6 us slower).
  // (Uniform 4-bit tiles of d = 64 are multiples of 256 in short launches: in tiles of 128, whose waves take
  // one batch each, every wave's largest probability is exactly 1 and its product with the value step then
  // rounds like the step, which is 3-5 % worse for unit-normal values: 512 tokens 5.29e-4 from 64 bits
  // against 5.05e-4, mean of 1600 inputs; a step of it takes 8.7 us in tiles of 128 and 9.2 in these.)
  bool long_launch = false, fine = true;
  auto short_gran = [&](const SeqDesc &d) { return d.method == UQ && D == 64 ? 256 : 128; };
  auto by_bytes = [&](const SeqDesc &d, double tb, int *chunk) {
    if (long_launch && (d.method == FP16 || d.method == H2O)) tb *= 2;
    return split(d, tb / token_bytes(d, D), fine || (d.method != UQ && d.method != KVQ) ? 64 : short_gran(d), chunk);
  };
  auto by_time = [&](const SeqDesc &d, double cost, int *chunk) {
    return split(d, cost / token_cost(d, D), short_gran(d), chunk);
  };
  auto count_at = [&](double size, auto rule) {
    long long n = 0;
    int c;
    for (int s = 0; s < S; ++s) n += (long long)Hkv * rule(L->seqs[s], size, &c);
    return n;
  };
  // the smallest size lo f^i below `hi` with at most `most` tiles, by bisection (the count falls with
  // the size); `hi` if there is none
  auto smallest = [&](double lo, double hi, double f, long long most, auto rule) {
    int a = 0, b = std::max(0, (int)std::ceil(std::log(hi / lo) / std::log(f)));
    while (a < b) {
      const int m = (a + b) / 2;
      if (count_at(lo * std::pow(f, m), rule) <= most) b = m;
      else a = m + 1;
    }
    return std::min(hi, lo * std::pow(f, a));
  };
  // whole rounds of resident workgroups: when the size rule leaves the last round partly idle,
  // smaller tiles (down to 16 KiB) fill it, the smallest size whose count still fits in the
  // rounds begun.
  auto fill_rounds = [&]() {
    const double most = tile_bytes_for(total);
    const long long cap = (count_at(most, by_bytes) + kTileSlots - 1) / kTileSlots * kTileSlots;
    return smallest(16384.0, most, 1.02, cap, by_bytes);
  };
  double tile_bytes = tile_bytes_for(total);
  long_launch = fine = count_at(tile_bytes, by_bytes) >= 3 * kTileSlots;
  enum { BY_BYTES, BY_TIME, BY_ROWS } rule = BY_BYTES;
  if (!long_launch && n_quant == 0) {
    // Short launches of fp16 rows alone: every workgroup starts at once, tile i on CU i mod 256, so the
    // fullest CU sets the time: its bytes, a set-up worth about 44 d = 128 rows per tile, and a rate that
    // drops with fewer than 3 workgroups on a CU.  The size with the least is taken.  (Sweeps of four
    // layers: 8 x 8192 tokens under H2O-20 117, 113, 116, 118, 116 us at 832, 448, 576, 384, 256 tiles;
    // H2O-40 162, 159, 159, 156, 167 at 1664, 1152, 704, 512, 448; 8 x 4096 FP16 145, 154, 144, 146 at
    // 1408, 1088, 704, 512.  The weights were fitted to these three; the model finds the best of each, but
    // does not order the others.)
    rule = BY_ROWS;
    double best = -1.0;
    float load[kCus];
    for (int c = 64; c <= 1024; c += 64) {
      const double bytes = c * 4.0 * D;
      const long long n = count_at(bytes, by_bytes);
      if (n > 3 * kTileSlots && c < 1024) continue;
      std::fill(load, load + kCus, 0.f);
      unsigned i = 0;
      for (int rocket = 0; rocket < 2; ++rocket)
        for (const SeqDesc &d : L->seqs) {
          if ((d.method == ROCKET) != (rocket == 1)) continue;
          int chunk;
          const int amax = d.method == ROCKET ? d.topk : d.cap, tiles = by_bytes(d, bytes, &chunk);
          const float full = 44 * 512.f + chunk * 4.f * D, last = 44 * 512.f + (amax - (tiles - 1) * chunk) * 4.f * D;
          for (int h = 0; h < Hkv; ++h) {
            for (int t = 0; t + 1 < tiles; ++t) load[i++ % kCus] += full;
            load[i++ % kCus] += last;
          }
        }
      // (a d = 64 workgroup has half the bytes in flight)
      const long long busy = (n + kCus - 1) / kCus * D / 64;
      const double cost = *std::max_element(load, load + kCus) *
                          (busy <= 2 ? 1.3 : busy == 3 ? 1.1 : busy == 4 ? 1.04 : 1.0);
      if (best < 0.0 || cost < best) {
        best = cost;
        tile_bytes = bytes;
      }
    }
  } else {
    // One round: quantized tiles alone, bound by the latency of their batches, are best all resident at once
    // (8 x 8192 tokens, three layers: uniform 4-bit 93 us at 704 tiles of 768 tokens against 105 at
    // 1408 of 384, KVQ at 4 bits 144 against 156; 16 ragged sequences of three kinds, two layers, 101
    // against 116): the smallest size that allows it, by time, up to 8 times the default.  The kernel for
    // groups of 8 heads of 128 takes 184 registers, which leaves room for 2 workgroups on a CU: KVQuant at 2
    // bits, 48 x 640-800 tokens, 2 kv heads, two layers, 48.0 us with 314 tiles, 58.0 with 602 (and 50.1
    // with 410 of the general rule).  Where no size has so few, as with more pairs than that, 3 on a CU.
    const int resident = D == 128 && G == 8 ? 2 * kCus : kTileSlots;
    for (const int slots : {resident, kTileSlots}) {
      if (long_launch || n_quant < S || rule == BY_TIME) break;
      const double c = smallest(4096.0, 8 * tile_bytes, 1.03, slots, by_time);
      if (count_at(c, by_time) <= slots) {
        tile_bytes = c;
        rule = BY_TIME;
      }
    }
    if (rule == BY_BYTES) tile_bytes = fill_rounds();
  }
  // (a layout that mkv_decode_attention_noalloc has room for under the general rule keeps it)
  if (rule != BY_BYTES || !fine) {
    const long long n = rule == BY_TIME ? count_at(tile_bytes, by_time) : count_at(tile_bytes, by_bytes);
    if (n * G * (D + 2) * sizeof(float) > kStaticScratchBytes) {
      rule = BY_BYTES;
      fine = true;
      tile_bytes = fill_rounds();
    }
  }
  int n_prep = 0, n_pairs = 0, n_comb = 0;
  for (int pass = 0; pass < 2; ++pass)
    for (SeqDesc &d : L->seqs) {
      if ((d.method == ROCKET) != (pass == 1)) continue;
      d.tile_count = rule == BY_TIME ? by_time(d, tile_bytes, &d.chunk) : by_bytes(d, tile_bytes, &d.chunk);
      d.tile_first = L->n_tiles;
      L->n_tiles += Hkv * d.tile_count;
      if (d.method == UQ) L->n_tiles_uq += Hkv * d.tile_count;
      if (pass == 1) L->n_tiles_rk += Hkv * d.tile_count;
      n_prep += Hkv * (pass == 1 ? score_parts(d) : 1);
      n_pairs += pass == 1 ? Hkv : 0;
      n_comb += Hkv * (d.method == H2O ? d.vparts : 1);
    }
  L->off_tables = off;
  L->off_seqs = take(sizeof(SeqDesc) * S);
  L->off_state = take(sizeof(int32_t) * S * Hkv * ST_WORDS);
  L->off_tiles = take(sizeof(int4) * L->n_tiles);
  L->off_prep = take(sizeof(int4) * n_prep);
  L->off_comb = take(sizeof(int4) * n_comb);
  L->off_rk_pairs = take(sizeof(int2) * n_pairs);
  L->off_lists = take(sizeof(int32_t) * S);
  L->off_cbtab = take(sizeof(float) * kCbRegionFloats);
  L->tables_end = off;
  L->off_partials = take(sizeof(float) * (size_t)L->n_tiles * G * (D + 2));
  L->total = off;
  if (lists) fill_lists(L, Hkv);
  return MKV_OK;
}

}  // namespace

struct mkv_cache {
  Shape sh{};
  std::vector<mkv_config> cfg;
  std::vector<SeqDesc> hs;  // absolute device pointers
  std::vector<SeqGroup> groups;
  char *arena = nullptr;
  Dev dv{};
  Phase phase = PH_CREATED;
  int steps = 0;
  bool any_h2o = false, any_rocket = false, h2o_done = false, snap_done = false;
  int topk_max = 0;
  int h2o_rows = 0, rocket_rows = 0;
  // profiling
  bool evict_pending = false;  // H2O: the last eviction call's victims await the next decode append
  int prof_mask = 0;  // bit k: launches of kind k are timed
  int prof_cap = 0;
  std::vector<hipEvent_t> ev[kProfKinds][2];
  int prof_n[kProfKinds] = {};
};

namespace {

// The timing events of the next launch of `kind` (none when that kind is not timed or its events
// are used up); the launch itself records its kernel's start and end in them.
LaunchEv prof_ev(mkv_cache *c, int kind) {
  if (!(c->prof_mask >> kind & 1)) return {};
  const int i = c->prof_n[kind];
  if (i >= c->prof_cap) return {};
  c->prof_n[kind] = i + 1;
  return LaunchEv{c->ev[kind][0][i], c->ev[kind][1][i]};
}

mkv_status check_hip(hipError_t e, const char *what) {
  return e == hipSuccess ? MKV_OK : hip_fail(e, what);
}

}  // namespace

namespace mkv {
mkv_status layout_tiles(const mkv_shape *shape, const mkv_config *cfg, const int32_t *prompt_len,
                        std::vector<int4> *tiles, std::vector<SeqDesc> *seqs) {
  Layout L;
  const mkv_status st = make_layout(shape, cfg, prompt_len, &L, true);
  if (st != MKV_OK) return st;
  *tiles = L.tiles;
  *seqs = L.seqs;
  return MKV_OK;
}
mkv_status layout_groups(const mkv_shape *shape, const mkv_config *cfg, const int32_t *prompt_len,
                         std::vector<SeqGroup> *groups, std::vector<int32_t> *lists) {
  Layout L;
  const mkv_status st = make_layout(shape, cfg, prompt_len, &L, true);
  if (st != MKV_OK) return st;
  *groups = L.groups;
  *lists = L.lists;
  return MKV_OK;
}
}  // namespace mkv

extern "C" {

const char *mkv_status_str(mkv_status s) {
  switch (s) {
    case MKV_OK: return "ok";
    case MKV_EINVAL: return "invalid argument";
    case MKV_ENOMEM: return "arena too small";
    case MKV_ECAPACITY: return "cache capacity exceeded";
    case MKV_ESTATE: return "call out of order";
    case MKV_EUNSUPPORTED: return "unsupported configuration";
    case MKV_EHIP: return "HIP runtime error";
  }
  return "unknown status";
}

const char *mkv_last_error(void) { return g_err.c_str(); }

mkv_status mkv_cache_bytes(const mkv_shape *shape, const mkv_config *cfg, const int32_t *prompt_len,
                           size_t *arena_bytes) {
  if (!arena_bytes) return fail(MKV_EINVAL, "arena_bytes is NULL");
  Layout L;
  mkv_status st = make_layout(shape, cfg, prompt_len, &L, false);
  if (st != MKV_OK) return st;
  *arena_bytes = L.total;
  return MKV_OK;
}

mkv_status mkv_cache_create(const mkv_shape *shape, const mkv_config *cfg, const int32_t *prompt_len,
                            const float *codebooks, void *arena, size_t arena_bytes, void *stream,
                            mkv_cache **out) {
  if (!out) return fail(MKV_EINVAL, "out is NULL");
  *out = nullptr;
  Layout L;
  mkv_status st = make_layout(shape, cfg, prompt_len, &L, true);
  if (st != MKV_OK) return st;
  if (!arena) return fail(MKV_EINVAL, "arena is NULL");
  if (((uintptr_t)arena & 255) != 0) return fail(MKV_EINVAL, "arena must be 256-byte aligned");
  if (arena_bytes < L.total)
    return fail(MKV_ENOMEM, "arena has %zu bytes, the cache needs %zu", arena_bytes, L.total);
  bool any_kvq = false;
  for (int s = 0; s < shape->n_seqs; ++s) any_kvq |= cfg[s].method == MKV_KVQ;
  float table[kCbRegionFloats] = {};
  if (any_kvq) {
    if (!codebooks) return fail(MKV_EINVAL, "codebooks are required for KVQ sequences");
    const float *src = codebooks;
    for (int b = 2; b <= 4; ++b) {
      const int nc = 1 << b;
      float *dst = table + cb_offset(b);
      for (int half = 0; half < 2; ++half) {
        for (int i = 0; i < nc; ++i) {
          const float x = src[half * nc + i];
          if (!std::isfinite(x)) return fail(MKV_EINVAL, "codebook entry is not finite");
          if (round_to_half(x) != x) return fail(MKV_EINVAL, "codebook entry %g is not an fp16 value", (double)x);
          if (i > 0 && !(x >= src[half * nc + i - 1])) return fail(MKV_EINVAL, "codebooks must be ascending");
          dst[half * nc + i] = x;
        }
        for (int i = 0; i + 1 < nc; ++i) {
          volatile float sum = src[half * nc + i] + src[half * nc + i + 1];
          dst[2 * nc + half * (nc - 1) + i] = sum * 0.5f;
        }
      }
      src += 2 * nc;
    }
    // the attention's lookup tables: packed fp16 codebook values per quad (b = 2) or pair of codes
    uint32_t *lut = reinterpret_cast<uint32_t *>(table + kLutBase);
    auto hb = [](float x) { return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)x); };
    for (int b = 2; b <= 4; ++b) {
      const int nc = 1 << b, half = lut_half_words(b);
      for (int which = 0; which < 2; ++which) {
        const float *cb = table + cb_offset(b) + which * nc;
        uint32_t *dst = lut + lut_offset(b) + which * half;
        if (b == 2) {
          for (int q = 0; q < 256; ++q) {
            dst[2 * q] = hb(cb[q & 3]) | hb(cb[(q >> 2) & 3]) << 16;
            dst[2 * q + 1] = hb(cb[(q >> 4) & 3]) | hb(cb[(q >> 6) & 3]) << 16;
          }
        } else {
          for (int f = 0; f < half; ++f) dst[f] = hb(cb[f & (nc - 1)]) | hb(cb[f >> b]) << 16;
        }
      }
    }
  }
  mkv_cache *c = new mkv_cache();
  c->sh = Shape{shape->n_seqs, shape->n_q_heads, shape->n_kv_heads, shape->head_dim,
                shape->n_q_heads / shape->n_kv_heads, shape->max_new_tokens};
  c->cfg.assign(cfg, cfg + shape->n_seqs);
  c->arena = static_cast<char *>(arena);
  const uint64_t base = (uint64_t)(uintptr_t)arena;
  c->hs = std::move(L.seqs);
  for (auto &d : c->hs) {
    for (uint64_t SeqDesc::*f : kRegionFields)
      if (d.*f) d.*f += base;
    if (d.method == H2O) {
      c->any_h2o = true;
      c->h2o_rows += d.n0;
    }
    if (d.method == ROCKET) {
      c->any_rocket = true;
      c->rocket_rows += d.window;
      c->topk_max = std::max(c->topk_max, d.topk);
    }
  }
  c->dv.seqs = reinterpret_cast<const SeqDesc *>(c->arena + L.off_seqs);
  c->dv.state = reinterpret_cast<int32_t *>(c->arena + L.off_state);
  c->dv.tiles = reinterpret_cast<const int4 *>(c->arena + L.off_tiles);
  c->dv.partials = reinterpret_cast<float *>(c->arena + L.off_partials);
  c->dv.cbtab = reinterpret_cast<const float *>(c->arena + L.off_cbtab);
  c->dv.n_tiles = L.n_tiles;
  c->dv.prep = reinterpret_cast<const int4 *>(c->arena + L.off_prep);
  c->dv.rk_pairs = reinterpret_cast<const int2 *>(c->arena + L.off_rk_pairs);
  c->dv.n_prep = (int)L.prep.size();
  c->dv.comb = reinterpret_cast<const int4 *>(c->arena + L.off_comb);
  c->dv.n_comb = (int)L.comb.size();
  c->dv.n_rk_pairs = (int)L.rk_pairs.size();
  c->dv.n_tiles_uq = L.n_tiles_uq;
  c->dv.n_tiles_rk = L.n_tiles_rk;
  const int32_t *list = reinterpret_cast<const int32_t *>(c->arena + L.off_lists);
  c->groups = std::move(L.groups);
  for (SeqGroup &sg : c->groups) {
    sg.list = list;
    list += sg.n;
  }
  hipStream_t hst = static_cast<hipStream_t>(stream);
  // the tables in one copy (each copy from pageable memory costs the host several microseconds)
  std::vector<char> tables(L.tables_end - L.off_tables);  // zero: the state words start so
  auto put = [&](size_t at, const void *src, size_t bytes) {
    if (bytes > 0) std::memcpy(tables.data() + (at - L.off_tables), src, bytes);
  };
  put(L.off_seqs, c->hs.data(), sizeof(SeqDesc) * c->hs.size());
  put(L.off_tiles, L.tiles.data(), sizeof(int4) * L.tiles.size());
  put(L.off_prep, L.prep.data(), sizeof(int4) * L.prep.size());
  put(L.off_comb, L.comb.data(), sizeof(int4) * L.comb.size());
  put(L.off_rk_pairs, L.rk_pairs.data(), sizeof(int2) * L.rk_pairs.size());
  put(L.off_lists, L.lists.data(), sizeof(int32_t) * L.lists.size());
  put(L.off_cbtab, table, sizeof table);
  hipError_t e = hipMemcpyAsync(c->arena + L.off_tables, tables.data(), tables.size(), hipMemcpyHostToDevice, hst);
  if (e == hipSuccess) e = hipStreamSynchronize(hst);
  if (e != hipSuccess) {
    mkv_cache_destroy(c);
    return hip_fail(e, "mkv_cache_create");
  }
  *out = c;
  return MKV_OK;
}

mkv_status mkv_cache_destroy(mkv_cache *c) {
  if (!c) return MKV_OK;
  for (int k = 0; k < kProfKinds; ++k)
    for (int w = 0; w < 2; ++w)
      for (hipEvent_t e : c->ev[k][w]) (void)hipEventDestroy(e);
  delete c;
  return MKV_OK;
}

namespace {

// The decode append of one row per sequence (the row counts are already known to be 1).
mkv_status decode_append(mkv_cache *c, const uint16_t *k, const uint16_t *v, hipStream_t hst) {
  if (!(c->phase == PH_READY || (c->phase == PH_ATTENDED && !c->any_h2o)))
    return fail(MKV_ESTATE, "decode append must follow prefill or a completed decode step");
  if (c->steps >= c->sh.max_new)
    return fail(MKV_ECAPACITY, "cache holds %d decode steps (max_new_tokens)", c->sh.max_new);
  hipError_t e = launch_append_decode(c->dv, c->sh, k, v, hst, prof_ev(c, 2));
  if (e != hipSuccess) return hip_fail(e, "decode append");
  c->evict_pending = false;
  c->steps++;
  c->phase = PH_APPENDED;
  return MKV_OK;
}

// One partial launch over the tiles of every sequence, then the combine.
mkv_status attend(mkv_cache *c, const Dev &dv, const uint16_t *q, float *out, hipStream_t hst) {
  hipError_t e = launch_attention_partial(dv, c->sh, q, hst, prof_ev(c, 0));
  if (e != hipSuccess) return hip_fail(e, "attention partial");
  e = launch_attention_combine(dv, c->sh, out, hst, prof_ev(c, 1));
  if (e != hipSuccess) return hip_fail(e, "attention combine");
  c->phase = PH_ATTENDED;
  return MKV_OK;
}

// A decode step's append and top-k selection: the appends with the RocketKV scores, then the
// selection (the caller has made every check of decode_append and mkv_topk_select).
mkv_status decode_append_select(mkv_cache *c, const uint16_t *k, const uint16_t *v, const uint16_t *q,
                                hipStream_t hst) {
  hipError_t e = launch_append_select(c->dv, c->sh, k, v, q, hst, prof_ev(c, 4), prof_ev(c, 3));
  if (e != hipSuccess) return hip_fail(e, "decode append and top-k select");
  c->evict_pending = false;
  c->steps++;
  c->phase = PH_SELECTED;
  return MKV_OK;
}

}  // namespace

mkv_status mkv_append_quantize(mkv_cache *c, const uint16_t *k, const uint16_t *v, const int32_t *cu_new,
                               void *stream) {
  if (!c) return fail(MKV_EINVAL, "cache is NULL");
  if (!k || !v || !cu_new) return fail(MKV_EINVAL, "k, v and cu_new must be non-NULL");
  const int S = c->sh.S;
  hipStream_t hst = static_cast<hipStream_t>(stream);
  if (cu_new[0] != 0) return fail(MKV_EINVAL, "cu_new[0] must be 0");
  if (c->phase == PH_CREATED) {
    for (int s = 0; s < S; ++s)
      if (cu_new[s + 1] - cu_new[s] != c->hs[s].n0)
        return fail(MKV_EINVAL, "prefill: seq %d appends %d rows, prompt_len is %d", s, cu_new[s + 1] - cu_new[s],
                    c->hs[s].n0);
    for (const SeqGroup &sg : c->groups) {
      hipError_t e = launch_prefill(c->dv, c->sh, sg, k, v, hst);
      if (e != hipSuccess) return hip_fail(e, "prefill append");
    }
    c->phase = (c->any_h2o || c->any_rocket) ? PH_PROMPT : PH_READY;
    return MKV_OK;
  }
  for (int s = 0; s < S; ++s)
    if (cu_new[s + 1] - cu_new[s] != 1) return fail(MKV_EINVAL, "decode: seq %d must append exactly 1 row", s);
  return decode_append(c, k, v, hst);
}

mkv_status mkv_h2o_update_evict(mkv_cache *c, const uint16_t *q_prompt, void *stream) {
  if (!c) return fail(MKV_EINVAL, "cache is NULL");
  hipStream_t hst = static_cast<hipStream_t>(stream);
  if (q_prompt != nullptr) {
    if (c->phase != PH_PROMPT || c->h2o_done)
      return fail(MKV_ESTATE, "H2O prefill scoring runs once, after the prefill append");
    for (const SeqGroup &sg : c->groups) {
      if (sg.method != H2O) continue;
      hipError_t e = launch_h2o_prefill(c->dv, c->sh, sg, q_prompt, hst);
      if (e != hipSuccess) return hip_fail(e, "H2O prefill");
    }
    c->h2o_done = true;
    if (!c->any_rocket || c->snap_done) c->phase = PH_READY;
    return MKV_OK;
  }
  if (c->phase == PH_PROMPT && c->any_h2o) return fail(MKV_EINVAL, "H2O prefill needs q_prompt");
  if (c->phase != PH_ATTENDED) return fail(MKV_ESTATE, "eviction must follow mkv_decode_attention");
  // the victim chosen by the attention pass leaves the retained set now (exports see it gone);
  // its slot is overwritten by the next decode append, which needs no extra launch for this
  c->evict_pending = c->any_h2o;
  c->phase = PH_READY;
  return MKV_OK;
}

mkv_status mkv_snap_prefill_evict(mkv_cache *c, const uint16_t *q_window, void *stream) {
  if (!c) return fail(MKV_EINVAL, "cache is NULL");
  if (!c->any_rocket) return MKV_OK;
  if (c->phase != PH_PROMPT || c->snap_done)
    return fail(MKV_ESTATE, "SnapKV prefill eviction runs once, after the prefill append");
  if (!q_window) return fail(MKV_EINVAL, "q_window is NULL");
  hipStream_t hst = static_cast<hipStream_t>(stream);
  for (const SeqGroup &sg : c->groups) {
    if (sg.method != ROCKET) continue;
    hipError_t e = launch_snap_prefill(c->dv, c->sh, sg, q_window, hst);
    if (e != hipSuccess) return hip_fail(e, "SnapKV prefill");
  }
  c->snap_done = true;
  if (!c->any_h2o || c->h2o_done) c->phase = PH_READY;
  return MKV_OK;
}

mkv_status mkv_topk_select(mkv_cache *c, const uint16_t *q, int32_t *pos_out, void *stream) {
  if (!c) return fail(MKV_EINVAL, "cache is NULL");
  if (c->phase != PH_APPENDED) return fail(MKV_ESTATE, "top-k selection must follow a decode append");
  if (c->any_rocket) {
    if (!q) return fail(MKV_EINVAL, "q is NULL");
    hipStream_t hst = static_cast<hipStream_t>(stream);
    const hipError_t e = launch_topk(c->dv, c->sh, q, pos_out, c->topk_max, hst, prof_ev(c, 3));
    if (e != hipSuccess) return hip_fail(e, "top-k select");
  }
  c->phase = PH_SELECTED;
  return MKV_OK;
}

mkv_status mkv_decode_attention(mkv_cache *c, const uint16_t *q, float *out, void *stream) {
  if (!c) return fail(MKV_EINVAL, "cache is NULL");
  if (!q || !out) return fail(MKV_EINVAL, "q and out must be non-NULL");
  if (!(c->phase == PH_SELECTED || (c->phase == PH_APPENDED && !c->any_rocket)))
    return fail(MKV_ESTATE, "attention must follow the decode append (and top-k selection)");
  return attend(c, c->dv, q, out, static_cast<hipStream_t>(stream));
}

mkv_status mkv_decode_attention_noalloc(mkv_cache *c, const uint16_t *q, float *out, void *stream) {
  if (!c) return fail(MKV_EINVAL, "cache is NULL");
  if (!q || !out) return fail(MKV_EINVAL, "q and out must be non-NULL");
  if (!(c->phase == PH_SELECTED || (c->phase == PH_APPENDED && !c->any_rocket)))
    return fail(MKV_ESTATE, "attention must follow the decode append (and top-k selection)");
  const size_t need = sizeof(float) * (size_t)c->dv.n_tiles * c->sh.G * (c->sh.D + 2);
  if (need > kStaticScratchBytes)
    return fail(MKV_ENOMEM, "split-K workspace of %zu bytes exceeds the %zu-byte static workspace", need,
                kStaticScratchBytes);
  float *ws = nullptr;
  size_t ws_bytes = 0;
  hipError_t e = static_scratch(&ws, &ws_bytes);
  if (e != hipSuccess) return hip_fail(e, "static workspace address");
  Dev dv = c->dv;
  dv.partials = ws;
  return attend(c, dv, q, out, static_cast<hipStream_t>(stream));
}

mkv_status mkv_decode_step(mkv_cache *c, const uint16_t *k, const uint16_t *v, const uint16_t *q, float *out,
                           void *stream) {
  if (!c) return fail(MKV_EINVAL, "cache is NULL");
  if (!k || !v || !q || !out) return fail(MKV_EINVAL, "k, v, q and out must be non-NULL");
  // every check of the four calls below, made before the first of them enqueues anything, so that
  // a rejected step leaves the handle as it was; past this point only a HIP launch can fail
  if (c->phase == PH_CREATED) return fail(MKV_ESTATE, "decode step before the prefill append");
  if (!(c->phase == PH_READY || (c->phase == PH_ATTENDED && !c->any_h2o)))
    return fail(MKV_ESTATE, "decode step must follow prefill or a completed decode step");
  if (c->steps >= c->sh.max_new)
    return fail(MKV_ECAPACITY, "cache holds %d decode steps (max_new_tokens)", c->sh.max_new);
  hipStream_t hst = static_cast<hipStream_t>(stream);
  mkv_status st = MKV_OK;
  if (c->any_rocket) {
    // the append, the scores and the top-k, in one launch or two
    st = decode_append_select(c, k, v, q, hst);
  } else if (c->prof_mask >> 2 & 1) {
    st = decode_append(c, k, v, hst);  // appends are timed: in a launch of their own
  } else {
    // the attention launch appends: 1.5-2 us less of a step of 11-17 us for one sequence of 300 tokens,
    // 2.4-5.2 of 19-28 for 40 of them, under every method, by steps that do append (RocketKV scores the
    // appended key before its selection, so its append stays where the scores are)
    Dev dv = c->dv;
    dv.k_new = k;
    dv.v_new = v;
    if ((st = attend(c, dv, q, out, hst)) != MKV_OK) return st;
    c->evict_pending = false;
    c->steps++;
    return mkv_h2o_update_evict(c, nullptr, stream);
  }
  if (st != MKV_OK) return st;
  if ((st = mkv_decode_attention(c, q, out, stream)) != MKV_OK) return st;
  return mkv_h2o_update_evict(c, nullptr, stream);
}

mkv_status mkv_kv_memory(const mkv_shape *shape, const mkv_config *cfg, int32_t prompt_len, int32_t n_generated,
                         size_t *resident, size_t *peak) {
  mkv_status st = check_shape(shape);
  if (st != MKV_OK) return st;
  if (!cfg || !resident || !peak) return fail(MKV_EINVAL, "cfg, resident and peak must be non-NULL");
  if (n_generated < 0) return fail(MKV_EINVAL, "n_generated must be >= 0");
  const int D = shape->head_dim, G = shape->n_q_heads / shape->n_kv_heads;
  if ((st = check_config(*cfg, prompt_len, D, 0)) != MKV_OK) return st;
  const long long n0 = prompt_len, gen = n_generated, n = n0 + gen, row = 4LL * D;  // K and V fp16 rows
  long long now = 0, top = 0;
  switch (cfg->method) {
    case MKV_FP16:
      now = top = n * row;
      break;
    case MKV_UQ: {
      const long long nb = n / 64;  // complete key blocks are codes, the rest fp16
      const long long k = nb * 64 * (D / 2) + nb * D * 8 + (n - nb * 64) * 2 * D;
      const long long v = n * (D / 2) + n * (D / 64) * 8;
      now = top = k + v;
      break;
    }
    case MKV_KVQ: {
      const long long bp = cfg->outlier_bp, codes = 2 * n * D * cfg->bits / 8;
      const long long n_o = (n0 * bp + 5000) / 10000, n_ov = ((long long)D * bp + 5000) / 10000;
      const long long slots = bp > 0 ? std::max(1LL, n_ov) : 1;
      // key outliers: at most n_o per channel over the prompt; decode tokens at their expected rate
      const long long kout = std::min(n_o, n0) * D + (gen * D * bp + 5000) / 10000;
      now = top = codes + D * 8 + n * 4 + (n + 1) * 4 + kout * 4 + n * slots * 8;
      break;
    }
    case MKV_H2O: {
      const long long B = (long long)cfg->budget_pct * n0 / 100, kept = std::min(B, n0);
      const long long slot = row + 8 + 4LL * G;  // rows, position, score, last logits
      now = std::min(B, kept + gen) * slot;
      // prefill: the whole prompt in fp16 with its scores, beside the kept slots; decode: B + 1
      const long long pre = n0 * row + n0 * 4 + kept * slot;
      top = std::max(pre, (gen > 0 ? std::min(B + 1, kept + gen) : kept) * slot);
      break;
    }
    case MKV_ROCKET: {
      const long long T = rocket_keep(*cfg, prompt_len), kept = std::min(T, n0);
      const long long topk = cfg->topk > 0 ? cfg->topk : T / 2;
      const long long slot = row + 2LL * D + 8;  // rows, channel-major key copy, position, score key
      now = (kept + gen) * slot + topk * 4;
      top = std::max(n0 * row + kept * slot, now);  // prefill: the whole prompt in fp16 before SnapKV
      break;
    }
  }
  *resident = (size_t)(now * shape->n_kv_heads);
  *peak = (size_t)(top * shape->n_kv_heads);
  return MKV_OK;
}

mkv_status mkv_attention_tiles(mkv_cache *c, int32_t *n_tiles, int32_t *n_tiles_uq, int32_t *n_tiles_rocket) {
  if (!c || !n_tiles) return fail(MKV_EINVAL, "NULL argument");
  *n_tiles = c->dv.n_tiles;
  if (n_tiles_uq) *n_tiles_uq = c->dv.n_tiles_uq;
  if (n_tiles_rocket) *n_tiles_rocket = c->dv.n_tiles_rk;
  return MKV_OK;
}

mkv_status mkv_probe_read_bandwidth(const void *buf, size_t bytes, uint32_t *sink, int32_t reps, double *gbs,
                                    void *stream) {
  constexpr size_t kChunk = 256 << 10;
  if (!buf || !sink || !gbs) return fail(MKV_EINVAL, "NULL argument");
  if (bytes == 0 || bytes % kChunk != 0) return fail(MKV_EINVAL, "bytes must be a positive multiple of 256 KiB");
  if (bytes / kChunk > 0x7FFFFFFFu) return fail(MKV_EINVAL, "buffer too large");
  if (reps < 1) return fail(MKV_EINVAL, "reps must be >= 1");
  hipStream_t st = static_cast<hipStream_t>(stream);
  hipEvent_t a = nullptr, b = nullptr;
  hipError_t e = hipEventCreate(&a);
  if (e == hipSuccess) e = hipEventCreate(&b);
  if (e == hipSuccess) e = launch_probe_read(buf, bytes, kChunk, sink, st);
  float best = 0.f;
  for (int r = 0; r < reps && e == hipSuccess; ++r) {
    e = hipEventRecord(a, st);
    if (e == hipSuccess) e = launch_probe_read(buf, bytes, kChunk, sink, st);
    if (e == hipSuccess) e = hipEventRecord(b, st);
    if (e == hipSuccess) e = hipEventSynchronize(b);
    float ms = 0.f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, a, b);
    if (e == hipSuccess && (best == 0.f || ms < best)) best = ms;
  }
  if (a) (void)hipEventDestroy(a);
  if (b) (void)hipEventDestroy(b);
  if (e != hipSuccess) return hip_fail(e, "read probe");
  *gbs = best > 0.f ? (double)bytes / (best * 1e-3) / 1e9 : 0.0;
  return MKV_OK;
}

mkv_status mkv_profile_enable(mkv_cache *c, int32_t enable, int32_t max_launches) {
  if (!c) return fail(MKV_EINVAL, "cache is NULL");
  if (enable < 0 || enable >= (1 << kProfKinds)) return fail(MKV_EINVAL, "enable must be a mask of kinds 0..%d", kProfKinds - 1);
  if (enable && max_launches < 1) return fail(MKV_EINVAL, "max_launches must be >= 1");
  hipError_t e = hipDeviceSynchronize();
  if (e != hipSuccess) return hip_fail(e, "profile enable");
  for (int k = 0; k < kProfKinds; ++k) {
    for (int w = 0; w < 2; ++w) {
      for (hipEvent_t ev : c->ev[k][w]) (void)hipEventDestroy(ev);
      c->ev[k][w].clear();
      if (enable >> k & 1)
        for (int i = 0; i < max_launches; ++i) {
          hipEvent_t ev;
          if ((e = hipEventCreate(&ev)) != hipSuccess) return hip_fail(e, "hipEventCreate");
          c->ev[k][w].push_back(ev);
        }
    }
    c->prof_n[k] = 0;
  }
  c->prof_mask = enable;
  c->prof_cap = enable ? max_launches : 0;
  return MKV_OK;
}

mkv_status mkv_profile_read(mkv_cache *c, int32_t kind, int32_t *launches, double *total_ms) {
  if (!c || !launches || !total_ms) return fail(MKV_EINVAL, "NULL argument");
  if (kind < 0 || kind >= kProfKinds) return fail(MKV_EINVAL, "kind out of range");
  double tot = 0.0;
  for (int i = 0; i < c->prof_n[kind]; ++i) {
    hipError_t e = hipEventSynchronize(c->ev[kind][1][i]);
    if (e != hipSuccess) return hip_fail(e, "hipEventSynchronize");
    float ms = 0.f;
    if ((e = hipEventElapsedTime(&ms, c->ev[kind][0][i], c->ev[kind][1][i])) != hipSuccess)
      return hip_fail(e, "hipEventElapsedTime");
    tot += ms;
  }
  *launches = c->prof_n[kind];
  *total_ms = tot;
  return MKV_OK;
}

}  // extern "C"

// ---- export -------------------------------------------------------------------------------------
namespace {

template <typename T>
mkv_status dget(std::vector<T> &dst, uint64_t src, size_t n) {
  dst.resize(n);
  if (n == 0) return MKV_OK;
  hipError_t e = hipMemcpy(dst.data(), reinterpret_cast<const void *>(src), n * sizeof(T), hipMemcpyDeviceToHost);
  return check_hip(e, "export copy");
}

// Code `i` of a packed bit string: bits [bits*i, bits*i + bits), little-endian.
int unpack_bits(const uint8_t *p, int i, int bits) {
  const int bit = bits * i;
  uint32_t w = p[bit >> 3];
  if ((bit & 7) + bits > 8) w |= (uint32_t)p[(bit >> 3) + 1] << 8;
  return (int)((w >> (bit & 7)) & ((1u << bits) - 1));
}

}  // namespace

extern "C" mkv_status mkv_export(mkv_cache *c, int32_t seq, int32_t h, int32_t what, void *host_dst, size_t cap,
                                 size_t *written) {
  if (!c || !written) return fail(MKV_EINVAL, "NULL argument");
  *written = 0;
  if (seq < 0 || seq >= c->sh.S || h < 0 || h >= c->sh.Hkv) return fail(MKV_EINVAL, "seq or kv_head out of range");
  hipError_t e = hipDeviceSynchronize();
  if (e != hipSuccess) return hip_fail(e, "export sync");
  const SeqDesc &d = c->hs[seq];
  const int D = c->sh.D, G = c->sh.G;
  std::vector<int32_t> stv;
  mkv_status st = dget(stv, (uint64_t)(uintptr_t)(c->dv.state + ((size_t)seq * c->sh.Hkv + h) * ST_WORDS), ST_WORDS);
  if (st != MKV_OK) return st;
  const int count = stv[ST_COUNT];
  // H2O: a victim whose eviction is pending is no longer part of the retained set (the lowest key
  // among the last attention pass's per-part candidates)
  int gone = -1;
  if (d.method == H2O && c->evict_pending) {
    std::vector<uint32_t> vb;
    if ((st = dget(vb, d.vbest + (uint64_t)h * d.vparts * 16, (size_t)d.vparts * 4)) != MKV_OK) return st;
    unsigned long long best = ~0ull;
    for (int p = 0; p < d.vparts; ++p) {
      const unsigned long long key = (unsigned long long)vb[4 * p] | ((unsigned long long)vb[4 * p + 1] << 32);
      if (key < best) {
        best = key;
        gone = (int)vb[4 * p + 2];
      }
    }
  }
  std::vector<uint8_t> out;
  auto put = [&](const void *p, size_t bytes) {
    const uint8_t *b = static_cast<const uint8_t *>(p);
    out.insert(out.end(), b, b + bytes);
  };
  switch (what) {
    case MKV_EXPORT_COUNTS: {
      const int held = gone >= 0 ? count - 1 : count;
      int32_t v[4] = {held, stv[ST_NEXT_POS], d.method == ROCKET ? stv[ST_SEL_COUNT] : held, stv[ST_KEPT]};
      put(v, sizeof v);
      break;
    }
    case MKV_EXPORT_POSITIONS:
    case MKV_EXPORT_SCORES: {
      if (d.method == H2O || d.method == ROCKET) {
        // slots 0..count-1 hold the retained tokens
        const int nread = count;
        std::vector<int32_t> pos;
        if ((st = dget(pos, d.pos + (uint64_t)h * stride_slots(d) * 4, nread)) != MKV_OK) return st;
        std::vector<float> sc;
        if (d.method == H2O && (st = dget(sc, d.score + (uint64_t)h * stride_slots(d) * 4, nread)) != MKV_OK) return st;
        std::vector<int> order;
        for (int i = 0; i < nread; ++i)
          if (pos[i] >= 0 && i != gone) order.push_back(i);
        std::sort(order.begin(), order.end(), [&](int a, int b) { return pos[a] < pos[b]; });
        for (int i : order) {
          if (what == MKV_EXPORT_POSITIONS) put(&pos[i], 4);
          else if (d.method == H2O) put(&sc[i], 4);
        }
        if (what == MKV_EXPORT_SCORES && d.method != H2O) return fail(MKV_EINVAL, "SCORES is for H2O sequences");
      } else {
        if (what == MKV_EXPORT_SCORES) return fail(MKV_EINVAL, "SCORES is for H2O sequences");
        for (int32_t i = 0; i < count; ++i) put(&i, 4);
      }
      break;
    }
    case MKV_EXPORT_CODES_K:
    case MKV_EXPORT_CODES_V: {
      if (d.method != KVQ && d.method != UQ) return fail(MKV_EINVAL, "codes exist for UQ and KVQ sequences");
      const bool isk = what == MKV_EXPORT_CODES_K;
      const int n = (d.method == UQ && isk) ? (count / 64) * 64 : count;
      const int bits = d.method == UQ ? 4 : d.bits;
      // values sit in 4-token blocks: KVQ code of channel c, token j at bit bits*(4c + j); UQ as
      // laid out by uq_vbit; key code rows are one token each
      const bool quad = !isk;
      const size_t nbytes = (size_t)(quad ? (n + 3) & ~3 : n) * d.rowbytes;
      std::vector<uint8_t> raw;
      if ((st = dget(raw, (isk ? d.kc : d.vc) + (uint64_t)h * stride_codes(d), nbytes)) != MKV_OK) return st;
      for (int t = 0; t < n; ++t)
        for (int ch = 0; ch < D; ++ch) {
          const uint8_t *blk = raw.data() + (size_t)(t / 4) * 4 * d.rowbytes;
          uint8_t code;
          if (!quad) code = (uint8_t)unpack_bits(raw.data() + (size_t)t * d.rowbytes, ch, bits);
          else if (d.method == KVQ) code = (uint8_t)unpack_bits(blk, 4 * ch + (t & 3), bits);
          else code = (uint8_t)((blk[uq_vbit(ch, t & 3, D) >> 3] >> (uq_vbit(ch, t & 3, D) & 7)) & 15u);
          put(&code, 1);
        }
      break;
    }
    case MKV_EXPORT_OUTLIERS_K:
    case MKV_EXPORT_OUTLIERS_V: {
      if (d.method != KVQ) return fail(MKV_EINVAL, "outliers exist for KVQ sequences");
      std::vector<int32_t> m((size_t)count * D, -1);
      if (what == MKV_EXPORT_OUTLIERS_K) {
        std::vector<uint32_t> row, pool;
        if ((st = dget(row, d.krow + (uint64_t)h * stride_krow(d) * 4, count + 1)) != MKV_OK) return st;
        if ((st = dget(pool, d.kout + (uint64_t)h * stride_kout(d) * 4, row[count])) != MKV_OK) return st;
        for (int t = 0; t < count; ++t)
          for (uint32_t e2 = row[t]; e2 < row[t + 1]; ++e2) m[(size_t)t * D + outlier_ch(pool[e2])] = (int32_t)(pool[e2] >> 16);
      } else {
        std::vector<uint32_t> vo;
        if ((st = dget(vo, d.vout + (uint64_t)h * stride_vout(d) * 4, (size_t)d.cap * d.nov_slots)) != MKV_OK)
          return st;
        for (int t = 0; t < count; ++t)
          for (int j = 0; j < d.nov_slots; ++j) {
            const uint32_t ent = vo[(size_t)j * d.cap + t];
            if (ent == kNoOutlier) break;
            m[(size_t)t * D + outlier_ch(ent)] = (int32_t)(ent >> 16);
          }
      }
      put(m.data(), m.size() * 4);
      break;
    }
    case MKV_EXPORT_SCALES_K:
    case MKV_EXPORT_SCALES_V: {
      if (d.method == KVQ) {
        if (what == MKV_EXPORT_SCALES_K) {
          std::vector<float> t2;
          if ((st = dget(t2, d.kmeta + (uint64_t)h * D * 8, (size_t)2 * D)) != MKV_OK) return st;
          for (int ch = 0; ch < D; ++ch) put(&t2[2 * ch], 4);
        } else {
          std::vector<float> s;
          if ((st = dget(s, d.vmeta + (uint64_t)h * stride_slots(d) * 4, count)) != MKV_OK) return st;
          put(s.data(), s.size() * 4);
        }
      } else if (d.method == UQ) {
        std::vector<float> m;
        if (what == MKV_EXPORT_SCALES_K) {
          if ((st = dget(m, d.kmeta + (uint64_t)h * stride_uq_kmeta(d, D) * 8, (size_t)(count / 64) * D * 2)) != MKV_OK)
            return st;
        } else {
          if ((st = dget(m, d.vmeta + (uint64_t)h * stride_uq_vmeta(d, D) * 8, (size_t)count * (D / 64) * 2)) != MKV_OK)
            return st;
        }
        put(m.data(), m.size() * 4);
      } else {
        return fail(MKV_EINVAL, "scales exist for UQ and KVQ sequences");
      }
      break;
    }
    case MKV_EXPORT_TOPK: {
      if (d.method != ROCKET) return fail(MKV_EINVAL, "TOPK is for ROCKET sequences");
      const int m = stv[ST_SEL_COUNT];
      std::vector<int32_t> sel, pos;
      if ((st = dget(sel, d.sel + (uint64_t)h * stride_sel(d) * 4, m)) != MKV_OK) return st;
      if ((st = dget(pos, d.pos + (uint64_t)h * stride_slots(d) * 4, count)) != MKV_OK) return st;
      for (int i = 0; i < m; ++i) put(&pos[sel[i]], 4);
      break;
    }
    case MKV_EXPORT_CHANNELS: {
      if (d.method != ROCKET) return fail(MKV_EINVAL, "CHANNELS is for ROCKET sequences");
      std::vector<int32_t> ch;
      if ((st = dget(ch, d.aux1 + (uint64_t)h * D * 4, d.nch)) != MKV_OK) return st;
      put(ch.data(), ch.size() * 4);
      break;
    }
    default:
      return fail(MKV_EINVAL, "unknown export kind %d", what);
  }
  (void)G;
  if (out.size() > cap) return fail(MKV_EINVAL, "export needs %zu bytes, cap is %zu", out.size(), cap);
  if (!out.empty()) std::memcpy(host_dst, out.data(), out.size());
  *written = out.size();
  return MKV_OK;
}
