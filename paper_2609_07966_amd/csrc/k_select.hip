// Token-selection kernels: RocketKV top-k, H2O eviction, H2O and SnapKV prefill eviction.
//
// MetaKV Section 2.1: H2O keeps the tokens with the highest accumulated attention and evicts the
// lowest-scoring older token once over budget; RocketKV first keeps the prompt tokens the
// observation window votes for (SnapKV), then attends to a top-k subset per decode step.
// Selections are block-wide radix selects on order-preserving 32-bit keys followed by an
// ascending-position compaction, so ties resolve by position exactly as specified.
#include "select_dev.h"

namespace mkv {

namespace {

constexpr int NT = 256;

// ---- RocketKV decode top-k ---------------------------------------------------------------------
// One workgroup of kTopkThreads threads per (sequence, kv head) over the tokens already appended
// (a decode step instead spreads the scores over several workgroups, in k_append.hip).
template <int D, int G>
__global__ __launch_bounds__(kTopkThreads, 8) void k_topk(const SeqDesc *__restrict__ seqs, int32_t *state,
                                                       const uint16_t *__restrict__ q, int32_t *pos_out,
                                                       int topk_max, int Hkv) {
  __shared__ TopkLds<D> L;
  const int seq = blockIdx.x / Hkv, h = blockIdx.x % Hkv;
  const SeqDesc &sd = seqs[seq];
  if (sd.method != ROCKET) return;
  int32_t *st = state + ((size_t)seq * Hkv + h) * ST_WORDS;
  topk_pair<D, G>(sd, st, seq, h, Hkv, st[ST_COUNT], q, pos_out, topk_max, L);
}

// ---- causal prefill attention statistics for H2O scoring, on the matrix cores ------------------
// A kv head's query rows are taken as virtual rows r = position * G + g (its G query heads at one
// position are adjacent in memory).  Logit tiles S^T = K Q^T of 32 keys x 32 virtual rows come from
// v_mfma_f32_32x32x16_f16: Q and K are fp16 exactly, products exact, sums in float32.  Operand lane
// roles (lr = lane % 32, lh = lane / 32): A key lr, B row lr, both channels 8 lh .. 8 lh + 7 of the
// k-step; result element i: key 8 (i / 4) + 4 lh + i % 4, row lr.  A lane thus owns one row of a
// tile and 16 of its keys: row statistics stay in the lane, and a row's (max, 1 / sum) is one pair
// per lane in the column sums.
//
// Both kernels hold 64 rows or keys per wave in registers (64 VGPRs at d = 128) and stream 64-item
// tiles of the other side through a double-buffered LDS stage shared by the 4 waves, so an operand
// read from LDS feeds two matrix instructions and an item is read from L2 once per 256 on the other
// side.  Tiles wholly below the diagonal take a path without masks, where a logit costs one fma, one
// exp2 and one add or fma (3.6 ns of a SIMD for a wave's exp2, 1.1 for each of the others, measured in
// loops of nothing else).  For 8 prompts of 8192 tokens these are 0.75 ms a pass and the products 1.9 at
// the rate of a large library product; the passes take 2.3 and 2.8, about the sum: a tile's exponentials
// wait for its products (counters: vector unit busy 71 % of the row statistics' cycles, matrix cores 53 %,
// at a clock of 1.7 GHz under this load).  Heads are the fastest grid index, so that with 8 kv heads each
// head's K and Q stay in one XCD's L2.  8 prompts of 8192 tokens, 32 query / 8 kv heads x 128: row
// statistics 4.75 -> 2.31 ms (950 TFLOP/s of causal products), column sums 7.30 -> 2.80 ms (790), where one
// workgroup per 64 rows or keys and launches per sequence stood before; a library matrix product reaches
// 1150 here.
// The column sums are held to 168 registers (three waves per SIMD; 2.90 ms at 220 and two).
typedef _Float16 h8v __attribute__((ext_vector_type(8)));
typedef float f16v __attribute__((ext_vector_type(16)));

MKV_DEV f16v mfma32(const uint4 &a, const uint4 &b, f16v c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8v, a), __builtin_bit_cast(h8v, b), c, 0, 0, 0);
}

constexpr int kScoreTile = 64;  // streamed items per LDS stage
constexpr int kScoreBlock = 4 * kScoreTile;  // resident rows or keys per workgroup

// A streamed tile: kScoreTile rows of D halves, padded by one 16-byte unit so that the 16 lanes of
// a read phase start in different banks.
template <int D>
struct ScoreStage {
  uint4 row[2][kScoreTile][D / 8 + 1];
};

// Sums over the 32 lanes of each half wave: lane lr gets the total of v[lr % N].  At step o the lanes
// with bit o clear keep the even values of each pair and the others the odd ones.
template <int N>
MKV_DEV float half_wave_sums(float (&v)[N]) {
  static_assert(N == 16 || N == 32, "a value per lane, or per two lanes");
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1, n = N; n > 1; o <<= 1, n >>= 1) {
    const bool odd = lane & o;
#pragma unroll
    for (int i = 0; i < n / 2; ++i) {
      const float keep = odd ? v[2 * i + 1] : v[2 * i], send = odd ? v[2 * i] : v[2 * i + 1];
      v[i] = keep + __shfl_xor(send, o);
    }
  }
  return N == 32 ? v[0] : v[0] + __shfl_xor(v[0], 16);
}

// Query row of virtual row r (clamped to the prompt) of kv head h, in 16-byte units.
template <int D>
MKV_DEV const uint4 *vrow_ptr(const uint16_t *q, const SeqDesc &sd, int r, int h, int Hq, int lg) {
  const int rc = min(r, (sd.n0 << lg) - 1);
  return reinterpret_cast<const uint4 *>(
      q + ((size_t)(sd.q_off + (rc >> lg)) * Hq + (h << lg) + (rc & ((1 << lg) - 1))) * D);
}

// Row statistics (reference m, 1 / sum of exp2(logit - m)) of every virtual row over its causal
// keys.  A workgroup takes kScoreBlock virtual rows, the longest first, and walks the key tiles up
// to the diagonal.  A lane's reference is the largest logit of its row's first tile and moves only
// when a tile's sum passes 2^80: float32 sums are as precise at any scale, so the tile maximum is
// not needed otherwise.
template <int D>
__global__ __launch_bounds__(NT) void k_h2o_rowstats(const SeqDesc *__restrict__ seqs,
                                                     const int32_t *__restrict__ list,
                                                     const uint16_t *__restrict__ q, int Hq, int Hkv, int lg,
                                                     float scale2) {
  constexpr int KS = D / 16, U = D / 8, PER = kScoreTile * U / NT;
  constexpr float kMove = 1.2089258196146292e24f;  // 2^80
  __shared__ ScoreStage<D> L;
  const SeqDesc &sd = seqs[list[blockIdx.y]];
  const int n0 = sd.n0, h = blockIdx.x % Hkv;
  const int rb = ((n0 << lg) + kScoreBlock - 1) / kScoreBlock - 1 - (int)blockIdx.x / Hkv;
  if (rb < 0) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 31, lh = lane >> 5;
  const int r0 = rb * kScoreBlock + 64 * wave;  // this wave's first virtual row
  const int p0 = min(r0 >> lg, n0 - 1), p1 = min((r0 + 63) >> lg, n0 - 1);
  uint4 qa[2][KS];
  int pos[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const uint4 *qp = vrow_ptr<D>(q, sd, r0 + 32 * t + lr, h, Hq, lg);
    pos[t] = min((r0 + 32 * t + lr) >> lg, n0 - 1);
#pragma unroll
    for (int s = 0; s < KS; ++s) qa[t][s] = gld16(qp + 2 * s + lh);
  }
  const uint4 *ks = reinterpret_cast<const uint4 *>(reinterpret_cast<const uint16_t *>(sd.stage_k) +
                                                    h * stride_stage(sd, D));
  float m[2] = {-INFINITY, -INFINITY}, l[2] = {0.f, 0.f};
  const int last = min((rb * kScoreBlock + kScoreBlock - 1) >> lg, n0 - 1) / kScoreTile;
  uint4 nxt[PER];
  auto load = [&](int kb) {
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int e = threadIdx.x + k * NT;
      nxt[k] = gld16(ks + (size_t)min(kb * kScoreTile + e / U, n0 - 1) * U + e % U);
    }
  };
  load(0);
  for (int kb = 0; kb <= last; ++kb) {
    // one barrier per tile: a stage is rewritten two tiles later, after every wave has passed the
    // barrier between
    auto &st = L.row[kb & 1];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int e = threadIdx.x + k * NT;
      st[e / U][e % U] = nxt[k];
    }
    __syncthreads();
    if (kb < last) load(kb + 1);
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
      const int key0 = kb * kScoreTile + 32 * sub;
      if (key0 > p1) break;
      f16v S[2] = {};
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const uint4 a = st[32 * sub + lr][2 * s + lh];
        S[0] = mfma32(a, qa[0][s], S[0]);
        S[1] = mfma32(a, qa[1][s], S[1]);
      }
      bool open = key0 + 31 <= p0 && key0 > 0;  // no mask, and every lane has a reference
      if (open) {
        float t[2][2] = {};
#pragma unroll
        for (int i = 0; i < 16; ++i)
#pragma unroll
          for (int u = 0; u < 2; ++u) t[u][i & 1] += fexp2(fmaf(S[u][i], scale2, -m[u]));
        t[0][0] += t[0][1];
        t[1][0] += t[1][1];
        open = !__any(!(t[0][0] < kMove && t[1][0] < kMove));
        if (open) {
          l[0] += t[0][0];
          l[1] += t[1][0];
        }
      }
      if (!open) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int rel = pos[u] - key0 - 4 * lh;  // compared with constants
          float mx = m[u];
#pragma unroll
          for (int i = 0; i < 16; ++i) mx = fmaxf(mx, 8 * (i / 4) + (i & 3) <= rel ? S[u][i] * scale2 : -INFINITY);
          if (mx == -INFINITY) continue;  // every key so far is masked
          l[u] *= fexp2(m[u] - mx);
          m[u] = mx;
#pragma unroll
          for (int i = 0; i < 16; ++i)
            l[u] += 8 * (i / 4) + (i & 3) <= rel ? fexp2(fmaf(S[u][i], scale2, -mx)) : 0.f;
        }
      }
    }
  }
  float2 *out = reinterpret_cast<float2 *>(sd.aux1) + ((size_t)h * n0 << lg);
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    // the two halves of a wave hold disjoint keys of the row (a half without keys: m = -inf, l = 0)
    const float mo = __shfl_xor(m[u], 32), lo = __shfl_xor(l[u], 32);
    const float M = fmaxf(m[u], mo);
    const float sum = (m[u] == -INFINITY ? 0.f : l[u] * fexp2(m[u] - M)) + (mo == -INFINITY ? 0.f : lo * fexp2(mo - M));
    const int r = r0 + 32 * u + lr;
    if (lh == 0 && r < (n0 << lg)) out[r] = make_float2(M, 1.f / sum);
  }
}

// Column sums S_j = sum_r p_rj of kScoreBlock keys over one segment of the virtual rows (those at or
// below the diagonal), into that segment's row of the partial sums; k_h2o_sum adds the segments in
// order.  Splitting the rows into up to kScoreSegs segments gives one prompt enough workgroups of
// similar length (a block of keys would otherwise carry up to all rows), and the workgroups in
// flight of one segment share its query rows in L2.
template <int D>
__global__ __launch_bounds__(NT, 3) void k_h2o_colsums(const SeqDesc *__restrict__ seqs,
                                                    const int32_t *__restrict__ list,
                                                    const uint16_t *__restrict__ q, int Hq, int Hkv, int lg,
                                                    float scale2) {
  constexpr int KS = D / 16, U = D / 8, PER = kScoreTile * U / NT;
  __shared__ ScoreStage<D> L;
  __shared__ float2 s_stat[2][kScoreTile];  // (reference, 1 / sum) of the streamed rows
  const SeqDesc &sd = seqs[list[blockIdx.y]];
  const int n0 = sd.n0, h = blockIdx.x % Hkv, V = n0 << lg;
  const int nkb = (n0 + kScoreBlock - 1) / kScoreBlock, item = (int)blockIdx.x / Hkv;
  const int seg = sd.nseg - 1 - item / nkb, kb = item % nkb;
  const int v0 = max(seg * sd.seg_rows, (kb * kScoreBlock) << lg), v1 = min((seg + 1) * sd.seg_rows, V);
  if (seg < 0 || v0 >= v1) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 31, lh = lane >> 5;
  const int key0 = kb * kScoreBlock + 64 * wave;
  const uint4 *ks = reinterpret_cast<const uint4 *>(reinterpret_cast<const uint16_t *>(sd.stage_k) +
                                                    h * stride_stage(sd, D));
  const float *stat = reinterpret_cast<const float *>(sd.aux1) + 2 * ((size_t)h * n0 << lg);
  uint4 ka[2][KS];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int s = 0; s < KS; ++s) ka[u][s] = gld16(ks + (size_t)min(key0 + 32 * u + lr, n0 - 1) * U + 2 * s + lh);
  float acc[32];
#pragma unroll
  for (int i = 0; i < 32; ++i) acc[i] = 0.f;
  // v0 is a multiple of kScoreTile (segments and key blocks are)
  // (a tile starts at a whole position: its rows' offsets from there are the same for every tile, up
  // to the clamp to the prompt, so addresses are a uniform base plus a 32-bit offset)
  uint4 nxt[PER];
  float Mn = 0.f, In = 0.f;  // the next tile's statistics: thread t < kScoreTile takes row t
  const uint32_t pitch = (uint32_t)Hq * D * 2;
  auto load = [&](int v) {
    const char *qt = reinterpret_cast<const char *>(q + ((size_t)(sd.q_off + (v >> lg)) * Hq + ((size_t)h << lg)) * D);
    const char *ml = reinterpret_cast<const char *>(stat + 2 * (size_t)v);
    const int end = V - 1 - v;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int r = min((int)(threadIdx.x / U) + k * (NT / U), end);
      nxt[k] = gld16(qt + ((uint32_t)(r >> lg) * pitch + (uint32_t)(r & ((1 << lg) - 1)) * (D * 2) + (threadIdx.x % U) * 16));
    }
    if (threadIdx.x < kScoreTile) {
      const float *p = reinterpret_cast<const float *>(ml + (uint32_t)min((int)threadIdx.x, end) * 8);
      Mn = gld(p);
      const float x = gld(p + 1);
      In = (int)threadIdx.x <= end ? x : 0.f;  // rows past the prompt add nothing
    }
  };
  load(v0);
  int buf = 0;
  for (int v = v0; v < v1; v += kScoreTile, buf ^= 1) {
    auto &st = L.row[buf];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int e = threadIdx.x + k * NT;
      st[e / U][e % U] = nxt[k];
    }
    if (threadIdx.x < kScoreTile) s_stat[buf][threadIdx.x] = make_float2(Mn, In);
    __syncthreads();
    if (v + kScoreTile < v1) load(v + kScoreTile);
#pragma unroll 1
    for (int t = 0; t < 2; ++t) {
      const int r = v + 32 * t;
      if (key0 > (r + 31) >> lg) continue;  // wholly above the diagonal
      const float2 mi = s_stat[buf][32 * t + lr];
      f16v S[2] = {};
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const uint4 b = st[32 * t + lr][2 * s + lh];
        S[0] = mfma32(ka[0][s], b, S[0]);
        S[1] = mfma32(ka[1][s], b, S[1]);
      }
      if (key0 + 63 <= r >> lg) {
#pragma unroll
        for (int i = 0; i < 32; ++i) acc[i] = fmaf(fexp2(fmaf(S[i / 16][i % 16], scale2, -mi.x)), mi.y, acc[i]);
      } else {
        const int rel = ((r + lr) >> lg) - key0 - 4 * lh;  // compared with constants
#pragma unroll
        for (int i = 0; i < 32; ++i) {
          const float p = fexp2(fmaf(S[i / 16][i % 16], scale2, -mi.x)) * mi.y;
          acc[i] += 8 * (i / 4) + (i & 3) <= rel ? p : 0.f;
        }
      }
    }
  }
  const float sum = half_wave_sums(acc);
  const int key = key0 + 32 * (lr / 16) + 8 * ((lr / 4) & 3) + 4 * lh + (lr & 3);
  if (key < n0) gst(reinterpret_cast<float *>(sd.colpart) + ((size_t)h * sd.nseg + seg) * n0 + key, sum);
}

// Scores: the segments' column sums added in ascending order (a key's first segment is the one its
// block's diagonal lies in).
__global__ __launch_bounds__(NT) void k_h2o_sum(const SeqDesc *__restrict__ seqs, const int32_t *__restrict__ list,
                                                int Hkv, int lg) {
  const SeqDesc &sd = seqs[list[blockIdx.y]];
  const int n0 = sd.n0, h = blockIdx.x % Hkv, j = (int)blockIdx.x / Hkv * NT + (int)threadIdx.x;
  if (j >= n0) return;
  const float *part = reinterpret_cast<const float *>(sd.colpart) + (size_t)h * sd.nseg * n0 + j;
  float acc = 0.f;
  for (int s = (j / kScoreBlock * kScoreBlock << lg) / sd.seg_rows; s < sd.nseg; ++s) acc += gld(part + (size_t)s * n0);
  gst(reinterpret_cast<float *>(sd.aux0) + (size_t)h * n0 + j, acc);
}

// Keys of the scores at and before p, in descending order of position.
struct ReversedScores {
  const float *p;
  MKV_DEV uint32_t operator()(int i) const { return float_key(gld(p - i)); }
  MKV_DEV uint4 four(int i) const {
    const uint4 x = gld16w(reinterpret_cast<const uint32_t *>(p - i - 3));
    return make_uint4(float_key(__uint_as_float(x.w)), float_key(__uint_as_float(x.z)),
                      float_key(__uint_as_float(x.y)), float_key(__uint_as_float(x.x)));
  }
};

// Keep the R most recent prompt tokens plus the top B - R scores of the rest (newer on ties): their
// positions into slots 0..kept-1 in ascending order, and the head's state.  The selection runs over
// the candidates in reverse order (index ncand - 1 - j), so that its lower-index tie rule prefers
// newer tokens; its ascending output, reversed, is ascending in position.
__global__ __launch_bounds__(kTopkThreads) void k_h2o_keep(const SeqDesc *__restrict__ seqs,
                                                           const int32_t *__restrict__ list, int32_t *state,
                                                           int Hkv) {
  __shared__ SelLds L;
  const int seq = list[blockIdx.y];
  const SeqDesc &sd = seqs[seq];
  const int h = blockIdx.x, n0 = sd.n0;
  const float *S = reinterpret_cast<const float *>(sd.aux0) + (size_t)h * n0;
  const int B = sd.B, R = sd.R;
  const bool all = B >= n0;
  const int ncand = all ? 0 : n0 - R;
  const int H = all ? 0 : B - R;
  const int kept = all ? n0 : min(B, sd.cap);
  int32_t *pos = reinterpret_cast<int32_t *>(sd.pos) + h * stride_slots(sd);
  if (all) {
    for (int j = threadIdx.x; j < n0; j += kTopkThreads) pos[j] = j;
  } else {
    if (H > 0) {
      // the scratch of the row statistics (no longer needed) takes the reversed selection
      int32_t *rsel = reinterpret_cast<int32_t *>(sd.aux1) + (size_t)h * n0;
      select_keys<kTopkThreads, 32>(ncand, H, ReversedScores{S + (ncand - 1)}, rsel, L);
      __syncthreads();
      for (int i = threadIdx.x; i < H; i += kTopkThreads) pos[H - 1 - i] = ncand - 1 - gld(rsel + i);
    }
    for (int i = threadIdx.x; i < R; i += kTopkThreads) pos[H + i] = ncand + i;
  }
  // no eviction candidates before the first attention pass
  uint32_t *vb = reinterpret_cast<uint32_t *>(sd.vbest) + (size_t)h * sd.vparts * 4;
  for (int p = threadIdx.x; p < sd.vparts; p += kTopkThreads) {
    vb[4 * p] = 0xFFFFFFFFu;
    vb[4 * p + 1] = 0xFFFFFFFFu;
    vb[4 * p + 2] = 0xFFFFFFFFu;
    vb[4 * p + 3] = 0u;
  }
  if (threadIdx.x == 0) {
    int32_t *st = state + ((size_t)seq * Hkv + h) * ST_WORDS;
    set_counts(st, kept, n0);
    st[ST_KEPT] = kept;
  }
}

// The kept rows and their scores, gathered from the staged prompt: a workgroup per kGatherSlots
// slots (selection and gather of 8 x 8192 prompts: 490 us with the gather in the selecting workgroup,
// one per kv head, and launches per sequence; 38 us apart and over all sequences).
constexpr int kGatherSlots = 64;
template <int D>
__global__ __launch_bounds__(NT) void k_h2o_gather(const SeqDesc *__restrict__ seqs, const int32_t *__restrict__ list,
                                                   int Hkv) {
  constexpr int U = D / 8, PER = kGatherSlots * U / NT;
  const SeqDesc &sd = seqs[list[blockIdx.y]];
  const int h = blockIdx.x % Hkv, s0 = (int)blockIdx.x / Hkv * kGatherSlots, n0 = sd.n0;
  const int kept = sd.B >= n0 ? n0 : min(sd.B, sd.cap);
  if (s0 >= kept) return;
  const int32_t *pos = reinterpret_cast<const int32_t *>(sd.pos) + h * stride_slots(sd);
  const uint16_t *sk = reinterpret_cast<const uint16_t *>(sd.stage_k) + h * stride_stage(sd, D);
  const uint16_t *sv = reinterpret_cast<const uint16_t *>(sd.stage_v) + h * stride_stage(sd, D);
  uint16_t *dk = reinterpret_cast<uint16_t *>(sd.k) + h * stride_rows(sd, D);
  uint16_t *dvv = reinterpret_cast<uint16_t *>(sd.v) + h * stride_rows(sd, D);
  int jj[PER];
  uint4 a[PER], b[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) jj[k] = gld(pos + min(s0 + (int)(threadIdx.x + k * NT) / U, kept - 1));
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int u = threadIdx.x % U;
    a[k] = gld16(sk + (size_t)jj[k] * D + 8 * u);
    b[k] = gld16(sv + (size_t)jj[k] * D + 8 * u);
  }
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int slot = s0 + (int)(threadIdx.x + k * NT) / U, u = threadIdx.x % U;
    if (slot >= kept) break;
    *reinterpret_cast<uint4 *>(dk + (size_t)slot * D + 8 * u) = a[k];
    *reinterpret_cast<uint4 *>(dvv + (size_t)slot * D + 8 * u) = b[k];
    if (u == 0)
      (reinterpret_cast<float *>(sd.score) + h * stride_slots(sd))[slot] =
          gld(reinterpret_cast<const float *>(sd.aux0) + (size_t)h * n0 + jj[k]);
  }
}

// ---- SnapKV prefill -------------------------------------------------------------------------------
// Window row r = i * G + g (query head h*G + g at position n0 - w + i; it attends to keys
// 0 .. n0 - w + i).  Pass 1: per chunk of keys the partial (max, sum of exp2) of every row.  Pass 2:
// each row's partials merged.  Pass 3: the votes of a span's keys, the logits recomputed.  Pass 4: max
// pooling into order-preserving keys.  Pass 5: the selection; pass 6: the kept rows gathered.  Every
// pass is one launch over a group's sequences (grid as for H2O).
//
// Logit tiles as in the H2O scoring: S^T = K Q^T, a lane owning one row and 16 keys of a 32 x 32 tile.
// A workgroup takes a span of keys and holds ROWS window rows in LDS; a wave holds 32 keys as operands,
// loaded while it computes the 32 before, so the loads of K run under the products and exponentials
// and the rows are staged once per span.  (With one chunk of 256 keys per workgroup and the rows
// staged 64 at a time, every workgroup waited for its keys and again for its rows.)
//
// The spans are chosen for the whole batch, so nothing may depend on them: a row's sum is taken per lane
// over 64 keys, those of a 256-key chunk folded in ascending order, then the two lane halves, then the
// chunks, whichever waves took them; a key's votes are summed over the rows alone.  (Sums over whole
// spans rounded differently in other batches, and a near-tie in a keep-set fell differently.)  The whole
// selection, with sums over spans and now: 4 prompts of 32768 tokens 215 and 214 us, one of them 82 and 88
// (spans of 512 keys were the best there), 40 of 1500 145 and 136, 6 of 400 38 and 37.
constexpr int SNAP_CHUNK = 256;  // keys of a partial; with one chunk a workgroup, its waves take 64 keys each
constexpr int SNAP_KEYS = 32 * (NT / 64);  // keys a workgroup takes at a time (votes)
static_assert(SNAP_CHUNK == 64 * (NT / 64), "a wave per 64 keys of a chunk");

// (max, sum) of two disjoint key sets; an empty set is (-inf, 0).
MKV_DEV void snap_fold(float &M, float &L, float m, float l) {
  const float mx = fmaxf(M, m), ref = mx == -INFINITY ? 0.f : mx;
  L = L * fexp2(M - ref) + l * fexp2(m - ref);
  M = mx;
}

// The window rows [r0, r0 + ROWS) (clamped to the last row) as fp16 operands in LDS.
template <int D, int ROWS>
MKV_DEV void stage_window(uint4 (*sq)[D / 8 + 1], const uint16_t *qw, const SeqDesc &sd, int h, int lg, int Hq, int rows,
                          int r0) {
  constexpr int U = D / 8;
  const int n = min(ROWS, (rows - r0 + 31) & ~31);
  for (int e = threadIdx.x; e < n * U; e += NT) {
    const int rr = e / U, u = e % U;
    const int r = min(r0 + rr, rows - 1), i = r >> lg, g = r & ((1 << lg) - 1);
    // the last w_eff of the `window` rows
    sq[rr][u] = gld16(reinterpret_cast<const uint4 *>(
                          qw + ((size_t)(sd.q_off + sd.window - sd.w_eff + i) * Hq + (h << lg) + g) * D) + u);
  }
}

// f(key0, operands) over a wave's steps of 32 keys in the span [a, b): key key0 + lr, channels
// 8 lh .. 8 lh + 7 of k-step s, the next step's loads in flight (keys past the prompt: its last).
template <int D, typename F>
MKV_DEV void snap_steps(const SeqDesc &sd, int h, int a, int b, F f) {
  constexpr int U = D / 8;
  const uint4 *ks = reinterpret_cast<const uint4 *>(reinterpret_cast<const uint16_t *>(sd.stage_k) +
                                                    h * stride_stage(sd, D));
  const int lane = threadIdx.x & 63, lr = lane & 31, lh = lane >> 5, last = sd.n0 - 1;
  auto load = [&](int key0, uint4 (&ka)[D / 16]) {
#pragma unroll
    for (int s = 0; s < D / 16; ++s) ka[s] = gld16(ks + (size_t)min(key0 + lr, last) * U + 2 * s + lh);
  };
  uint4 x[D / 16], y[D / 16];
  int key0 = a + 32 * (threadIdx.x >> 6);
  if (key0 < b) load(key0, x);
  for (; key0 < b; key0 += 2 * SNAP_KEYS) {
    load(key0 + SNAP_KEYS, y);
    f(key0, x);
    if (key0 + SNAP_KEYS >= b) break;
    load(key0 + 2 * SNAP_KEYS, x);
    f(key0 + SNAP_KEYS, y);
  }
}

template <int D>
MKV_DEV f16v snap_logits(const uint4 (&ka)[D / 16], const uint4 (*sq)[D / 8 + 1], int row, int lh) {
  f16v S = {};
#pragma unroll
  for (int s = 0; s < D / 16; ++s) S = mfma32(ka[s], sq[row][2 * s + lh], S);
  return S;
}

// span: SNAP_CHUNK (the chunk's waves take 64 keys each), or a multiple of 4 chunks (a wave takes whole
// chunks).  Partials: [head][chunk][row].
template <int D, int ROWS>
__global__ __launch_bounds__(NT) void k_snap_rowstats(const SeqDesc *__restrict__ seqs,
                                                      const int32_t *__restrict__ list,
                                                      const uint16_t *__restrict__ qw, int Hq, int Hkv, int lg,
                                                      int span, float scale2) {
  constexpr int kTiles = ROWS / 32, kParts = 2 * (NT / 64), U = D / 8;
  __shared__ uint4 sq[ROWS][D / 8 + 1];
  float2(*s_part)[ROWS] = reinterpret_cast<float2(*)[ROWS]>(&sq[0][0]);  // once the rows are used
  static_assert(sizeof(float2) * kParts * ROWS <= sizeof(sq), "the partials fit the rows");
  const SeqDesc &sd = seqs[list[blockIdx.y]];
  const int n0 = sd.n0, w = sd.w_eff, h = blockIdx.x % Hkv, a = (int)blockIdx.x / Hkv * span;
  if (a >= n0 || sd.T >= n0) return;
  const int nchunk = (n0 + SNAP_CHUNK - 1) / SNAP_CHUNK, b = min(a + span, n0);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 31, lh = lane >> 5;
  const int rows = w << lg;
  const bool split = span == SNAP_CHUNK;
  const int run = split ? 64 : SNAP_CHUNK;  // consecutive keys a wave takes
  float2 *part = reinterpret_cast<float2 *>(sd.aux1) + (size_t)h * nchunk * rows;
  const uint4 *ks = reinterpret_cast<const uint4 *>(reinterpret_cast<const uint16_t *>(sd.stage_k) +
                                                    h * stride_stage(sd, D));
  auto load = [&](int key0, uint4 (&ka)[D / 16]) {
#pragma unroll
    for (int s = 0; s < D / 16; ++s) ka[s] = gld16(ks + (size_t)min(key0 + lr, n0 - 1) * U + 2 * s + lh);
  };
  for (int r0 = 0; r0 < rows; r0 += ROWS) {
    if (r0 > 0) __syncthreads();
    stage_window<D, ROWS>(sq, qw, sd, h, lg, Hq, rows, r0);
    __syncthreads();
    // of row r0 + 32 t + lr over the lane's own keys: (max, sum of exp2) of the 64 keys in progress, and
    // of those before them in the chunk
    float m[kTiles], l[kTiles], cm[kTiles], cl[kTiles];
#pragma unroll
    for (int t = 0; t < kTiles; ++t) m[t] = cm[t] = -INFINITY, l[t] = cl[t] = 0.f;
    auto step = [&](int key0, const uint4 (&ka)[D / 16]) {
      const bool end64 = (key0 + 32) % 64 == 0 || key0 + 32 >= b;
      const bool end_run = (key0 + 32) % run == 0 || key0 + 32 >= b;
#pragma unroll
      for (int t = 0; t < kTiles; ++t) {
        if (r0 + 32 * t >= rows) continue;
        f16v S = snap_logits<D>(ka, sq, 32 * t + lr, lh);
        if (key0 + 31 > n0 - w) {
          const int rel = n0 - w + ((r0 + 32 * t + lr) >> lg) - key0 - 4 * lh;  // compared with constants
          const int end = n0 - 1 - key0 - 4 * lh;
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int c = 8 * (i / 4) + (i & 3);
            S[i] = c <= min(rel, end) ? S[i] : -INFINITY;
          }
        }
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < 16; ++i) mx = fmaxf(mx, S[i]);
        mx = fmaxf(m[t], mx * scale2);
        const float ref = mx == -INFINITY ? 0.f : mx;  // no visible key yet: a sum of 0
        float u[2] = {l[t] * fexp2(m[t] - ref), 0.f};
#pragma unroll
        for (int i = 0; i < 16; ++i) u[i & 1] += fexp2(fmaf(S[i], scale2, -ref));
        l[t] = u[0] + u[1];
        m[t] = mx;
        if (end64) {
          snap_fold(cm[t], cl[t], m[t], l[t]);
          m[t] = -INFINITY, l[t] = 0.f;
        }
        if (end_run && !split) {
          const float mo = __shfl_xor(cm[t], 32), lo = __shfl_xor(cl[t], 32);
          snap_fold(cm[t], cl[t], mo, lo);
          const int r = r0 + 32 * t + lr;
          if (lh == 0 && r < rows) part[(size_t)(key0 / SNAP_CHUNK) * rows + r] = make_float2(cm[t], cl[t]);
          cm[t] = -INFINITY, cl[t] = 0.f;
        }
      }
    };
    // the next step's keys load while one is computed; after a run the wave skips those of the others
    // (loads past the span repeat rows of the prompt)
    auto next = [&](int key0) {
      key0 += 32;
      return key0 % run == 0 ? key0 + 3 * run : key0;
    };
    int key0 = a + run * wave;
    uint4 x[D / 16], y[D / 16];
    if (key0 < b) load(key0, x);
    while (key0 < b) {
      int to = next(key0);
      load(to, y);
      step(key0, x);
      if (to >= b) break;
      key0 = to;
      to = next(key0);
      load(to, x);
      step(key0, y);
      key0 = to;
    }
    if (!split) continue;
    __syncthreads();
#pragma unroll
    for (int t = 0; t < kTiles; ++t) s_part[2 * wave + lh][32 * t + lr] = make_float2(cm[t], cl[t]);
    __syncthreads();
    for (int r = threadIdx.x; r < ROWS && r0 + r < rows; r += NT) {
      float M[2] = {-INFINITY, -INFINITY}, L[2] = {0.f, 0.f};
#pragma unroll
      for (int v = 0; v < kParts; ++v) snap_fold(M[v & 1], L[v & 1], s_part[v][r].x, s_part[v][r].y);
      snap_fold(M[0], L[0], M[1], L[1]);
      part[(size_t)(a / SNAP_CHUNK) * rows + r0 + r] = make_float2(M[0], L[0]);
    }
  }
}

// Merge the window rows' partials, 32 rows a workgroup, every eighth chunk to a thread; chunk 0's entry
// of a row then holds (max, 1 / sum of exp2) over all its keys.
constexpr int kMergeRows = 32;
__global__ __launch_bounds__(NT) void k_snap_merge(const SeqDesc *__restrict__ seqs, const int32_t *__restrict__ list,
                                                   int Hkv, int lg) {
  constexpr int kSlices = NT / kMergeRows;
  __shared__ float2 s_part[kSlices][kMergeRows];
  const SeqDesc &sd = seqs[list[blockIdx.y]];
  const int n0 = sd.n0, rows = sd.w_eff << lg, h = blockIdx.x % Hkv, r0 = (int)blockIdx.x / Hkv * kMergeRows;
  const int np = (n0 + SNAP_CHUNK - 1) / SNAP_CHUNK;
  if (r0 >= rows || sd.T >= n0) return;
  const int rl = threadIdx.x % kMergeRows, sl = threadIdx.x / kMergeRows, r = min(r0 + rl, rows - 1);
  float2 *pr = reinterpret_cast<float2 *>(sd.aux1) + (size_t)h * np * rows + r;
  float m = -INFINITY, l = 0.f;
#pragma unroll 4
  for (int e = sl; e < np; e += kSlices) {
    const float *p = reinterpret_cast<const float *>(pr + (size_t)e * rows);
    snap_fold(m, l, gld(p), gld(p + 1));
  }
  s_part[sl][rl] = make_float2(m, l);
  __syncthreads();
  if (sl > 0) return;
  for (int v = 1; v < kSlices; ++v) snap_fold(m, l, s_part[v][rl].x, s_part[v][rl].y);
  if (r0 + rl < rows) pr[0] = make_float2(m, 1.f / l);
}

// Votes of a span's keys before the window: sum over the window rows of exp2(s - M_r) / L_r.  (Window
// keys get sums too, over rows that do not see them; they are not written.)
template <int D, int ROWS>
__global__ __launch_bounds__(NT) void k_snap_votes(const SeqDesc *__restrict__ seqs, const int32_t *__restrict__ list,
                                                   const uint16_t *__restrict__ qw, int Hq, int Hkv, int lg,
                                                   int span, float scale2) {
  constexpr int kTiles = ROWS / 32;
  __shared__ uint4 sq[ROWS][D / 8 + 1];
  __shared__ float2 sml[ROWS];  // (M, 1 / L) of the staged rows
  const SeqDesc &sd = seqs[list[blockIdx.y]];
  const int n0 = sd.n0, w = sd.w_eff, h = blockIdx.x % Hkv, a = (int)blockIdx.x / Hkv * span;
  if (a >= n0 - w || sd.T >= n0) return;
  const int nchunk = (n0 + SNAP_CHUNK - 1) / SNAP_CHUNK, b = min(a + span, n0 - w);
  const int lane = threadIdx.x & 63, lr = lane & 31, lh = lane >> 5;
  const int rows = w << lg;
  const float2 *part = reinterpret_cast<const float2 *>(sd.aux1) + (size_t)h * nchunk * rows;
  float *votes = reinterpret_cast<float *>(sd.aux0) + (size_t)h * n0;
  for (int r0 = 0; r0 < rows; r0 += ROWS) {
    if (r0 > 0) __syncthreads();
    stage_window<D, ROWS>(sq, qw, sd, h, lg, Hq, rows, r0);
    for (int t = threadIdx.x; t < ROWS; t += NT) {
      const float *ml = reinterpret_cast<const float *>(part + min(r0 + t, rows - 1));
      const float iL = gld(ml + 1);
      sml[t] = make_float2(gld(ml), r0 + t < rows ? iL : 0.f);
    }
    __syncthreads();
    snap_steps<D>(sd, h, a, b, [&](int key0, const uint4 (&ka)[D / 16]) {
      float acc[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
      for (int t = 0; t < kTiles; ++t) {
        if (r0 + 32 * t >= rows) continue;
        const f16v S = snap_logits<D>(ka, sq, 32 * t + lr, lh);
        const float2 mi = sml[32 * t + lr];
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = fmaf(fexp2(fmaf(S[i], scale2, -mi.x)), mi.y, acc[i]);
      }
      const float sum = half_wave_sums(acc);
      const int key = key0 + 8 * ((lr / 4) & 3) + 4 * lh + (lr & 3);
      if (lr < 16 && key < b) {
        if (r0 > 0) votes[key] += sum;
        else votes[key] = sum;
      }
    });
  }
}

// Max pooling of the candidates' votes (odd kernel `pool`, clipped to [0, n0 - w)) into
// order-preserving keys, one thread per candidate.
__global__ __launch_bounds__(NT) void k_snap_pool(const SeqDesc *__restrict__ seqs, const int32_t *__restrict__ list,
                                                  int Hkv) {
  const SeqDesc &sd = seqs[list[blockIdx.y]];
  const int n0 = sd.n0, ncand = n0 - sd.w_eff, h = blockIdx.x % Hkv, half = sd.pool / 2;
  const int j = (int)blockIdx.x / Hkv * NT + (int)threadIdx.x;
  if (j >= ncand || sd.T >= n0) return;
  const float *votes = reinterpret_cast<const float *>(sd.aux0) + (size_t)h * n0;
  float m = gld(votes + j);
  const int lo = max(0, j - half), hi = min(ncand - 1, j + half);
  for (int x = lo; x <= hi; ++x) m = fmaxf(m, gld(votes + x));
  gst(reinterpret_cast<uint32_t *>(sd.aux1) + (size_t)h * n0 + j, float_key(m));
}

// Keep the T - w highest pooled votes among the candidates (lower position on a tie) and the w
// window tokens: their positions into slots 0..kept-1 in ascending order, and the head's state.
__global__ __launch_bounds__(kTopkThreads) void k_snap_keep(const SeqDesc *__restrict__ seqs,
                                                            const int32_t *__restrict__ list, int32_t *state,
                                                            int Hkv) {
  __shared__ SelLds L;
  const int seq = list[blockIdx.y], h = blockIdx.x;
  const SeqDesc &sd = seqs[seq];
  const int n0 = sd.n0, w = sd.w_eff;
  const bool all = sd.T >= n0;
  const int ncand = n0 - w, want = sd.T - w;
  const int kept = all ? n0 : sd.T;
  int32_t *pos = reinterpret_cast<int32_t *>(sd.pos) + h * stride_slots(sd);
  if (all) {
    for (int j = threadIdx.x; j < n0; j += kTopkThreads) pos[j] = j;
  } else {
    if (want > 0) {
      const uint32_t *keys = reinterpret_cast<const uint32_t *>(sd.aux1) + (size_t)h * n0;
      select_keys<kTopkThreads, 32>(ncand, want, KeyRow{keys}, pos, L);
    }
    for (int i = threadIdx.x; i < w; i += kTopkThreads) pos[want + i] = ncand + i;
  }
  if (threadIdx.x == 0) {
    int32_t *st = state + ((size_t)seq * Hkv + h) * ST_WORDS;
    set_counts(st, kept, n0);
    st[ST_KEPT] = kept;
  }
}

// The kept rows and their channel-major key copy, a workgroup per kGatherSlots slots: rows are read
// and written 16 bytes a lane, the key tile transposed through LDS so that the copy is written 8
// slots (16 bytes) a lane.  (In the selecting workgroup, one per kv head, with 2-byte stores into the
// copy, selection and gather of 4 prompts of 32768 tokens took 935 us; 67 apart.)
template <int D>
__global__ __launch_bounds__(NT) void k_snap_gather(const SeqDesc *__restrict__ seqs, const int32_t *__restrict__ list,
                                                    int Hkv) {
  constexpr int U = D / 8, PER = kGatherSlots * U / NT, PITCH = D + 2;  // halves; odd in words
  __shared__ __attribute__((aligned(16))) uint16_t tile[kGatherSlots * PITCH];
  const SeqDesc &sd = seqs[list[blockIdx.y]];
  const int h = blockIdx.x % Hkv, s0 = (int)blockIdx.x / Hkv * kGatherSlots, kept = min(sd.T, sd.n0);
  if (s0 >= kept) return;
  const int32_t *pos = reinterpret_cast<const int32_t *>(sd.pos) + h * stride_slots(sd);
  const uint16_t *sk = reinterpret_cast<const uint16_t *>(sd.stage_k) + h * stride_stage(sd, D);
  const uint16_t *sv = reinterpret_cast<const uint16_t *>(sd.stage_v) + h * stride_stage(sd, D);
  uint16_t *dk = reinterpret_cast<uint16_t *>(sd.k) + h * stride_rows(sd, D);
  uint16_t *dvv = reinterpret_cast<uint16_t *>(sd.v) + h * stride_rows(sd, D);
  uint16_t *kcm = reinterpret_cast<uint16_t *>(sd.kcm) + h * stride_kcm(sd, D);
  const int u = threadIdx.x % U;
  int jj[PER];
  uint4 a[PER], b[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) jj[k] = gld(pos + min(s0 + (int)(threadIdx.x + k * NT) / U, kept - 1));
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    a[k] = gld16(sk + (size_t)jj[k] * D + 8 * u);
    b[k] = gld16(sv + (size_t)jj[k] * D + 8 * u);
  }
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int rr = (int)(threadIdx.x + k * NT) / U, slot = s0 + rr;
    uint32_t *t = reinterpret_cast<uint32_t *>(tile + rr * PITCH + 8 * u);
    t[0] = a[k].x;
    t[1] = a[k].y;
    t[2] = a[k].z;
    t[3] = a[k].w;
    if (slot >= kept) continue;
    *reinterpret_cast<uint4 *>(dk + (size_t)slot * D + 8 * u) = a[k];
    *reinterpret_cast<uint4 *>(dvv + (size_t)slot * D + 8 * u) = b[k];
  }
  __syncthreads();
  // 8 slots of one channel per item, the channels fastest; slots past the kept ones (below the row's
  // stride, a multiple of 8) repeat the last kept token until an append writes them
  for (int e = threadIdx.x; e < D * (kGatherSlots / 8); e += NT) {
    const int c = e % D, o = 8 * (e / D);
    if (s0 + o >= kept) break;
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      w[i] = (uint32_t)tile[(o + 2 * i) * PITCH + c] | (uint32_t)tile[(o + 2 * i + 1) * PITCH + c] << 16;
    *reinterpret_cast<uint4 *>(kcm + (size_t)c * sd.cstride + s0 + o) = make_uint4(w[0], w[1], w[2], w[3]);
  }
}

template <int D, int G>
hipError_t topk_impl(const Dev &dv, const Shape &sh, const uint16_t *q, int32_t *pos_out, int topk_max,
                     hipStream_t st, LaunchEv ev) {
  hipExtLaunchKernelGGL((k_topk<D, G>), dim3(sh.S * sh.Hkv), dim3(kTopkThreads), 0, st, ev.start, ev.stop, 0,
                        dv.seqs, dv.state, q, pos_out, topk_max, sh.Hkv);
  return hipGetLastError();
}

template <int D>
hipError_t h2o_prefill_impl(const Dev &dv, const Shape &sh, const SeqGroup &sg, const uint16_t *q, hipStream_t st) {
  const float scale2 = kLog2e / sqrtf((float)D);
  const int lg = __builtin_ctz((unsigned)sh.G);
  // grid x: kv heads (fastest) x the longest prompt's blocks; workgroups past a shorter prompt's end
  // leave at once
  const unsigned vblocks = (unsigned)((((int64_t)sg.longest << lg) + kScoreBlock - 1) / kScoreBlock);
  const unsigned kblocks = (sg.longest + kScoreBlock - 1) / kScoreBlock, H = sh.Hkv, n = sg.n;
  hipLaunchKernelGGL(k_h2o_rowstats<D>, dim3(H * vblocks, n), dim3(NT), 0, st, dv.seqs, sg.list, q, sh.Hq, sh.Hkv, lg,
                     scale2);
  hipLaunchKernelGGL(k_h2o_colsums<D>, dim3(H * kblocks * kScoreSegs, n), dim3(NT), 0, st, dv.seqs, sg.list, q, sh.Hq,
                     sh.Hkv, lg, scale2);
  hipLaunchKernelGGL(k_h2o_sum, dim3(H * ((sg.longest + NT - 1) / NT), n), dim3(NT), 0, st, dv.seqs, sg.list, sh.Hkv,
                     lg);
  hipLaunchKernelGGL(k_h2o_keep, dim3(H, n), dim3(kTopkThreads), 0, st, dv.seqs, sg.list, dv.state, sh.Hkv);
  hipLaunchKernelGGL(k_h2o_gather<D>, dim3(H * ((sg.max_kept + kGatherSlots - 1) / kGatherSlots), n), dim3(NT), 0, st,
                     dv.seqs, sg.list, sh.Hkv);
  return hipGetLastError();
}

template <int D>
hipError_t snap_prefill_impl(const Dev &dv, const Shape &sh, const SeqGroup &sg, const uint16_t *qw, hipStream_t st) {
  const float scale2 = kLog2e / sqrtf((float)D);
  const int lg = __builtin_ctz((unsigned)sh.G);
  const unsigned H = sh.Hkv, n = sg.n, rows = (unsigned)sg.max_vote_rows << lg;
  // Keys per workgroup: the span whose rounds of workgroups (two per CU) take the least time, a round
  // its keys and the set-up, as long as about 200 of them; for the row statistics one chunk or whole
  // chunks for each wave.  (4 prompts of 32768 tokens: one round of 2048 keys 78 and 62 us, row statistics
  // and votes, two of 1024 89 and 66, four waves a CU with 4096 80 and 82.)
  const auto best_span = [&](int step) {
    int span = SNAP_CHUNK;
    int64_t best = INT64_MAX;
    for (int s = SNAP_CHUNK; s <= 2048; s = s + step - s % step) {
      const int64_t wgs = (int64_t)H * n * ((sg.longest + s - 1) / s);
      const int64_t time = (wgs + 2 * kCus - 1) / (2 * kCus) * (s + 200);
      if (time < best) best = time, span = s;
    }
    return span;
  };
  const int sspan = best_span(4 * SNAP_CHUNK), vspan = best_span(SNAP_KEYS);
  const unsigned sspans = (sg.longest + sspan - 1) / sspan, vspans = (sg.longest + vspan - 1) / vspan;
  if (rows > 0) {  // some sequence keeps less than its prompt
    // all rows of 32-token windows of up to 4, or of 8 query heads, in LDS at once: K is read once a pass
    // (8 prompts of 6000-9000 tokens of 8 heads: 152 us with 128 rows and two passes over K, 137 with 256)
    hipLaunchKernelGGL((rows <= 128 ? k_snap_rowstats<D, 128> : k_snap_rowstats<D, 256>), dim3(H * sspans, n), dim3(NT),
                       0, st, dv.seqs, sg.list, qw, sh.Hq, sh.Hkv, lg, sspan, scale2);
    hipLaunchKernelGGL(k_snap_merge, dim3(H * ((rows + kMergeRows - 1) / kMergeRows), n), dim3(NT), 0, st, dv.seqs,
                       sg.list, sh.Hkv, lg);
    hipLaunchKernelGGL((rows <= 128 ? k_snap_votes<D, 128> : k_snap_votes<D, 256>), dim3(H * vspans, n), dim3(NT), 0,
                       st, dv.seqs, sg.list, qw, sh.Hq, sh.Hkv, lg, vspan, scale2);
    hipLaunchKernelGGL(k_snap_pool, dim3(H * ((sg.longest + NT - 1) / NT), n), dim3(NT), 0, st, dv.seqs, sg.list,
                       sh.Hkv);
  }
  hipLaunchKernelGGL(k_snap_keep, dim3(H, n), dim3(kTopkThreads), 0, st, dv.seqs, sg.list, dv.state, sh.Hkv);
  hipLaunchKernelGGL(k_snap_gather<D>, dim3(H * ((sg.max_kept + kGatherSlots - 1) / kGatherSlots), n), dim3(NT), 0, st,
                     dv.seqs, sg.list, sh.Hkv);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_topk(const Dev &dv, const Shape &sh, const uint16_t *q, int32_t *pos_out, int topk_max,
                       hipStream_t st, LaunchEv ev) {
  switch (sh.D * 16 + sh.G) {
    case 64 * 16 + 1: return topk_impl<64, 1>(dv, sh, q, pos_out, topk_max, st, ev);
    case 64 * 16 + 2: return topk_impl<64, 2>(dv, sh, q, pos_out, topk_max, st, ev);
    case 64 * 16 + 4: return topk_impl<64, 4>(dv, sh, q, pos_out, topk_max, st, ev);
    case 64 * 16 + 8: return topk_impl<64, 8>(dv, sh, q, pos_out, topk_max, st, ev);
    case 128 * 16 + 1: return topk_impl<128, 1>(dv, sh, q, pos_out, topk_max, st, ev);
    case 128 * 16 + 2: return topk_impl<128, 2>(dv, sh, q, pos_out, topk_max, st, ev);
    case 128 * 16 + 4: return topk_impl<128, 4>(dv, sh, q, pos_out, topk_max, st, ev);
    case 128 * 16 + 8: return topk_impl<128, 8>(dv, sh, q, pos_out, topk_max, st, ev);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_h2o_prefill(const Dev &dv, const Shape &sh, const SeqGroup &sg, const uint16_t *q_rows,
                              hipStream_t st) {
  return sh.D == 64 ? h2o_prefill_impl<64>(dv, sh, sg, q_rows, st) : h2o_prefill_impl<128>(dv, sh, sg, q_rows, st);
}

hipError_t launch_snap_prefill(const Dev &dv, const Shape &sh, const SeqGroup &sg, const uint16_t *q_window,
                               hipStream_t st) {
  return sh.D == 64 ? snap_prefill_impl<64>(dv, sh, sg, q_window, st) : snap_prefill_impl<128>(dv, sh, sg, q_window, st);
}

}  // namespace mkv
