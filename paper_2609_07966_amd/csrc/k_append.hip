// Append and quantize-on-append kernels: prompts, and the decode appends that have a launch of their
// own (what a method's append writes: append_dev.h).
#include "append_dev.h"
#include "select_dev.h"

namespace mkv {

namespace {

// A workgroup of D threads appends the token of (seq, h) and moves the pair's state on.
template <int D>
MKV_DEV void append_alone(const SeqDesc &sd, int32_t *st, int seq, int h, int Hkv, const uint16_t *__restrict__ k,
                          const uint16_t *__restrict__ v, const float *__restrict__ cbtab, AppendLds<D> &L) {
  const NewToken tok = load_token<D, D>(sd, st, seq, h, Hkv, k, v, cbtab, L);
  const int count = st[ST_COUNT], pos = st[ST_NEXT_POS];
  int victim;
  const int slot = append_slot(sd, h, count, &victim);
  if (append_pair<D, D>(sd, st, tok, h, count, pos, slot, victim, L) && threadIdx.x == 0)
    set_counts(st, count + (victim < 0 ? 1 : 0), pos + 1);
}

// One workgroup of D threads per (sequence, kv head).
template <int D>
__global__ __launch_bounds__(128) void k_append_decode(const SeqDesc *__restrict__ seqs, int32_t *state,
                                                      const uint16_t *__restrict__ k,
                                                      const uint16_t *__restrict__ v,
                                                      const float *__restrict__ cbtab, int Hkv) {
  __shared__ AppendLds<D> L;
  const int seq = blockIdx.x / Hkv, h = blockIdx.x % Hkv;
  append_alone<D>(seqs[seq], state + ((size_t)seq * Hkv + h) * ST_WORDS, seq, h, Hkv, k, v, cbtab, L);
}

// The selection of a pair with n tokens (the new one included, if there was room for it) from the keys
// src(j), and the pair's state after the step; count and pos are those before it, read by every thread
// before a barrier.
template <int NTH, int KR, typename Src>
MKV_DEV void rocket_select(const SeqDesc &sd, int32_t *st, int h, int n, bool room, int count, int pos, Src src,
                           SelLds &L) {
  const int k = sd.topk;
  int32_t *sel = reinterpret_cast<int32_t *>(sd.sel) + h * stride_sel(sd);
  if (k >= n) {
    for (int j = threadIdx.x; j < n; j += NTH) sel[j] = j;
  } else {
    select_keys<NTH, KR>(n, k, src, sel, L);
  }
  __syncthreads();  // every thread has read the state
  if (threadIdx.x == 0) {
    st[ST_SEL_COUNT] = min(k, n);
    if (room) set_counts(st, count + 1, pos + 1);
  }
}

// The decode step's first two launches when RocketKV sequences are present.
//
// k_append_score, workgroups of kScoreThreads threads over a work list (int4: seq, kv head,
// part, parts): part -1 appends the token of a non-RocketKV pair on its first D threads (the
// other waves leave at once; a barrier waits only for waves that have not ended).  A RocketKV pair
// has ceil(cap / kScoreTokens) parts: part 0 appends its token (rows, channel-major copy,
// position) and every part picks the channels and scores its kScoreTokens tokens, the new one
// from the key it holds in LDS.  The state of a RocketKV pair is left to the selecting launch.  Where
// every pair has one part (SELECT: caps up to kScoreTokens tokens), that workgroup selects from the
// keys it has in LDS and there is no selecting launch.
//
// k_rocket_select, one workgroup of kTopkThreads threads per RocketKV pair (int2: seq, kv head):
// the top-k of the scores, then the pair's state (count, next position, selection count).
template <int D, int G, bool SELECT>
__global__ __launch_bounds__(kScoreThreads) void k_append_score(const SeqDesc *__restrict__ seqs, int32_t *state,
                                                                const int4 *__restrict__ items,
                                                                const uint16_t *__restrict__ k,
                                                                const uint16_t *__restrict__ v,
                                                                const uint16_t *__restrict__ q,
                                                                const float *__restrict__ cbtab, int Hkv) {
  __shared__ union {
    AppendLds<D> a;
    ChanLds<D, kScoreThreads> c;
  } L;
  __shared__ SelLds s_sel;
  __shared__ uint32_t s_keys[SELECT ? kScoreTokens : 1];
  const int4 it = items[blockIdx.x];
  const int seq = it.x, h = it.y, part = it.z, c = threadIdx.x;
  const SeqDesc &sd = seqs[seq];
  int32_t *st = state + ((size_t)seq * Hkv + h) * ST_WORDS;
  if (part < 0) {
    if (c >= D) return;
    append_alone<D>(sd, st, seq, h, Hkv, k, v, cbtab, L.a);
    return;
  }
  // the query channels first: their address needs only the work item
  uint16_t qr[G];
  load_qcol<D, G>(q + ((size_t)seq * Hkv * G + h * G) * D, qr);
  const size_t at = ((size_t)seq * Hkv + h) * D + min(c, D - 1);
  const uint16_t kb = k[at], vb = part == 0 ? v[at] : (uint16_t)0;
  const int count = st[ST_COUNT], pos = st[ST_NEXT_POS];
  // a full region (reachable only by replaying a captured decode step past max_new_tokens) drops
  // the token, as the separate append does
  const bool room = count < sd.cap;
  if (room && c < D) {
    L.c.knew[c] = kb;
    if (part == 0) {
      (reinterpret_cast<uint16_t *>(sd.k) + h * stride_rows(sd, D))[(size_t)count * D + c] = kb;
      (reinterpret_cast<uint16_t *>(sd.v) + h * stride_rows(sd, D))[(size_t)count * D + c] = vb;
      (reinterpret_cast<uint16_t *>(sd.kcm) + h * stride_kcm(sd, D))[(size_t)c * sd.cstride + count] = kb;
      if (c == 0) (reinterpret_cast<int32_t *>(sd.pos) + h * stride_slots(sd))[count] = pos;
    }
  }
  const int n = room ? count + 1 : count;
  uint32_t *akeys = reinterpret_cast<uint32_t *>(sd.akeys) + h * stride_slots(sd);
  score_part<D, G>(sd, h, n, part, room, qr, L.c, [&](int j, uint32_t key) {
    if constexpr (SELECT) s_keys[j] = key;
    else gst(akeys + j, key);
  });
  if constexpr (SELECT) {
    __syncthreads();
    rocket_select<kScoreThreads, kScoreTokens / kScoreThreads>(
        sd, st, h, n, room, count, pos, LdsKeys{s_keys}, s_sel);
  }
}

template <int D>
__global__ __launch_bounds__(kTopkThreads) void k_rocket_select(const SeqDesc *__restrict__ seqs, int32_t *state,
                                                                const int2 *__restrict__ pairs, int Hkv) {
  __shared__ SelLds L;
  const int2 pr = pairs[blockIdx.x];
  const int seq = pr.x, h = pr.y;
  const SeqDesc &sd = seqs[seq];
  int32_t *st = state + ((size_t)seq * Hkv + h) * ST_WORDS;
  const int count = st[ST_COUNT], pos = st[ST_NEXT_POS];
  const bool room = count < sd.cap;
  const uint32_t *akeys = reinterpret_cast<const uint32_t *>(sd.akeys) + h * stride_slots(sd);
  rocket_select<kTopkThreads, kRegKeys>(
      sd, st, h, room ? count + 1 : count, room, count, pos, KeyRow{akeys}, L);
}

// ---- prefill: a group of a method's sequences in one launch per stage ----------------------------
// Grid: x = kv head (fastest) x blocks of the longest prompt, y = sequence (longest first);
// workgroups past a shorter prompt's end leave at once.  Launches per sequence left the chip idle
// between them: a 20-sequence batch of 100-700 tokens enqueued about 100 of them, most under 5 us.

// The state of (seq, h) after the append of an n0-token prompt; `count` tokens are held (0 until a
// prefill selection has chosen them).
MKV_DEV void write_prompt_state(int32_t *state, int seq, int h, int Hkv, int n0, int count) {
  int32_t *st = state + ((size_t)seq * Hkv + h) * ST_WORDS;
  set_counts(st, count, n0);
  st[ST_KEPT] = n0;
}

// Copy prompt rows [n0][Hkv][D] (input layout) into per-head rows: a sequence's cache (FP16) or its
// staging (H2O, RocketKV).
template <int D>
__global__ __launch_bounds__(256) void k_prefill_copy(const SeqDesc *__restrict__ seqs,
                                                      const int32_t *__restrict__ list, int32_t *state,
                                                      const uint16_t *__restrict__ k, const uint16_t *__restrict__ v,
                                                      int Hkv) {
  const int seq = list[blockIdx.y];
  const SeqDesc &sd = seqs[seq];
  const int n0 = sd.n0;
  const bool staged = sd.method != FP16;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;   // one 16-byte chunk
  const int64_t total = (int64_t)n0 * Hkv * (D / 8);
  if (i >= total) return;
  const int ch = (int)(i % (D / 8));
  const int h = (int)((i / (D / 8)) % Hkv);
  const int64_t t = i / ((D / 8) * Hkv);
  if (t == 0 && ch == 0) write_prompt_state(state, seq, h, Hkv, n0, staged ? 0 : n0);
  const int64_t first = (int64_t)sd.row0 * Hkv * (D / 8);
  const uint4 a = reinterpret_cast<const uint4 *>(k)[first + i];
  const uint4 b = reinterpret_cast<const uint4 *>(v)[first + i];
  const int64_t at = h * (staged ? stride_stage(sd, D) : stride_rows(sd, D)) + t * D + ch * 8;
  *reinterpret_cast<uint4 *>(reinterpret_cast<uint16_t *>(staged ? sd.stage_k : sd.k) + at) = a;
  *reinterpret_cast<uint4 *>(reinterpret_cast<uint16_t *>(staged ? sd.stage_v : sd.v) + at) = b;
}

// In the quantizing kernels lanes take 8 consecutive channels of a token (one 16-byte load), LT = D / 8
// lanes a token, so that reductions over a token's channels are 3 or 4 DPP steps for 4 or 8 tokens at
// once and codes pack within a lane.
constexpr int kQuantThreads = 256;
constexpr int kQuantTokens = 64;  // tokens per workgroup

template <int LT, typename Op>
MKV_DEV float lane_group_reduce(float x, Op op) {  // over aligned groups of LT (8 or 16) lanes
  x = op(x, dpp<0xB1>(x));
  x = op(x, dpp<0x4E>(x));
  x = op(x, dpp<0x141>(x));
  if constexpr (LT == 16) x = op(x, dpp<0x140>(x));
  return x;
}
template <int LT>
MKV_DEV int lane_group_sum(int x) {
  auto step = [](int v, auto ctrl) { return __builtin_amdgcn_update_dpp(0, v, decltype(ctrl)::value, 0xF, 0xF, false); };
  x += step(x, std::integral_constant<int, 0xB1>{});
  x += step(x, std::integral_constant<int, 0x4E>{});
  x += step(x, std::integral_constant<int, 0x141>{});
  if constexpr (LT == 16) x += step(x, std::integral_constant<int, 0x140>{});
  return x;
}
// Sum of x over the lower lanes of the group.
template <int LT>
MKV_DEV int lane_group_before(int x) {
  int inc = x;
#pragma unroll
  for (int o = 1; o < LT; o <<= 1) {
    const int y = __shfl_up(inc, o, LT);
    inc += (int)(threadIdx.x % LT) >= o ? y : 0;
  }
  return inc - x;
}

// ---- uniform 4-bit prompts ------------------------------------------------------------------------
// 6 prompts of 1.2-19 thousand tokens (8 kv heads x 128; 219 MB of K and V): 67 + 40 us, against
// 176 + 138 with launches per sequence, one 128-thread workgroup per 4-token value block and key blocks
// read twice at 2 bytes a lane.

// The clamped 4-bit code of x in a group of minimum mn.
MKV_DEV int uq_code(float x, float mn, float inv) {
  return (int)fminf(fmaxf(rintf(__fmul_rn(__fsub_rn(x, mn), inv)), 0.f), 15.f);
}

// Key blocks of 64 tokens, a workgroup each: per-channel (min, step) over the block's tokens (in the
// lane, across the wave's lane groups, then the waves), codes of a lane's 8 channels as one word of the
// token's row.  The last workgroup of a head copies the incomplete block's rows and writes the state.
template <int D>
__global__ __launch_bounds__(kQuantThreads) void k_uq_keys(const SeqDesc *__restrict__ seqs,
                                                           const int32_t *__restrict__ list, int32_t *state,
                                                           const uint16_t *__restrict__ k, int Hkv) {
  constexpr int LT = D / 8, NW = kQuantThreads / 64, TPI = kQuantThreads / LT, NI = kQuantTokens / TPI;
  __shared__ float2 s_mm[NW][D];
  const int seq = list[blockIdx.y];
  const SeqDesc &sd = seqs[seq];
  const int n0 = sd.n0, h = blockIdx.x % Hkv, blk = (int)blockIdx.x / Hkv, nfull = n0 / 64;
  if (blk > nfull) return;
  const int l = threadIdx.x % LT, tl = threadIdx.x / LT, wave = threadIdx.x >> 6;
  const uint16_t *kp = k + ((size_t)(sd.row0 + 64 * blk) * Hkv + h) * D + 8 * l;
  if (blk == nfull) {
    uint16_t *res = reinterpret_cast<uint16_t *>(sd.kres) + (size_t)h * 64 * D;
    for (int t = tl; t < n0 - 64 * nfull; t += TPI)
      *reinterpret_cast<uint4 *>(res + t * D + 8 * l) = gld16h(kp + (size_t)t * Hkv * D);
    if (threadIdx.x == 0) write_prompt_state(state, seq, h, Hkv, n0, n0);
    return;
  }
  uint4 w[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) w[i] = gld16h(kp + (size_t)(i * TPI + tl) * Hkv * D);
  float mn[8], mx[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    mn[e] = INFINITY;
    mx[e] = -INFINITY;
  }
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    float x[8];
    unpack8(w[i], x);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      mn[e] = fminf(mn[e], x[e]);
      mx[e] = fmaxf(mx[e], x[e]);
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) {
#pragma unroll
    for (int o = LT; o < 64; o <<= 1) {
      mn[e] = fminf(mn[e], __shfl_xor(mn[e], o));
      mx[e] = fmaxf(mx[e], __shfl_xor(mx[e], o));
    }
    if ((int)(threadIdx.x & 63) < LT) s_mm[wave][8 * l + e] = make_float2(mn[e], mx[e]);
  }
  __syncthreads();
  float inv[8];
  float2 *meta = reinterpret_cast<float2 *>(sd.kmeta) + h * stride_uq_kmeta(sd, D) + (size_t)blk * D;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    float2 m = s_mm[0][8 * l + e];
#pragma unroll
    for (int v = 1; v < NW; ++v) {
      const float2 o = s_mm[v][8 * l + e];
      m = make_float2(fminf(m.x, o.x), fmaxf(m.y, o.y));
    }
    const float r = __fsub_rn(m.y, m.x);
    mn[e] = m.x;
    inv[e] = r > 0.f ? __fdiv_rn(15.0f, r) : 0.f;
    if (tl == 0) meta[8 * l + e] = make_float2(m.x, __fdiv_rn(r, 15.0f));
  }
  uint8_t *rows = reinterpret_cast<uint8_t *>(sd.kc) + h * stride_codes(sd) + (size_t)blk * 64 * (D / 2);
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    float x[8];
    unpack8(w[i], x);
    uint32_t word = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) word |= (uint32_t)uq_code(x[e], mn[e], inv[e]) << (4 * e);
    gst(reinterpret_cast<uint32_t *>(rows + (size_t)(i * TPI + tl) * (D / 2)) + l, word);
  }
}

// Values: 64-channel groups (8 lanes), codes in 4-token blocks in the attention's operand order
// (uq_vbit): a lane's 8 channels are two words of each of two segments, the four tokens' nibbles OR-ed
// across their lanes.
template <int D>
__global__ __launch_bounds__(kQuantThreads) void k_uq_values(const SeqDesc *__restrict__ seqs,
                                                             const int32_t *__restrict__ list,
                                                             const uint16_t *__restrict__ v, int Hkv) {
  constexpr int LT = D / 8, TPI = kQuantThreads / LT, NI = kQuantTokens / TPI;
  const SeqDesc &sd = seqs[list[blockIdx.y]];
  const int n0 = sd.n0, h = blockIdx.x % Hkv, t0 = kQuantTokens * (int)(blockIdx.x / Hkv);
  if (t0 >= n0) return;
  const int l = threadIdx.x % LT, tl = threadIdx.x / LT, j = tl & 3, gr = l / 8;
  const uint16_t *vp = v + ((size_t)sd.row0 * Hkv + h) * D + 8 * l;
  uint8_t *blocks = reinterpret_cast<uint8_t *>(sd.vc) + h * stride_codes(sd);
  float2 *meta = reinterpret_cast<float2 *>(sd.vmeta) + h * stride_uq_vmeta(sd, D);
  uint4 nx = gld16h(vp + (size_t)min(t0 + tl, n0 - 1) * Hkv * D);
#pragma unroll 1
  for (int i = 0; i < NI; ++i) {
    const int t = t0 + i * TPI + tl;
    const uint4 w = nx;
    if (i + 1 < NI) nx = gld16h(vp + (size_t)min(t + TPI, n0 - 1) * Hkv * D);
    float x[8];
    unpack8(w, x);
    float mn = x[0], mx = x[0];
#pragma unroll
    for (int e = 1; e < 8; ++e) {
      mn = fminf(mn, x[e]);
      mx = fmaxf(mx, x[e]);
    }
    mn = lane_group_reduce<8>(mn, [](float a, float b) { return fminf(a, b); });
    mx = lane_group_reduce<8>(mx, [](float a, float b) { return fmaxf(a, b); });
    const float r = __fsub_rn(mx, mn);
    const float inv = r > 0.f ? __fdiv_rn(15.0f, r) : 0.f;
    // channels 8 l .. 8 l + 3 and + 4 .. + 7: segments 2 (l % 8) and + 1, words 2 gr and + 1 of each;
    // token j's nibble of channel parity b is 2 b + 4 (j % 2) + j / 2
    const int sh = 4 * (4 * (j & 1) + (j >> 1));
    uint32_t word[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t c0 = (uint32_t)uq_code(x[2 * q], mn, inv), c1 = (uint32_t)uq_code(x[2 * q + 1], mn, inv);
      word[q] = t < n0 ? (c0 | c1 << 8) << sh : 0u;
    }
    uint32_t mine = 0;  // lane group j stores word j
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      word[q] |= (uint32_t)__shfl_xor((int)word[q], LT);
      word[q] |= (uint32_t)__shfl_xor((int)word[q], 2 * LT);
      mine = j == q ? word[q] : mine;
    }
    if (t - j < n0)
      gst(reinterpret_cast<uint32_t *>(blocks + (size_t)(t - j) * sd.rowbytes) + (2 * (l % 8) + (j >> 1)) * (D / 32) +
              2 * gr + (j & 1),
          mine);
    if (t < n0 && l % 8 == 0) meta[(size_t)t * (D / 64) + gr] = make_float2(mn, __fdiv_rn(r, 15.0f));
  }
}

// ---- KVQ prompts ----------------------------------------------------------------------------------
// 8 prompts of 3000-6000 tokens (8 kv heads x 128), where launches per sequence, one workgroup per
// token (keys) or 4-token block (values) and 16 workgroups per calibration stood before: thresholds
// 1176 -> 39 us, key codes and outliers 364 -> 54, values 201 -> 57, scan 72 -> 5.  Reading K or V once
// takes 15 us here; the codes' compares bound the quantizing kernels, load latency the calibration.

// KVQ key thresholds: the n_o-th largest |k| (0-based) of every channel over the prompt, by a
// two-pass radix select on the 15-bit fp16 magnitude.  A workgroup takes 32 channels of one kv head;
// its waves read 16 tokens per load, kCalibBatch loads counted while the next are in flight, into one
// 256-bin histogram per channel by LDS atomics (in the second pass only keys of the selected digit);
// then a wave per channel finds its digit by a scan.  32 channels instead of 64 per workgroup give 256
// of them on 8 sequences, and 16 waves the loads in flight that one workgroup per CU needs: 8 prompts
// of 3000-6000 tokens 39 us, with 8 waves 58 (counting only the keys that may still matter: no gain).
constexpr int kCalibThreads = 1024;
constexpr int kCalibBatch = 2;
constexpr int kCalibChannels = 32;
template <int D>
__global__ __launch_bounds__(kCalibThreads) void k_kvq_calibrate(const SeqDesc *__restrict__ seqs,
                                                                 const int32_t *__restrict__ list,
                                                                 const uint16_t *__restrict__ k, int Hkv) {
  constexpr int NW = kCalibThreads / 64, LC = kCalibChannels / 8, TPL = 64 / LC;  // lanes a token, tokens a load
  __shared__ __attribute__((aligned(16))) uint32_t hist[kCalibChannels][260];
  __shared__ uint32_t s_sel[kCalibChannels], s_rem[kCalibChannels];
  const SeqDesc &sd = seqs[list[blockIdx.y]];
  const int n0 = sd.n0, h = blockIdx.x % Hkv, c0 = kCalibChannels * (int)(blockIdx.x / Hkv);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float2 *tau = reinterpret_cast<float2 *>(sd.kmeta) + (size_t)h * D + c0;
  const int want = sd.bp > 0 ? sd.n_o : 0;  // 0-based rank from the top
  if (want >= n0) {  // fewer prompt tokens than the rank: no threshold (every key is an inlier)
    if (threadIdx.x < kCalibChannels) tau[threadIdx.x] = make_float2(0.f, 0.f);
    return;
  }
  if (threadIdx.x < kCalibChannels) s_rem[threadIdx.x] = (uint32_t)want + 1;  // 1-based rank
  const int cl = 8 * (lane % LC);  // this lane's first channel of the workgroup's
  const uint16_t *kc = k + ((size_t)sd.row0 * Hkv + h) * D + c0 + cl;
  const size_t pitch = (size_t)Hkv * D;
  constexpr int kStep = NW * TPL;  // tokens a load of every wave takes
  auto load = [&](int t, uint4 (&w)[kCalibBatch]) {
#pragma unroll
    for (int b = 0; b < kCalibBatch; ++b) w[b] = gld16h(kc + (size_t)min(t + b * kStep, n0 - 1) * pitch);
  };
  const int tl = wave * TPL + lane / LC;
  for (int pass = 0; pass < 2; ++pass) {
    uint4 x[kCalibBatch], y[kCalibBatch];
    load(tl, x);
    for (int e = threadIdx.x; e < kCalibChannels * 260; e += kCalibThreads) (&hist[0][0])[e] = 0u;
    __syncthreads();
    uint32_t sel[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) sel[e] = pass == 0 ? 0u : s_sel[cl + e];
    auto count = [&](int t, const uint4 (&w)[kCalibBatch]) {
#pragma unroll
      for (int b = 0; b < kCalibBatch; ++b) {
        if (t + b * kStep >= n0) break;
        const uint32_t ww[4] = {w[b].x, w[b].y, w[b].z, w[b].w};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const uint32_t key = (ww[e / 2] >> (16 * (e & 1))) & 0x7FFFu;
          if (pass == 0) atomicAdd(&hist[cl + e][key >> 8], 1u);
          else if ((key >> 8) == sel[e]) atomicAdd(&hist[cl + e][key & 255u], 1u);
        }
      }
    };
    for (int t = tl; t - tl < n0; t += 2 * kCalibBatch * kStep) {
      load(t + kCalibBatch * kStep, y);
      count(t, x);
      load(t + 2 * kCalibBatch * kStep, x);
      count(t + kCalibBatch * kStep, y);
    }
    __syncthreads();
    for (int c = wave; c < kCalibChannels; c += NW) {
      // lane l owns digits 255 - 4l .. 252 - 4l, so the scan over lanes counts the larger digits
      const uint4 h4 = *reinterpret_cast<const uint4 *>(&hist[c][252 - 4 * lane]);
      const int cnt[4] = {(int)h4.w, (int)h4.z, (int)h4.y, (int)h4.x};
      const int rem = (int)s_rem[c], tot = cnt[0] + cnt[1] + cnt[2] + cnt[3];
      int above = wave_incl_scan(tot) - tot;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (above < rem && rem <= above + cnt[i]) {  // in exactly one lane
          const uint32_t dg = 255 - (4 * lane + i);
          if (pass == 0) {
            s_sel[c] = dg;
            s_rem[c] = (uint32_t)(rem - above);
          } else {
            const float t = h2f((s_sel[c] << 8) | dg);
            tau[c] = make_float2(t, t > 0.f ? __fdiv_rn(1.0f, t) : 0.f);
          }
        }
        above += cnt[i];
      }
    }
    __syncthreads();
  }
}

// A lane's 8 key codes are 8 * BITS consecutive bits of its token's packed row (see packed_word).
template <int BITS>
MKV_DEV void store_key_codes(const int (&code)[8], uint8_t *row, int l) {
  uint32_t v = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e) v |= (uint32_t)code[e] << (BITS * e);
  if constexpr (BITS == 4) {
    gst(reinterpret_cast<uint32_t *>(row) + l, v);
  } else if constexpr (BITS == 2) {
    gst(reinterpret_cast<uint16_t *>(row) + l, (uint16_t)v);
  } else {
    // four lanes' 24-bit pieces make three words: word i takes piece i from bit 8 i up and the foot of
    // piece i + 1
    const uint32_t nx = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xF9, 0xF, 0xF, false);  // quad_perm [1,2,3,3]
    const int i = l & 3;
    if (i < 3) gst(reinterpret_cast<uint32_t *>(row) + 3 * (l >> 2) + i, (v >> (8 * i)) | (nx << (24 - 8 * i)));
  }
}

// A lane's 8 channels of key thresholds, as kvq_key_tau gives them.
MKV_DEV void load_tau8(const SeqDesc &sd, int h, int c, int D, float (&tau)[8], float (&inv)[8]) {
  const uint32_t *p = reinterpret_cast<const uint32_t *>(sd.kmeta) + 2 * ((size_t)h * D + c);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint4 u = gld16(p + 4 * e);
    tau[2 * e] = __builtin_bit_cast(float, u.x);
    inv[2 * e] = __builtin_bit_cast(float, u.y);
    tau[2 * e + 1] = __builtin_bit_cast(float, u.z);
    inv[2 * e + 1] = __builtin_bit_cast(float, u.w);
  }
}

// KVQ prompt keys: codes, and each token's outlier count into krow[t + 1].
template <int D>
__global__ __launch_bounds__(kQuantThreads) void k_kvq_keys(const SeqDesc *__restrict__ seqs,
                                                          const int32_t *__restrict__ list,
                                                          const uint16_t *__restrict__ k,
                                                          const float *__restrict__ cbtab, int Hkv) {
  constexpr int LT = D / 8, TPW = 64 / LT, TPI = TPW * kQuantThreads / 64, NI = kQuantTokens / TPI;
  const SeqDesc &sd = seqs[list[blockIdx.y]];
  const int n0 = sd.n0, h = blockIdx.x % Hkv, t0 = kQuantTokens * (int)(blockIdx.x / Hkv);
  if (t0 >= n0) return;
  const int l = threadIdx.x % LT, tl = threadIdx.x / LT;
  const uint16_t *kp = k + ((size_t)sd.row0 * Hkv + h) * D + 8 * l;
  uint4 nx = gld16h(kp + (size_t)min(t0 + tl, n0 - 1) * Hkv * D);
  float tau[8], inv[8];
  load_tau8(sd, h, 8 * l, D, tau, inv);
  const bool outliers = sd.bp > 0;
  uint8_t *rows = reinterpret_cast<uint8_t *>(sd.kc) + h * stride_codes(sd);
  uint32_t *krow = reinterpret_cast<uint32_t *>(sd.krow) + h * stride_krow(sd);
  auto run = [&](auto bits_tag) {
    constexpr int BITS = decltype(bits_tag)::value, NC = 1 << BITS;
    const float *mid = cbtab + cb_offset(BITS) + 2 * NC;
#pragma unroll 1
    for (int i = 0; i < NI; ++i) {
      const int t = t0 + i * TPI + tl;
      const uint4 w = nx;
      if (i + 1 < NI) nx = gld16h(kp + (size_t)min(t + TPI, n0 - 1) * Hkv * D);
      float x[8];
      unpack8(w, x);
      int code[8], n = 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        code[e] = code_from_mid(__fmul_rn(x[e], inv[e]), mid, NC - 1);
        n += outliers && fabsf(x[e]) > tau[e] ? 1 : 0;
      }
      n = lane_group_sum<LT>(n);
      if (t < n0) {
        store_key_codes<BITS>(code, rows + (size_t)t * sd.rowbytes, l);
        if (l == 0) gst(krow + t + 1, (uint32_t)n);
      }
    }
  };
  if (sd.bits == 4) run(std::integral_constant<int, 4>{});
  else if (sd.bits == 3) run(std::integral_constant<int, 3>{});
  else run(std::integral_constant<int, 2>{});
}

// In-place inclusive scan of krow[1..n0] (per-token outlier counts) per kv head, 4 tokens a thread;
// and the head's state after the prompt.
constexpr int kScanThreads = 1024;
__global__ __launch_bounds__(kScanThreads) void k_kvq_scan(const SeqDesc *__restrict__ seqs,
                                                           const int32_t *__restrict__ list, int32_t *state,
                                                           int Hkv) {
  __shared__ int s_tmp[kScanThreads / 64];
  const int seq = list[blockIdx.y], h = blockIdx.x;
  const SeqDesc &sd = seqs[seq];
  const int n0 = sd.n0;
  uint32_t *krow = reinterpret_cast<uint32_t *>(sd.krow) + h * stride_krow(sd);
  int run = 0;
  for (int a = 4 * (int)threadIdx.x; a - 4 * (int)threadIdx.x < n0; a += 4 * kScanThreads) {
    int x[4], sum = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[i] = a + i < n0 ? (int)gld(krow + a + i + 1) : 0;
      sum += x[i];
    }
    int total;
    int pre = run + block_exclusive_scan<kScanThreads>(sum, s_tmp, &total);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      pre += x[i];
      if (a + i < n0) gst(krow + a + i + 1, (uint32_t)pre);
    }
    run += total;
  }
  if (threadIdx.x == 0) {
    krow[0] = 0;
    write_prompt_state(state, seq, h, Hkv, n0, n0);
    state[((size_t)seq * Hkv + h) * ST_WORDS + ST_KOUT_FILL] = run;
  }
}

// KVQ prompt keys: the outlier entries at their CSR offsets, ascending channels; codes come from the
// rows that k_kvq_keys wrote.
template <int D>
__global__ __launch_bounds__(kQuantThreads) void k_kvq_outliers(const SeqDesc *__restrict__ seqs,
                                                              const int32_t *__restrict__ list,
                                                              const uint16_t *__restrict__ k, int Hkv) {
  constexpr int LT = D / 8, TPW = 64 / LT, TPI = TPW * kQuantThreads / 64, NI = kQuantTokens / TPI;
  const SeqDesc &sd = seqs[list[blockIdx.y]];
  const int n0 = sd.n0, h = blockIdx.x % Hkv, t0 = kQuantTokens * (int)(blockIdx.x / Hkv);
  if (t0 >= n0 || sd.bp <= 0) return;
  const int l = threadIdx.x % LT, tl = threadIdx.x / LT;
  const uint16_t *kp = k + ((size_t)sd.row0 * Hkv + h) * D + 8 * l;
  const uint32_t *krow = reinterpret_cast<const uint32_t *>(sd.krow) + h * stride_krow(sd);
  uint32_t *ko = reinterpret_cast<uint32_t *>(sd.kout) + h * stride_kout(sd);
  uint4 w[NI];
  uint32_t at[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int t = min(t0 + i * TPI + tl, n0 - 1);
    w[i] = gld16h(kp + (size_t)t * Hkv * D);
    at[i] = gld(krow + t);
  }
  float tau[8], inv[8];  // (inv unused)
  load_tau8(sd, h, 8 * l, D, tau, inv);
  const int bits = sd.bits;
  const uint8_t *rows = reinterpret_cast<const uint8_t *>(sd.kc) + h * stride_codes(sd);
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int t = t0 + i * TPI + tl;
    float x[8];
    unpack8(w[i], x);
    uint32_t m = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) m |= fabsf(x[e]) > tau[e] ? 1u << e : 0u;
    m = t < n0 ? m : 0u;
    uint32_t *dst = ko + at[i] + lane_group_before<LT>(__popc(m));
    // the 8 codes of this lane are the 8 * bits bits at byte l * bits of the token's row
    for (; m != 0; m &= m - 1) {
      const int e = __builtin_ctz(m), bit = bits * e;
      const uint8_t *c = rows + (size_t)t * sd.rowbytes + l * bits;
      const uint32_t lo = gld(c + (bit >> 3)), hi = gld(c + min((bit >> 3) + 1, bits - 1));
      const int code = (int)((lo | hi << 8) >> (bit & 7)) & ((1 << bits) - 1);
      gst(dst++, outlier_entry(gld(kp + (size_t)t * Hkv * D + e), t, code, 8 * l + e));
    }
  }
}

// KVQ prompt values: per-token scale (the n_ov-th largest |v|, 0-based), codes in 4-token blocks, and
// the outliers, whose slots go by ascending channel.  A wave holds whole 4-token blocks: the four
// tokens' codes of a lane's 8 channels are BITS words of the block, OR-ed across their lanes.
template <int D>
__global__ __launch_bounds__(kQuantThreads) void k_kvq_values(const SeqDesc *__restrict__ seqs,
                                                            const int32_t *__restrict__ list,
                                                            const uint16_t *__restrict__ v,
                                                            const float *__restrict__ cbtab, int Hkv) {
  constexpr int LT = D / 8, TPW = 64 / LT, TPI = TPW * kQuantThreads / 64, NI = kQuantTokens / TPI;
  const SeqDesc &sd = seqs[list[blockIdx.y]];
  const int n0 = sd.n0, h = blockIdx.x % Hkv, t0 = kQuantTokens * (int)(blockIdx.x / Hkv);
  if (t0 >= n0) return;
  const int l = threadIdx.x % LT, tl = threadIdx.x / LT, j = tl & 3;
  const uint16_t *vp = v + ((size_t)sd.row0 * Hkv + h) * D + 8 * l;
  uint4 nx = gld16h(vp + (size_t)min(t0 + tl, n0 - 1) * Hkv * D);
  const int nov = sd.bp > 0 ? sd.n_ov : 0, slots = sd.nov_slots;
  const bool outliers = sd.bp > 0;
  uint8_t *blocks = reinterpret_cast<uint8_t *>(sd.vc) + h * stride_codes(sd);
  float *scale = reinterpret_cast<float *>(sd.vmeta) + h * stride_slots(sd);
  uint32_t *vo = reinterpret_cast<uint32_t *>(sd.vout) + h * stride_vout(sd);
  uint32_t *vd = reinterpret_cast<uint32_t *>(sd.vdel) + h * stride_vout(sd);
  auto run = [&](auto bits_tag) {
    constexpr int BITS = decltype(bits_tag)::value, NC = 1 << BITS;
    const float *cb = cbtab + cb_offset(BITS) + NC, *mid = cbtab + cb_offset(BITS) + 2 * NC + (NC - 1);
#pragma unroll 1
    for (int i = 0; i < NI; ++i) {
      const int t = t0 + i * TPI + tl;
      const uint4 w = nx;
      if (i + 1 < NI) nx = gld16h(vp + (size_t)min(t + TPI, n0 - 1) * Hkv * D);
      const uint32_t valid = t < n0 ? ~0u : 0u;
      float x[8], ax[8];
      unpack8(w, x);
#pragma unroll
      for (int e = 0; e < 8; ++e) ax[e] = fabsf(x[e]);
      // the largest values one after another, with their multiplicities, until nov of them lie above
      float s = 0.f;
      int above = 0;
      bool found = false;
      for (int r = 0; r <= nov && __any(!found); ++r) {
        float m = -1.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) m = fmaxf(m, r == 0 || ax[e] < s ? ax[e] : -1.f);
        m = lane_group_reduce<LT>(m, [](float a, float b) { return fmaxf(a, b); });
        int c = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) c += ax[e] == m ? 1 : 0;
        c = lane_group_sum<LT>(c);
        if (!found) {
          s = m;
          above += c;
          found = above > nov;
        }
      }
      const float inv = s > 0.f ? __fdiv_rn(1.0f, s) : 0.f;
      int code[8];
      uint32_t word[BITS] = {}, om = 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        code[e] = code_from_mid(__fmul_rn(x[e], inv), mid, NC - 1);
        om |= ax[e] > s ? 1u << e : 0u;
        const uint32_t f = (uint32_t)code[e] << (BITS * j);
        const int bit = 4 * BITS * e, sh = bit & 31;
        word[bit >> 5] |= f << sh;
        if (sh + 4 * BITS > 32) word[(bit >> 5) + 1] |= f >> (32 - sh);
      }
      if (!outliers) om = 0;
      om &= valid;
      uint32_t mine = 0;  // lane group j stores word j of each lane's BITS words
#pragma unroll
      for (int b = 0; b < BITS; ++b) {
        word[b] &= valid;
        word[b] |= (uint32_t)__shfl_xor((int)word[b], LT);
        word[b] |= (uint32_t)__shfl_xor((int)word[b], 2 * LT);
        mine = j == b ? word[b] : mine;
      }
      if (j < BITS && t - j < n0)
        gst(reinterpret_cast<uint32_t *>(blocks + (size_t)(t - j) * sd.rowbytes) + l * BITS + j, mine);
      const int before = lane_group_before<LT>(__popc(om)), total = lane_group_sum<LT>(__popc(om));
      if (t < n0) {
        if (l == 0) gst(scale + t, s);
        if (om) {
          // (values and codes re-read, or counted again, for the few outliers only)
          int r = before;
          for (uint32_t m = om; m != 0; m &= m - 1, ++r) {
            const int e = __builtin_ctz(m);
            if (r >= slots) break;
            const uint32_t bits = gld(vp + (size_t)t * Hkv * D + e);
            const float y = h2f(bits);
            const int c = code_from_mid(__fmul_rn(y, inv), mid, NC - 1);
            gst(vo + (size_t)r * sd.cap + t, outlier_entry(bits, t, c, 8 * l + e));
            // the attention's form: the outlier minus the value its code stands for, and the channel
            gst(vd + (size_t)r * sd.cap + t, vdel_pack(__fsub_rn(y, __fmul_rn(s, gld(cb + c))), 8 * l + e));
          }
        }
        for (int r = total + l; r < slots; r += LT) {
          gst(vo + (size_t)r * sd.cap + t, kNoOutlier);
          gst(vd + (size_t)r * sd.cap + t, 0u);
        }
      }
    }
  };
  if (sd.bits == 4) run(std::integral_constant<int, 4>{});
  else if (sd.bits == 3) run(std::integral_constant<int, 3>{});
  else run(std::integral_constant<int, 2>{});
}

template <int D>
hipError_t append_decode_impl(const Dev &dv, const Shape &sh, const uint16_t *k, const uint16_t *v,
                              hipStream_t st, LaunchEv ev) {
  hipExtLaunchKernelGGL(k_append_decode<D>, dim3(sh.S * sh.Hkv), dim3(D), 0, st, ev.start, ev.stop, 0, dv.seqs,
                        dv.state, k, v, dv.cbtab, sh.Hkv);
  return hipGetLastError();
}

template <int D, int G>
hipError_t append_select_impl(const Dev &dv, const Shape &sh, const uint16_t *k, const uint16_t *v,
                              const uint16_t *q, hipStream_t st, LaunchEv ev_score, LaunchEv ev_select) {
  // one item per (sequence, kv head): every RocketKV pair has one part, which selects (unless the
  // selections are timed).  Per step, 8 kv heads, keeping an eighth: one sequence of 300 tokens 19.9 us
  // with the second launch, 16.7 without; 48 of 500 tokens 25.5 and 20.7.  Pairs of more parts would
  // wait for all of them, or score over 1024 tokens on one CU.
  const bool fused = dv.n_prep == sh.S * sh.Hkv && ev_select.start == nullptr;
  auto kernel = fused ? k_append_score<D, G, true> : k_append_score<D, G, false>;
  hipExtLaunchKernelGGL(kernel, dim3(dv.n_prep), dim3(kScoreThreads), 0, st, ev_score.start, ev_score.stop, 0,
                        dv.seqs, dv.state, dv.prep, k, v, q, dv.cbtab, sh.Hkv);
  if (fused) return hipGetLastError();
  hipExtLaunchKernelGGL(k_rocket_select<D>, dim3(dv.n_rk_pairs), dim3(kTopkThreads), 0, st, ev_select.start,
                        ev_select.stop, 0, dv.seqs, dv.state, dv.rk_pairs, sh.Hkv);
  return hipGetLastError();
}

template <int D>
hipError_t prefill_impl(const Dev &dv, const Shape &sh, const SeqGroup &sg, const uint16_t *k, const uint16_t *v,
                        hipStream_t st) {
  const int Hkv = sh.Hkv;
  const unsigned H = Hkv, n = sg.n, blocks = (sg.longest + kQuantTokens - 1) / kQuantTokens;
  switch (sg.method) {
    case FP16:
    case H2O:
    case ROCKET: {
      const int64_t chunks = (int64_t)sg.longest * Hkv * (D / 8);
      hipLaunchKernelGGL(k_prefill_copy<D>, dim3((unsigned)((chunks + 255) / 256), n), dim3(256), 0, st, dv.seqs,
                         sg.list, dv.state, k, v, Hkv);
      break;
    }
    case UQ:
      hipLaunchKernelGGL(k_uq_values<D>, dim3(H * blocks, n), dim3(kQuantThreads), 0, st, dv.seqs, sg.list, v, Hkv);
      hipLaunchKernelGGL(k_uq_keys<D>, dim3(H * (sg.longest / 64 + 1), n), dim3(kQuantThreads), 0, st, dv.seqs,
                         sg.list, dv.state, k, Hkv);
      break;
    case KVQ:
      hipLaunchKernelGGL(k_kvq_calibrate<D>, dim3(H * (D / kCalibChannels), n), dim3(kCalibThreads), 0, st, dv.seqs,
                         sg.list, k, Hkv);
      hipLaunchKernelGGL(k_kvq_keys<D>, dim3(H * blocks, n), dim3(kQuantThreads), 0, st, dv.seqs, sg.list, k, dv.cbtab,
                         Hkv);
      hipLaunchKernelGGL(k_kvq_scan, dim3(H, n), dim3(kScanThreads), 0, st, dv.seqs, sg.list, dv.state, Hkv);
      hipLaunchKernelGGL(k_kvq_outliers<D>, dim3(H * blocks, n), dim3(kQuantThreads), 0, st, dv.seqs, sg.list, k, Hkv);
      hipLaunchKernelGGL(k_kvq_values<D>, dim3(H * blocks, n), dim3(kQuantThreads), 0, st, dv.seqs, sg.list, v,
                         dv.cbtab, Hkv);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_append_decode(const Dev &dv, const Shape &sh, const uint16_t *k, const uint16_t *v,
                                hipStream_t st, LaunchEv ev) {
  return sh.D == 64 ? append_decode_impl<64>(dv, sh, k, v, st, ev) : append_decode_impl<128>(dv, sh, k, v, st, ev);
}

hipError_t launch_append_select(const Dev &dv, const Shape &sh, const uint16_t *k, const uint16_t *v,
                                const uint16_t *q, hipStream_t st, LaunchEv ev_score, LaunchEv ev_select) {
  switch (sh.D * 16 + sh.G) {
    case 64 * 16 + 1: return append_select_impl<64, 1>(dv, sh, k, v, q, st, ev_score, ev_select);
    case 64 * 16 + 2: return append_select_impl<64, 2>(dv, sh, k, v, q, st, ev_score, ev_select);
    case 64 * 16 + 4: return append_select_impl<64, 4>(dv, sh, k, v, q, st, ev_score, ev_select);
    case 64 * 16 + 8: return append_select_impl<64, 8>(dv, sh, k, v, q, st, ev_score, ev_select);
    case 128 * 16 + 1: return append_select_impl<128, 1>(dv, sh, k, v, q, st, ev_score, ev_select);
    case 128 * 16 + 2: return append_select_impl<128, 2>(dv, sh, k, v, q, st, ev_score, ev_select);
    case 128 * 16 + 4: return append_select_impl<128, 4>(dv, sh, k, v, q, st, ev_score, ev_select);
    case 128 * 16 + 8: return append_select_impl<128, 8>(dv, sh, k, v, q, st, ev_score, ev_select);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_prefill(const Dev &dv, const Shape &sh, const SeqGroup &sg, const uint16_t *k, const uint16_t *v,
                          hipStream_t st) {
  return sh.D == 64 ? prefill_impl<64>(dv, sh, sg, k, v, st) : prefill_impl<128>(dv, sh, sg, k, v, st);
}

}  // namespace mkv
