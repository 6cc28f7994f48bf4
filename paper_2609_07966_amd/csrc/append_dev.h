// The decode append, device side: one token of one (sequence, kv head) written into its cache by a
// workgroup, shared by the append launches and by the attention launch of a decode step, whose tile that
// owns the token's slot appends it first.
//
// Every method first writes the new token's key and value into its cache (MetaKV Section 2.1):
// plain fp16 rows (FP16, H2O, RocketKV), uniform 4-bit group codes, or KVQuant-style codes with
// per-channel key thresholds calibrated on the prompt and fp16 outliers.  The quantizer steps are
// written with explicit round-to-nearest float32 operations (__fmul_rn, __fsub_rn, __fdiv_rn)
// so that codes are reproducible bit for bit.
//
// Workgroups of NT >= D threads: thread c < D takes channel c, the others only keep the barriers.
#pragma once

#include "kernels_common.h"

namespace mkv {

namespace {

// ---- shared quantizer pieces -----------------------------------------------------------------

MKV_DEV int code_from_mid(float xhat, const float *mid, int nmid) {
  int c = 0;
  for (int i = 0; i < nmid; ++i) c += (xhat > mid[i]) ? 1 : 0;
  return c;
}

// Outlier entry of token slot t (layout in outlier_pack): the (clamped) code stays in the entry.
MKV_DEV uint32_t outlier_entry(uint32_t bits16, int t, int code, int ch) {
  return outlier_pack(bits16 & 0xFFFFu, t, code, ch);
}

// Word w of a packed code row: code i sits at bits [bits*i, bits*i + bits) of the row (bit 0 =
// least significant bit of byte 0), so two consecutive codes form one 2*bits-bit field.
MKV_DEV uint32_t packed_word(const uint8_t *codes, int n, int bits, int w) {
  uint32_t word = 0;
  const int lo = 32 * w;
  const int first = max(0, lo / bits - 1), last = min(n, (lo + 32) / bits + 1);
  for (int i = first; i < last; ++i) {
    const int off = bits * i - lo;
    const uint32_t code = codes[i];
    if (off >= 0 && off < 32) word |= code << off;
    else if (off < 0 && off > -bits) word |= code >> (-off);
  }
  return word;
}

// Pack one code per thread (thread c = channel c of threads 0..D-1) into a key row (see
// packed_word).  `s_code` is D bytes of LDS.
template <int D>
MKV_DEV void pack_row(int code, int bits, uint8_t *s_code, uint8_t *row) {
  const int c = threadIdx.x;
  if (c < D) s_code[c] = (uint8_t)code;
  __syncthreads();
  const int words = D * bits / 32;
  if (c < words) gst(reinterpret_cast<uint32_t *>(row) + c, packed_word(s_code, D, bits, c));
  __syncthreads();
}

// Value codes are stored in blocks of 4 tokens: code (channel c, token j) at bit bits*(4c + j)
// of the block, so the 4 tokens of a channel form two 2*bits-bit fields.  OR one code per thread
// into the LDS copy `s_blk` of a block.
MKV_DEV void or_quad_code(uint32_t *s_blk, int c, int j, int code, int bits) {
  const int bit = bits * (4 * c + j);
  atomicOr(&s_blk[bit >> 5], (uint32_t)code << (bit & 31));
  const int spill = (bit & 31) + bits - 32;
  if (spill > 0) atomicOr(&s_blk[(bit >> 5) + 1], (uint32_t)code >> (bits - spill));
}

// Rank among the flagged threads 0..D-1 (of up to 256; the others are not flagged).
template <int D>
MKV_DEV int flag_rank(bool f, int *s_tmp, int *total) {
  const uint64_t m = __ballot(f);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int before = __popcll(m & ((lane == 0) ? 0ull : (~0ull >> (64 - lane))));
  if (lane == 0) s_tmp[w] = __popcll(m);
  __syncthreads();
  int base = 0, tot = 0;
  for (int i = 0; i < D / 64; ++i) {
    if (i < w) base += s_tmp[i];
    tot += s_tmp[i];
  }
  __syncthreads();
  *total = tot;
  return base + before;
}

// KVQ value of one token: per-token scale = n_ov-th largest |v| (0-based), outliers (written),
// and this thread's code (returned; the caller places it in the token's 4-token block).
template <int D>
MKV_DEV int kvq_value_token(const SeqDesc &sd, int h, int t, uint32_t vbits, const float *cbtab,
                            float *s_abs, float *s_scale, int *s_tmp) {
  const int c = threadIdx.x;
  const bool act = c < D;
  const float x = h2f(vbits);
  const float ax = fabsf(x);
  const int nov = sd.bp > 0 ? sd.n_ov : 0;
  float s;
  if (nov <= 1) {
    // the largest |v| or, for n_ov = 1, the largest after one occurrence of it is set aside:
    // wave maxima with their multiplicities, then (maximum unique) the largest value below it
    constexpr int NWV = D / 64;
    const int lane = c & 63, w = c >> 6;
    const float wm = wave_max(ax);
    const int wc = __popcll(__ballot(ax == wm));
    if (lane == 0) {
      s_abs[w] = wm;
      s_tmp[w] = wc;
    }
    __syncthreads();
    float m1 = s_abs[0];
#pragma unroll
    for (int i = 1; i < NWV; ++i) m1 = fmaxf(m1, s_abs[i]);
    int cnt = 0;
#pragma unroll
    for (int i = 0; i < NWV; ++i) cnt += s_abs[i] == m1 ? s_tmp[i] : 0;
    s = m1;
    if (nov == 1 && cnt < 2) {  // block-uniform
      __syncthreads();
      const float wm2 = wave_max(ax < m1 ? ax : -1.f);
      if (lane == 0) s_abs[w] = wm2;
      __syncthreads();
      s = s_abs[0];
#pragma unroll
      for (int i = 1; i < NWV; ++i) s = fmaxf(s, s_abs[i]);
    }
    __syncthreads();  // s_abs and s_tmp are free again
  } else {
    if (act) s_abs[c] = ax;
    __syncthreads();
    int gt = 0, ge = 0;
    for (int j = 0; j < D; ++j) {
      const float y = s_abs[j];
      gt += (y > ax) ? 1 : 0;
      ge += (y >= ax) ? 1 : 0;
    }
    if (act && gt <= nov && nov < ge) *s_scale = ax;
    __syncthreads();
    s = *s_scale;
    __syncthreads();
  }
  const float inv = s > 0.f ? __fdiv_rn(1.0f, s) : 0.f;
  const float xhat = __fmul_rn(x, inv);
  const int nc = 1 << sd.bits;
  const float *mid = cbtab + cb_offset(sd.bits) + 2 * nc + (nc - 1);
  const int code = code_from_mid(xhat, mid, nc - 1);
  const bool outl = act && sd.bp > 0 && ax > s;
  int total;
  const int r = flag_rank<D>(outl, s_tmp, &total);
  // slot-major: entry r of token t at r * cap + t
  uint32_t *vo = reinterpret_cast<uint32_t *>(sd.vout) + h * stride_vout(sd) + t;
  uint32_t *vd = reinterpret_cast<uint32_t *>(sd.vdel) + h * stride_vout(sd) + t;
  if (outl && r < sd.nov_slots) {
    vo[(size_t)r * sd.cap] = outlier_entry(vbits, t, code, c);
    // the attention's form: the outlier minus the value its code stands for, and the channel
    const float cbv = cbtab[cb_offset(sd.bits) + nc + code];
    vd[(size_t)r * sd.cap] = vdel_pack(__fsub_rn(x, __fmul_rn(s, cbv)), c);
  }
  if (c >= total && c < sd.nov_slots) {
    vo[(size_t)c * sd.cap] = kNoOutlier;
    vd[(size_t)c * sd.cap] = 0u;
  }
  if (c == 0) (reinterpret_cast<float *>(sd.vmeta) + h * stride_slots(sd))[t] = s;
  return code;
}

// Write the value codes of tokens t0..t0+3 (one 4-token block) from an LDS block image.
template <int NT>
MKV_DEV void store_quad(const SeqDesc &sd, int h, int t0, const uint32_t *s_blk, int D) {
  const int words = D * sd.bits / 8;  // 4 tokens x D codes x bits / 32
  uint32_t *dst = reinterpret_cast<uint32_t *>(reinterpret_cast<uint8_t *>(sd.vc) + h * stride_codes(sd) +
                                               (size_t)(t0 / 4) * 4 * sd.rowbytes);
  for (int w = threadIdx.x; w < words; w += NT) gst(dst + w, s_blk[w]);
}

// The frozen (threshold, 1 / threshold) pair of KVQ key channel c of kv head h.
MKV_DEV float2 kvq_key_tau(const SeqDesc &sd, int h, int c, int D) {
  return (reinterpret_cast<const float2 *>(sd.kmeta) + (size_t)h * D)[c];
}

// KVQ key of one token: code under the frozen per-channel threshold ti (kvq_key_tau), and the
// outlier flag.
MKV_DEV int kvq_key_code(const SeqDesc &sd, float2 ti, uint32_t kbits, const float *cbtab, bool *outl) {
  const float x = h2f(kbits);
  const float xhat = __fmul_rn(x, ti.y);
  const int nc = 1 << sd.bits;
  const float *mid = cbtab + cb_offset(sd.bits) + 2 * nc;
  *outl = sd.bp > 0 && fabsf(x) > ti.x;
  return code_from_mid(xhat, mid, nc - 1);
}

// UQ value of one token: 64-channel groups, one wave per group; returns this thread's code
// (the caller places it in the token's 4-token block) and writes the group's (min, step).
template <int D>
MKV_DEV int uq_value_token(const SeqDesc &sd, int h, int t, uint32_t vbits) {
  const int c = threadIdx.x;
  const float x = h2f(vbits);
  const float mn = wave_min(x), mx = wave_max(x);
  const float r = __fsub_rn(mx, mn);
  const float inv = r > 0.f ? __fdiv_rn(15.0f, r) : 0.f;
  const float y = __fmul_rn(__fsub_rn(x, mn), inv);
  const int code = (int)fminf(fmaxf(rintf(y), 0.f), 15.f);
  if ((c & 63) == 0 && c < D)
    (reinterpret_cast<float2 *>(sd.vmeta) + h * stride_uq_vmeta(sd, D))[(size_t)t * (D / 64) + c / 64] =
        make_float2(mn, __fdiv_rn(r, 15.0f));
  return code;
}

// OR a UQ value code into an LDS image of its 4-token block (nibbles never straddle words).
MKV_DEV void or_uq_code(uint32_t *s_blk, int ch, int j, int code, int D) {
  const int bit = uq_vbit(ch, j, D);
  atomicOr(&s_blk[bit >> 5], (uint32_t)code << (bit & 31));
}

// Write a 4-token block (D/2 words) from an LDS image by NT threads; t0 is the block's first slot.
template <int NT>
MKV_DEV void store_block(uint8_t *codes, int h_stride_bytes, int h, int t0, int rowbytes, const uint32_t *s_blk,
                         int words) {
  uint32_t *dst = reinterpret_cast<uint32_t *>(codes + (size_t)h * h_stride_bytes + (size_t)(t0 / 4) * 4 * rowbytes);
  for (int w = threadIdx.x; w < words; w += NT) gst(dst + w, s_blk[w]);
}

// UQ key block: thread c quantizes channel c over 64 tokens read through `get(t)`.
template <int D, typename Get>
MKV_DEV void uq_key_block(const SeqDesc &sd, int h, int blk, Get get) {
  const int c = threadIdx.x;
  float mn = INFINITY, mx = -INFINITY;
  for (int t = 0; t < 64; ++t) {
    const float x = h2f(get(t));
    mn = fminf(mn, x);
    mx = fmaxf(mx, x);
  }
  const float r = __fsub_rn(mx, mn);
  const float inv = r > 0.f ? __fdiv_rn(15.0f, r) : 0.f;
  uint8_t *base = reinterpret_cast<uint8_t *>(sd.kc) + h * stride_codes(sd) + (size_t)blk * 64 * (D / 2);
  for (int t = 0; t < 64; ++t) {
    const float x = h2f(get(t));
    const float y = __fmul_rn(__fsub_rn(x, mn), inv);
    const int code = (int)fminf(fmaxf(rintf(y), 0.f), 15.f);
    const int partner = __shfl_down(code, 1);
    if ((c & 1) == 0) base[(size_t)t * (D / 2) + c / 2] = (uint8_t)(code | (partner << 4));
  }
  (reinterpret_cast<float2 *>(sd.kmeta) + h * stride_uq_kmeta(sd, D))[(size_t)blk * D + c] =
      make_float2(mn, __fdiv_rn(r, 15.0f));
}

// ---- the append ---------------------------------------------------------------------------------
template <int D>
struct AppendLds {
  float abs[D];
  float scale;
  uint8_t code[D];
  int tmp[4];
  uint32_t blk[D / 2];
  float cbt[kCbTableFloats];  // codebooks and midpoints, read many times below
};

// H2O: the slot the last attention pass chose for eviction (-1: none), the lowest (score,
// position) key among its per-part candidates (uniform, so that the loads are scalar and overlap).
MKV_DEV int h2o_victim(const SeqDesc &sd, int h) {
  const uint32_t *vb = reinterpret_cast<const uint32_t *>(sd.vbest) + (size_t)h * sd.vparts * 4;
  unsigned long long best = ~0ull;
  int slot = -1;
  for (int p = 0; p < sd.vparts; ++p) {
    const unsigned long long key = (unsigned long long)vb[4 * p] | ((unsigned long long)vb[4 * p + 1] << 32);
    if (key < best) {
      best = key;
      slot = (int)vb[4 * p + 2];
    }
  }
  return slot;
}

// Slot the next token of (seq, h) goes to: an H2O victim's, else the end.  It is not below the capacity
// where the region is full.
MKV_DEV int append_slot(const SeqDesc &sd, int h, int count, int *victim) {
  *victim = sd.method == H2O ? h2o_victim(sd, h) : -1;
  return *victim >= 0 ? *victim : count;
}

// What thread c appends, and the reads of the append that need only the descriptor, issued together
// (the codebooks before the method is known: into LDS, for a barrier of append_pair).
struct NewToken {
  uint32_t k, v;  // fp16 bits
  float2 tau;     // KVQ: the key channel's thresholds
  int kfill;      // KVQ: ST_KOUT_FILL
};

template <int D, int NT>
MKV_DEV NewToken load_token(const SeqDesc &sd, const int32_t *st, int seq, int h, int Hkv,
                            const uint16_t *__restrict__ k, const uint16_t *__restrict__ v,
                            const float *__restrict__ cbtab, AppendLds<D> &L) {
  for (int i = threadIdx.x; i < kCbTableFloats; i += NT) L.cbt[i] = cbtab[i];
  const int c = NT == D ? (int)threadIdx.x : min((int)threadIdx.x, D - 1);
  const size_t at = ((size_t)seq * Hkv + h) * D + c;
  return {k[at], v[at], sd.method == KVQ ? kvq_key_tau(sd, h, c, D) : make_float2(0.f, 0.f), st[ST_KOUT_FILL]};
}

// Append the new token of (seq, h), which goes to `slot` (append_slot), by a workgroup of NT threads
// that all call this.  False, with nothing written, if a region is full (reachable only by replaying a
// captured decode step past max_new_tokens: the token is dropped instead of written past the region).
// Only the counts are left to the caller: those after the append are (count + (victim < 0),
// position + 1).  A workgroup that goes on to read what was written waits for its stores and a barrier;
// one that goes on to use the LDS of L for something else needs that barrier after either result (a
// dropped token leaves load_token's stores into L unordered between the waves).
template <int D, int NT>
MKV_DEV bool append_pair(const SeqDesc &sd, int32_t *st, const NewToken &tok, int h, int count, int pos, int slot,
                         int victim, AppendLds<D> &L) {
  float *s_abs = L.abs, *s_cbt = L.cbt;
  uint8_t *s_code = L.code;
  int *s_tmp = L.tmp;
  uint32_t *s_blk = L.blk;
  const int c = threadIdx.x;
  const bool act = NT == D || c < D;
  const uint32_t kb = tok.k, vb = tok.v;
  const float2 ti = tok.tau;
  const int kfill = tok.kfill;
  if (slot >= sd.cap || (sd.method == KVQ && sd.bp > 0 && kfill + D > sd.pool_cap)) return false;
  __syncthreads();  // every thread has read the state before thread 0 updates it
  switch (sd.method) {
    case FP16:
    case H2O:
    case ROCKET: {
      if (act) {
        (reinterpret_cast<uint16_t *>(sd.k) + h * stride_rows(sd, D))[(size_t)slot * D + c] = (uint16_t)kb;
        (reinterpret_cast<uint16_t *>(sd.v) + h * stride_rows(sd, D))[(size_t)slot * D + c] = (uint16_t)vb;
        if (sd.method == ROCKET)
          (reinterpret_cast<uint16_t *>(sd.kcm) + h * stride_kcm(sd, D))[(size_t)c * sd.cstride + slot] = (uint16_t)kb;
      }
      if (c == 0 && sd.method != FP16) (reinterpret_cast<int32_t *>(sd.pos) + h * stride_slots(sd))[slot] = pos;
      if (c == 0 && sd.method == H2O) (reinterpret_cast<float *>(sd.score) + h * stride_slots(sd))[slot] = 0.f;
      break;
    }
    case UQ: {
      const int vcode = uq_value_token<D>(sd, h, count, vb);
      // the value code goes into its 4-token block: zero for the block's first token, otherwise
      // the stored block
      const int j = count & 3, words = D / 2;
      const uint32_t *blk = reinterpret_cast<const uint32_t *>(reinterpret_cast<const uint8_t *>(sd.vc) +
                                                               h * stride_codes(sd) + (size_t)(count / 4) * 4 * sd.rowbytes);
      for (int w = c; w < words; w += NT) s_blk[w] = j == 0 ? 0u : gld(blk + w);
      __syncthreads();
      if (act) or_uq_code(s_blk, c, j, vcode, D);
      __syncthreads();
      store_block<NT>(reinterpret_cast<uint8_t *>(sd.vc), (int)stride_codes(sd), h, count & ~3, sd.rowbytes, s_blk, words);
      uint16_t *res = reinterpret_cast<uint16_t *>(sd.kres) + (size_t)h * 64 * D;
      if (act) res[(size_t)(count & 63) * D + c] = (uint16_t)kb;
      if ((count & 63) == 63) {
        // the block is complete: thread c quantizes channel c of the 64 residual rows it wrote
        __syncthreads();
        if (act) uq_key_block<D>(sd, h, count >> 6, [&](int t) { return (uint32_t)res[(size_t)t * D + c]; });
      }
      break;
    }
    case KVQ: {
      bool outl;
      const int code = kvq_key_code(sd, ti, kb, s_cbt, &outl);
      outl = outl && act;
      uint8_t *row = reinterpret_cast<uint8_t *>(sd.kc) + h * stride_codes(sd) + (size_t)count * sd.rowbytes;
      pack_row<D>(code, sd.bits, s_code, row);
      int total;
      const int r = flag_rank<D>(outl, s_tmp, &total);
      uint32_t *ko = reinterpret_cast<uint32_t *>(sd.kout) + h * stride_kout(sd);
      if (outl) ko[kfill + r] = outlier_entry(kb, count, code, c);
      const int vcode = kvq_value_token<D>(sd, h, count, vb, s_cbt, s_abs, &L.scale, s_tmp);
      // the value code goes into its 4-token block: the block's first token writes the whole
      // block (other tokens' codes zero); later tokens OR their bits into the stored words
      const int j = count & 3, words = D * sd.bits / 8;
      if (j == 0) {
        for (int w = c; w < words; w += NT) s_blk[w] = 0u;
        __syncthreads();
        if (act) or_quad_code(s_blk, c, j, vcode, sd.bits);
        __syncthreads();
        store_quad<NT>(sd, h, count & ~3, s_blk, D);
      } else if (act) {
        uint32_t *blk = reinterpret_cast<uint32_t *>(reinterpret_cast<uint8_t *>(sd.vc) + h * stride_codes(sd) +
                                                     (size_t)(count / 4) * 4 * sd.rowbytes);
        const int bit = sd.bits * (4 * c + j);
        atomicOr(blk + (bit >> 5), (uint32_t)vcode << (bit & 31));
        const int spill = (bit & 31) + sd.bits - 32;
        if (spill > 0) atomicOr(blk + (bit >> 5) + 1, (uint32_t)vcode >> (sd.bits - spill));
      }
      if (c == 0) {
        (reinterpret_cast<uint32_t *>(sd.krow) + h * stride_krow(sd))[count + 1] = (uint32_t)(kfill + total);
        st[ST_KOUT_FILL] = kfill + total;
      }
      break;
    }
    default:
      break;
  }
  return true;
}

}  // namespace

}  // namespace mkv
