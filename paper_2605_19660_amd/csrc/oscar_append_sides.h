// The encoder's form for the smallest launches (append_in_sides): two workgroups of 512 threads a block of 128
// tokens, one for the keys and one for the values, which touch different arrays.
//
// Bound: latency.  The chain is kernel arguments, lengths, loads, transform, tail, codes, so
//  * the arguments are asked for at once, and the lengths and the page by scalar loads that nothing else waits on;
//  * every load of the block and of the tail goes out together, as buffer loads without branches: where a token
//    is not there the offset lies past the resource's end.  The tokens of a block that begins with the old window
//    came one branch after another before, each behind the whole of the last one's answer, and the tail's behind
//    the block's transform (whole calls in us, bf16 INT2, 8 heads, the calls' host part alike: pieces of 2 x 500
//    8.75 -> 7.7, of 1 x 100 7.45 -> 6.9, fp32 8 x 64 6.1 -> 5.8).
#pragma once
#include "oscar_append_kernel.h"

#pragma clang fp contract(off)

namespace {

// A thread of the 512 holds four tokens of the block, every second pass of 16: thread group 0 (tid < 256) the
// even ones, group 1 the odd ones, which are the two halves of a packed value piece.
template <typename IO, typename META, int BITS, int KG, int XF>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(sizeof(IO) == 4 ? (XF == XF_ALL_HEADS ? 2 : 3) : 4)))
void oscar_append_sides_kernel(AppendParams P) {
  static_assert(XF == XF_PUBLISHED || XF == XF_ALL_HEADS);   // (the norms over all heads are there: first launch)
  constexpr bool NORM_ALL = XF == XF_ALL_HEADS;
  constexpr int NP = 4, ROWS = 32;
  __shared__ EncoderLds<META, BITS, KG, NP> s;
  const int b = blockIdx.z >> 1, kvh = blockIdx.x, blk = blockIdx.y;
  const int tid = threadIdx.x, row = tid >> 4;
  const int slot = row & 15, grp = tid >> 8, qj = tid & 3;
  const int cg = channel_group_of_row_lane(tid & 15);
  auto token = [&](int j) { return 16 * (2 * j + grp) + slot; };   // of the block, in register j
  const int Hkv = P.c.cfg.n_kv_heads;
  const bool zp_min = P.c.cfg.zp_mode == OSCAR_ZP_MIN;
  uint32_t sgn[4];
#pragma unroll
  for (int st = 0; st < 4; ++st) sgn[st] = ((cg >> st) & 1) ? 0x80000000u : 0u;

  // every parameter is asked for in front of the lengths (the scalar loads come back in any order, so what is
  // asked for behind them waits for them)
  asm volatile("" ::"s"(P.k), "s"(P.v), "s"(P.c.res_k), "s"(P.c.res_v), "s"(P.c.res_norm), "s"(P.c.block_table),
               "s"(P.c.seq_lens), "s"(P.c.res_lens), "s"(P.new_lens), "s"(P.T), "s"(P.flags), "s"(Hkv),
               "s"(P.c.max_pages_per_seq), "s"(P.c.tickets), "s"(P.c.dev_status), "s"(P.g.k_codes_bytes),
               "s"(P.g.k_meta_bytes), "s"(P.g.k_norms_bytes), "s"(P.g.v_codes_bytes), "s"(P.g.v_meta_bytes),
               "s"(P.c.k_norms), "s"(P.c.cfg.zp_mode));
  const SeqPlan sp = plan_sequence<true>(P, b);
  if (sp.n > 0 && !sp.ok && tid == 0 && blk == 0 && kvh == 0 && P.c.dev_status) *P.c.dev_status = OSCAR_ERR_CAPACITY;
  const bool active = sp.n > 0 && sp.ok;
  const bool do_block = active && blk < sp.nq;
  // the new tokens that stay in the window: first of them, its slot there, their number (block 0's workgroup)
  const int src0 = sp.nq == 0 ? 0 : sp.nq * R - sp.r0, dst0 = sp.nq == 0 ? sp.r0 : 0;
  const int cnt = active && blk == 0 ? sp.n - src0 : 0;
  const int old = do_block && blk == 0 ? sp.r0 : 0;   // tokens of the block that are the old window
  // (a scalar load without a branch around it: nothing waits for it before it is used)
  const int phys = ((ScalarInts)P.c.block_table)[do_block ? (size_t)b * P.c.max_pages_per_seq + sp.packed_pages + blk : 0];
  auto page = [&]() { return (size_t)phys * Hkv + kvh; };
  const size_t res_base = ((size_t)b * Hkv + kvh) * R;
  __half* res_k = reinterpret_cast<__half*>(P.c.res_k) + res_base * D;
  IO* res_v = reinterpret_cast<IO*>(P.c.res_v) + res_base * D;
  META* res_norm = reinterpret_cast<META*>(P.c.res_norm) + res_base;
  auto rsrc = [](auto* p, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<std::remove_const_t<std::remove_pointer_t<decltype(p)>>*>(p), 0,
                                             bytes, 0x00020000);
  };

  int my_ticket = -1;
  auto draw = [&]() { my_ticket = draw_ticket(P.c.tickets, P.c.tickets != nullptr, tid); };
  auto advance_if_last = [&]() {
    if (P.c.tickets && tid < 64 && ticket_answer(my_ticket) == (int)(gridDim.x * gridDim.y * gridDim.z) - 1)
      advance_all(P, tid, 64);
  };

  // ---- loads: every one a buffer load without a branch around it, void where there is nothing.  with_old: of a
  // block that may begin with the old window ----
  struct Keys {
    Raw8<IO> fresh[NP];   // the block's new tokens
    uint4 held[NP];       // its old ones, K_u as it is
    META held_norm[NORM_ALL ? NP : 1], page_norm[NORM_ALL ? NP : 1];
  };
  auto load_keys = [&](Keys& k, auto with_old) {
    const auto rows = block_rows<IO>(P, P.k, b, kvh, blk, sp.r0, do_block);
#pragma unroll
    for (int j = 0; j < NP; ++j) k.fresh[j].load(rows, block_row_offset<IO>(P, blk, sp.r0, token(j), cg), 0);
    const auto rk = rsrc(res_k, old * D * 2), rn = rsrc(res_norm, old * (int)sizeof(META));
    if constexpr (with_old) {
#pragma unroll
      for (int j = 0; j < NP; ++j) k.held[j] = load_once(rk, (token(j) * D + cg * 8) * 2, 0);
    }
    if constexpr (NORM_ALL) {
      // norms of new tokens: the first launch wrote them into the page's slots
      const auto pn = rsrc(static_cast<uint8_t*>(P.c.k_norms) + page() * P.g.k_norms_bytes,
                           do_block ? R * (int)sizeof(META) : 0);
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        if constexpr (with_old) k.held_norm[j] = load_meta_elem<META>(rn, token(j));
        k.page_norm[j] = load_meta_elem<META>(pn, tok_meta_pos(token(j)));
      }
    } else if constexpr (with_old) {
      k.held_norm[0] = load_meta_elem<META>(rn, token(qj));   // (of the token whose norm this lane will have)
    }
  };
  struct Values {
    Raw8<IO> fresh[NP], held[NP];
  };
  auto load_values = [&](Values& v, auto with_old) {
    const auto rows = block_rows<IO>(P, P.v, b, kvh, blk, sp.r0, do_block);
#pragma unroll
    for (int j = 0; j < NP; ++j) v.fresh[j].load(rows, block_row_offset<IO>(P, blk, sp.r0, token(j), cg), 0);
    if constexpr (with_old) {
      const auto rv = rsrc(res_v, old * D * (int)sizeof(IO));
#pragma unroll
      for (int j = 0; j < NP; ++j) v.held[j].load(rv, (token(j) * D + cg * 8) * (int)sizeof(IO), 0);
    }
  };
  // the tail: token i = 32 * j + row of it in register j
  struct Tail {
    Raw8<IO> x[NP];
    META norm[NORM_ALL ? NP : 1];
  };
  auto load_tail = [&](Tail& t, const void* side, bool with_norms) {
    const auto rows = token_rows<IO>(P, side, b, kvh, src0, cnt);
#pragma unroll
    for (int j = 0; j < NP; ++j) t.x[j].load(rows, ((ROWS * j + row) * Hkv * D + cg * 8) * (int)sizeof(IO), 0);
    if constexpr (NORM_ALL) {
      const auto rn = rsrc(res_norm + dst0, with_norms ? cnt * (int)sizeof(META) : 0);
#pragma unroll
      for (int j = 0; j < NP; ++j) t.norm[j] = load_meta_elem<META>(rn, ROWS * j + row);
    }
  };

  // ---- the key transform of the block ----
  auto transform = [&](const Keys& k, auto with_old, uint4 (&ku)[NP], float (&nrm)[NP], float (&nrm_q)[1]) {
    uint4 nu[NP];
    if constexpr (NORM_ALL) {
      const int tail_len = sp.tail_len;
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        float x[8];
        k.fresh[j].widen(x);
        const float pn = to_f32<META>(k.page_norm[j]);
        nu[j] = key_transform8_given<META>(x, sgn, pn, P.c.cfg.rotation == OSCAR_ROTATION_ON);
        // (a window place that the new tail takes holds the tail's norm by now, and the page the old one)
        if constexpr (with_old) nrm[j] = token(j) < old && token(j) >= tail_len ? to_f32<META>(k.held_norm[j]) : pn;
        else nrm[j] = pn;
      }
    } else {
      float x[NP][8], nq;
#pragma unroll
      for (int j = 0; j < NP; ++j) k.fresh[j].widen(x[j]);
      key_transform_4tokens<META>(x, sgn, qj, nq, nu);
      if constexpr (with_old) nrm_q[0] = token(qj) < old ? to_f32<META>(k.held_norm[0]) : nq;
      else nrm_q[0] = nq;
    }
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      if constexpr (!with_old) {
        ku[j] = nu[j];
        continue;
      }
      const bool o = token(j) < old;
      ku[j].x = o ? k.held[j].x : nu[j].x;
      ku[j].y = o ? k.held[j].y : nu[j].y;
      ku[j].z = o ? k.held[j].z : nu[j].z;
      ku[j].w = o ? k.held[j].w : nu[j].w;
    }
  };
  // ---- the tail, behind a barrier that follows every read of the old window ----
  auto store_key_tail = [&](const Tail& t) {
    if (cnt <= ROWS) {   // a token a row or none
      float x[8], nn;
      t.x[0].widen(x);
      uint4 u;
      if constexpr (NORM_ALL)
        u = key_transform8_given<META>(x, sgn, to_f32<META>(t.norm[0]), P.c.cfg.rotation == OSCAR_ROTATION_ON);
      else u = key_transform8<META>(x, sgn, nn);
      if (row < cnt) {
        *reinterpret_cast<uint4*>(res_k + (size_t)(dst0 + row) * D + cg * 8) = u;
        if (!NORM_ALL && cg == 0) res_norm[dst0 + row] = from_f32<META>(nn);
      }
      return;
    }
    uint4 nu[NP];
    float nq = 0.0f;
    if constexpr (NORM_ALL) {
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        float x[8];
        t.x[j].widen(x);
        nu[j] = key_transform8_given<META>(x, sgn, to_f32<META>(t.norm[j]), P.c.cfg.rotation == OSCAR_ROTATION_ON);
      }
    } else {
      float x[NP][8];
#pragma unroll
      for (int j = 0; j < NP; ++j) t.x[j].widen(x[j]);
      key_transform_4tokens<META>(x, sgn, qj, nq, nu);
    }
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      const int i = ROWS * j + row;
      if (i < cnt) {
        *reinterpret_cast<uint4*>(res_k + (size_t)(dst0 + i) * D + cg * 8) = nu[j];
        if (!NORM_ALL && (tid & 15) == j) res_norm[dst0 + i] = from_f32<META>(nq);   // lane j of the first quad has norm j
      }
    }
  };
  auto store_value_tail = [&](const Tail& t) {
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      const int i = ROWS * j + row;
      if (i < cnt) t.x[j].store(res_v + (size_t)(dst0 + i) * D + cg * 8);
    }
  };
  auto merged = [&](const Values& v, auto with_old, Raw8<IO> (&vraw)[NP]) {
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      vraw[j] = v.fresh[j];
      if constexpr (with_old) vraw[j].merge(v.held[j]);
    }
  };

  // Branches around all of a block's work, not around its loads: where branches meet again the compiler waits for
  // what any of them may have asked for.  Blocks of a sequence without an old window, a first prompt's, leave out
  // its loads, which take their turns in the CU's address unit also where they bring nothing; not those of a later
  // block behind one, whose neighbours run the other code: two codes in a launch are fetched twice.  (Whole calls
  // with two clears in front, us, with the void loads / without: 1 x 128 tokens 9.25 / 9.05, 1 x 1024 9.25 / 9.10, 1 x 1000
  // 10.65 / 10.42, fp32 2 x 512 9.59 / 9.31; chosen by block, pieces of 2 x 500 behind 60 tokens 10.7 / 10.95.)
  // The same for the loads of a tail where there is none, in fp32 alone (2 x 512 9.31 / 9.16, INT4 9.51 / 9.33; bf16
  // 1 x 1024 9.10 / 9.14).
  if ((blockIdx.z & 1) == 0) {
    Tail t;
    uint4 ku[NP];
    float nrm[NP] = {}, nrm_q[1] = {};
    auto block = [&](auto with_old, auto with_tail) {
      Keys k;
      load_keys(k, with_old);
      if constexpr (with_tail) load_tail(t, P.k, true);
      __builtin_amdgcn_sched_barrier(0);
      transform(k, with_old, ku, nrm, nrm_q);
    };
    if (do_block && sp.r0 > 0) block(std::true_type(), std::true_type());
    else if (do_block && (cnt > 0 || sizeof(IO) < 4)) block(std::false_type(), std::true_type());
    else if (do_block) block(std::false_type(), std::false_type());
    else load_tail(t, P.k, true);
    __syncthreads();
    draw();
    if (cnt > 0) store_key_tail(t);
    if (do_block) quantize_keys<META, BITS, KG, NP>(s, ku, !NORM_ALL, nrm, nrm_q, P.c, P.g, page(), zp_min, tid, cg);
  } else {
    Tail t;
    Raw8<IO> vraw[NP];
    auto block = [&](auto with_old, auto with_tail) {
      Values v;
      load_values(v, with_old);
      if constexpr (with_tail) load_tail(t, P.v, false);
      __builtin_amdgcn_sched_barrier(0);
      merged(v, with_old, vraw);
    };
    if (do_block && sp.r0 > 0) block(std::true_type(), std::true_type());
    else if (do_block && (cnt > 0 || sizeof(IO) < 4)) block(std::false_type(), std::true_type());
    else if (do_block) block(std::false_type(), std::false_type());
    else load_tail(t, P.v, false);
    __syncthreads();
    draw();
    if (cnt > 0) store_value_tail(t);
    if (do_block) quantize_values<META, BITS, KG, NP>(s, vraw, P.c, P.g, page(), zp_min, tid, cg);
  }
  // ---- length update: whoever draws the last ticket advances the lengths of all sequences.  Every other
  // workgroup's waves consumed their loads of seq_lens / res_lens before the barrier in front of its draw, so no
  // fence is needed; the new lengths become visible to later kernels at the end of this one. ----
  advance_if_last();
}

template <typename IO, typename META, int BITS, int XF>
int launch_sides(const AppendParams& P, dim3 blocks, hipStream_t st) {
  const dim3 grid(blocks.x, blocks.y, 2 * blocks.z), block(512);
  switch (P.g.k_group) {
    case 32: hipLaunchKernelGGL((oscar_append_sides_kernel<IO, META, BITS, 32, XF>), grid, block, 0, st, P); break;
    case 64: hipLaunchKernelGGL((oscar_append_sides_kernel<IO, META, BITS, 64, XF>), grid, block, 0, st, P); break;
    case 128: hipLaunchKernelGGL((oscar_append_sides_kernel<IO, META, BITS, 128, XF>), grid, block, 0, st, P); break;
    default: return OSCAR_ERR_UNSUPPORTED;
  }
  return OSCAR_OK;
}
template <typename IO, int XF> int launch_sides_of_type(const AppendParams& P, dim3 grid, hipStream_t st) {
  const bool two = P.g.bits == 2;
  if (!two && P.g.bits != 4) return OSCAR_ERR_UNSUPPORTED;
  if (P.c.cfg.meta_dtype == OSCAR_F16)
    return two ? launch_sides<IO, __half, 2, XF>(P, grid, st) : launch_sides<IO, __half, 4, XF>(P, grid, st);
  return two ? launch_sides<IO, float, 2, XF>(P, grid, st) : launch_sides<IO, float, 4, XF>(P, grid, st);
}
template <int XF> int launch_sides_all_types(const AppendParams& P, dim3 grid, hipStream_t st) {
  switch (P.c.cfg.io_dtype) {
    case OSCAR_F32: return launch_sides_of_type<float, XF>(P, grid, st);
    case OSCAR_BF16: return launch_sides_of_type<__hip_bfloat16, XF>(P, grid, st);
    case OSCAR_F16: return launch_sides_of_type<__half, XF>(P, grid, st);
    default: return OSCAR_ERR_UNSUPPORTED;
  }
}

}  // namespace
