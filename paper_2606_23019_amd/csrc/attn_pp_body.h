// Body of the ping-pong kernels (attn_fwd.hip, where it is described), included in
// bsattn_fwd_pp_kernel, bsattn_split_kernel and bsattn_mask_split_kernel; not a
// header of its own.
  using T = Tile<BQ, BK, D>;
  constexpr int kSlots = PingPong<BQ, BK, D>::kItems;  // places for an item in a workgroup
  constexpr int kItems = kSlots / PARTS;               // items per workgroup
  __shared__ __attribute__((aligned(1024))) __bf16 Ks_all[kSlots][BK * D];
  __shared__ __attribute__((aligned(1024))) __bf16 Vs_all[kSlots][BK * D];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int grp = __builtin_amdgcn_readfirstlane(wave >> 2);
  const int slot = __builtin_amdgcn_readfirstlane(wave / T::kWaves);
  const int mine = slot % kItems;  // this wave's item
  const int part = slot / kItems;  // and its part of it
  const int gwave = wave % T::kWaves;  // wavefront inside its item
  const int half = lane >> 5;
  const int l32 = lane & 31;
  __bf16* Ks = Ks_all[slot];
  __bf16* Vs = Vs_all[slot];

  // Workgroup b on XCD b mod 8 takes items kItems (b / 8) .. + kItems - 1 of
  // that XCD's sequence: the launch positions x + 8 j of the one-item layout
  // (maskless: from place0 on).
  const int from = DENSE ? place0 : 0;
  auto pos_of = [&](int sl) -> int64_t {
    return (int64_t)(blockIdx.x % kXcds) +
           kXcds * (from + kItems * (int64_t)(blockIdx.x / kXcds) + sl);
  };
  // The look-ups are branch-free (positions clamped, validity applied after
  // the loads), so that the scalar loads of all items go out together:
  // every order entry, then every count and this item's first key block, in
  // two rounds of memory latency instead of one chain per item.
  int it_of[kItems];
#pragma unroll
  for (int sl = 0; sl < kItems; ++sl) {
    const int64_t pos = min(pos_of(sl), (int64_t)n_items - 1);
    if (DENSE || FROM_MASK) {
      int uu;
      const int unit = xcd_slice(pos, n_items / n_qb, n_qb, &uu);
      it_of[sl] = min(max(unit * n_qb + uu, 0), n_items - 1);
    } else {
      it_of[sl] = order[pos];
    }
  }
  __builtin_amdgcn_sched_barrier(0);  // all order loads issued before any is used
  int c_of[kItems];
  int item = 0;
#pragma unroll
  for (int sl = 0; sl < kItems; ++sl) {
    const int it = min(max(it_of[sl], 0), n_items - 1);
    c_of[sl] = DENSE || FROM_MASK ? n_kb : counts[(it / n_qb) % H * n_qb + it % n_qb];
    if (sl == mine) item = it;
  }
  const int bh = item / n_qb;
  const int u = item - bh * n_qb;
  const int h = bh % H;
  const int row = h * n_qb + u;
  const int32_t* list = DENSE || FROM_MASK ? nullptr : lists + (int64_t)row * n_kb;
  // FROM_MASK: the row's words (by scalar loads: vector ones would wait for the tile
  // copies), the walk's current one, and its blocks not yet taken
  const int words = (n_kb + 63) / 64;
  using MaskWord = const __attribute__((address_space(4))) uint64_t;
  MaskWord* mrow = FROM_MASK ? (MaskWord*)(uintptr_t)(mask + (int64_t)row * words) : nullptr;
  auto word_at = [&](int w) {
    const int real = n_kb - 64 * w;  // bits of the word that name a key block, >= 1
    return mrow[w] & (real < 64 ? (1ull << real) - 1ull : ~0ull);
  };
  int w_cur = 0;
  uint64_t left = 0;
  if constexpr (FROM_MASK) {
    static_assert(kItems == 1, "one row a workgroup");
    // all words requested before the first is counted; past the row's end its
    // last word, which does not count
    uint64_t word[kMaskWords];
#pragma unroll
    for (int w = 0; w < kMaskWords; ++w) word[w] = word_at(min(w, words - 1));
    c_of[0] = 0;
#pragma unroll
    for (int w = 0; w < kMaskWords; ++w) c_of[0] += w < words ? __popcll(word[w]) : 0;
    left = word[0];
  }
  // takes the row's next block; there has to be one
  auto next_block = [&]() {
    while (left == 0 && w_cur + 1 < words) left = word_at(++w_cur);
    const int bit = left ? __builtin_ctzll(left) : 0;
    left &= left - 1;
    return 64 * w_cur + bit;
  };
  int t0 = 0;  // place of this group's first key block (maskless)
  auto kblk = [&](int t) { return DENSE ? t0 + t : min(max(list[t], 0), n_kb - 1); };
  int first = FROM_MASK ? 0 : kblk(0);  // in range for every row (n_kb >= 1): read before cnt is known
  asm volatile("" : "+s"(first));     // keeps that load here, not inside the cnt > 0 branch
  __builtin_amdgcn_sched_barrier(0);  // counts and the first key block issued together
  // every item's count: all groups run as many iterations as the longest walk takes
  auto run_of = [&](int c) { return c > kAlone<PARTS> ? (c + PARTS - 1) / PARTS : c; };
  int cnt = 0, n_iter = 0;
  bool shared = false;  // an item of this workgroup is
#pragma unroll
  for (int sl = 0; sl < kItems; ++sl) {
    const int c = pos_of(sl) < n_items ? min(max(c_of[sl], 0), n_kb) : 0;
    n_iter = max(n_iter, run_of(c));
    if (PARTS > 1 && c > kAlone<PARTS>) shared = true;
    if (sl == mine) cnt = c;
  }
  if constexpr (PARTS > 1) {
    const int run = run_of(cnt);
    t0 = min(part * run, cnt);
    cnt = min(run, cnt - t0);
    if constexpr (FROM_MASK) {
      if (cnt > 0) {
        // to block t0: past the words wholly before it, then past the bits
        int skip = t0;
        for (; w_cur + 1 < words; left = word_at(++w_cur)) {
          const int n = __popcll(left);
          if (skip < n) break;
          skip -= n;
        }
        int bit = 0;  // of the word's block of rank skip
#pragma unroll
        for (int step = 32; step > 0; step /= 2)
          if (__popcll(left & ((1ull << (bit + step)) - 1ull)) <= skip) bit += step;
        left &= ~0ull << bit;
        first = next_block();
      }
    } else {
      if (!DENSE) list += t0;
      if (cnt > 0) first = kblk(0);
    }
  }
  int now = first;  // FROM_MASK: the block whose K tile was requested last
  const bool has_item = pos_of(mine) < n_items;

  const int64_t base = (int64_t)(bh / H) * sb + (int64_t)h * sh;
  const __bf16* Qb = Q + base;
  const __bf16* Kb = K + base - kCopyShift;  // read by tile copies only
  const __bf16* Vb = V + base - kCopyShift;

  const int gwave_u = __builtin_amdgcn_readfirstlane(gwave);
  CopyPlan<T, D> cp;
  cp.init(gwave_u, lane, sn);
  if (cnt > 0) issue_tile_copy<T, BK, D>(Ks, Kb, first * BK, N, sn, gwave_u, lane, cp);

  // Q^T fragments (B operand): lane holds Q[row gwave 32 + l32 of the item]
  // [16 dc + 8 half .. +7].  With square tiles the item's Q rows come in as
  // one more tile copy, into its V tile (free until the first softmax phase
  // issues V[0]), and are read from there after the barriers below: rows of
  // 256 contiguous bytes per four lanes instead of 32 rows per load
  // instruction.  In a ragged last query block, rows past N hold row N - 1
  // (their outputs are not stored); a workgroup slot without an item copies
  // the clamped item's rows and stores nothing.
  constexpr bool kStageQ = BQ == BK;
  const int qrow = u * BQ + gwave * 32 + l32;
  bf16x8 qf[D / 16];
  if constexpr (kStageQ) {
    issue_tile_copy<T, BK, D>(Vs, Qb - kCopyShift, u * BQ, N, sn, gwave_u, lane, cp);
  } else {
#pragma unroll
    for (int dc = 0; dc < D / 16; ++dc) {
      if (has_item && qrow < N)
        qf[dc] = *(const bf16x8*)(Qb + (int64_t)qrow * sn + dc * 16 + half * 8);
      else
        qf[dc] = bf16x8{};
    }
  }
  __builtin_amdgcn_s_waitcnt(0xF70);  // vmcnt(0): Q and K[0] landed

  f32x16 o[D / 32];
#pragma unroll
  for (int dg = 0; dg < D / 32; ++dg) o[dg] = f32x16{};
  float m_run = -INFINITY;
  float l_run = 0.f;
  const int g = lane >> 4;
  const int j = lane & 15;
  bf16x8 pf[BK / 16];
#pragma unroll
  for (int c = 0; c < BK / 16; ++c) pf[c] = bf16x8{};

  if (grp == 1) barrier_lds_reads_done();  // the second group runs one phase behind
  barrier_lds_reads_done();                // both groups' K[0] (and Q) tiles are in LDS
  if constexpr (kStageQ) {
    // every wavefront's Q copy landed before the first barrier; the group's
    // reads complete before the barrier that ends its first MFMA phase,
    // after which its first softmax phase reuses the tile for V[0]
    const int qr = gwave * 32 + l32;
#pragma unroll
    for (int dc = 0; dc < D / 16; ++dc)
      qf[dc] = lds_read_b128(Vs + qr * D + (((2 * dc + half) ^ swz<D>(qr)) << 3));
  }

  for (int t = 0; t <= n_iter; ++t) {
    // ---- MFMA phase: P V of block t - 1, then S of block t
    if (t >= 1 && t - 1 < cnt) {
#pragma unroll
      for (int c = 0; c < BK / 16; ++c) {
#pragma unroll
        for (int dg = 0; dg < D / 32; ++dg) {
          const int dd = dg * 32 + 16 * (g & 1) + (j & 3) * 4;
          const int r0 = c * 16 + 8 * (g >> 1) + (j >> 2);
          const int r1 = r0 + 4;
          const bf16x4 lo = lds_read_tr16_b64(Vs + r0 * D + (((dd >> 3) ^ swz<D>(r0)) << 3) + (dd & 7));
          const bf16x4 hi = lds_read_tr16_b64(Vs + r1 * D + (((dd >> 3) ^ swz<D>(r1)) << 3) + (dd & 7));
          const bf16x8 a = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
          o[dg] = mfma32x32x16(a, pf[c], o[dg]);
        }
      }
    }
    f32x16 s[BK / 32];
#pragma unroll
    for (int kg = 0; kg < BK / 32; ++kg) s[kg] = f32x16{};
    const bool do_s = t < cnt;
    if (do_s && !kReadAhead<BQ, DENSE, PARTS>) {
#pragma unroll
      for (int dc = 0; dc < D / 16; ++dc) {
#pragma unroll
        for (int kg = 0; kg < BK / 32; ++kg) {
          const int kr = kg * 32 + key_of_row(l32);
          const bf16x8 a = lds_read_b128(Ks + kr * D + (((2 * dc + half) ^ swz<D>(kr)) << 3));
          s[kg] = mfma32x32x16(a, qf[dc], s[kg]);
        }
      }
    } else if (do_s) {
      bf16x8 kf[2][BK / 32];
      auto read_k = [&](int dc, bf16x8 (&f)[BK / 32]) {
#pragma unroll
        for (int kg = 0; kg < BK / 32; ++kg) {
          const int kr = kg * 32 + key_of_row(l32);
          f[kg] = lds_read_b128(Ks + kr * D + (((2 * dc + half) ^ swz<D>(kr)) << 3));
        }
      };
      read_k(0, kf[0]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int dc = 0; dc < D / 16; ++dc) {
        if (dc + 1 < D / 16) read_k(dc + 1, kf[(dc + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kg = 0; kg < BK / 32; ++kg) s[kg] = mfma32x32x16(kf[dc & 1][kg], qf[dc], s[kg]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    barrier_lds_reads_done();  // this group's Ks and Vs are free
    if (t == n_iter) break;

    // ---- softmax phase of block t; copies of V[t] and K[t + 1]
    if (do_s) {
      const int key0 = (FROM_MASK ? now : kblk(t)) * BK;
      const bool more = t + 1 < cnt;
      issue_tile_copy<T, BK, D>(Vs, Vb, key0, N, sn, gwave_u, lane, cp);
      if (key0 + BK > N) {
#pragma unroll
        for (int kg = 0; kg < BK / 32; ++kg)
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int key = key0 + kg * 32 + 16 * (i >> 3) + 8 * half + (i & 7);
            if (key >= N) s[kg][i] = -INFINITY;
          }
      }
      float mx = -INFINITY;
#pragma unroll
      for (int kg = 0; kg < BK / 32; ++kg)
#pragma unroll
        for (int i = 0; i < 16; ++i) mx = fmaxf(mx, s[kg][i]);
      mx = pair_max(mx) * c_log2;
      if (more) {
        if (FROM_MASK) now = next_block();
        issue_tile_copy<T, BK, D>(Ks, Kb, (FROM_MASK ? now : kblk(t + 1)) * BK, N, sn, gwave_u, lane, cp);
      }
      const bool grow = mx > m_run;
      if (__any(grow)) {
        const float m_new = grow ? mx : m_run;
        const float alpha = fast_exp2(m_run - m_new);
        m_run = m_new;
        l_run *= alpha;
#pragma unroll
        for (int dg = 0; dg < D / 32; ++dg) o[dg] *= alpha;
      }
      const float m_exp = PARTS > 1 ? fmaxf(m_run, part_floor<PARTS>(part)) : m_run;
      float lsum = 0.f;
#pragma unroll
      for (int kg = 0; kg < BK / 32; ++kg)
#pragma unroll
        for (int j8 = 0; j8 < 2; ++j8)
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float p = fast_exp2(fmaf(s[kg][8 * j8 + e], c_log2, -m_exp));
            lsum += p;
            pf[2 * kg + j8][e] = (__bf16)p;
          }
      l_run += lsum;
    }
    barrier_copies_landed<0>();  // this group's V[t] and K[t + 1] landed
  }
  if (grp == 0) barrier_lds_reads_done();  // matches the second group's extra barrier

  float l_tot = pair_sum(l_run);
  const int lane_e = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  if constexpr (PARTS > 1)
    if (shared)
      merge_parts<PARTS, kItems * T::kWaves, D, (int)sizeof(Ks_all)>(
          o, m_run, l_tot, (char*)Ks_all, (char*)Vs_all, part, mine * T::kWaves + gwave_u,
          lane_e);
  const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
  const int l32_e = lane_e & 31;
  const int half_e = lane_e >> 5;
  const int row0 = u * BQ + gwave_u * 32;
  if constexpr (kStagedStore<BQ, BK, D, OutT>) {
    // every wavefront's LDS reads and copies are over (the last barrier
    // above), so this item's K and V tiles are free: wavefront w of the item
    // stages its rows in bytes [w S, (w + 1) S) of [Ks | Vs], S = 32 D sizeof(OutT)
    if (has_item && part == 0) {
      if (half_e == 0 && row0 + l32_e < N)
        LSE[(int64_t)bh * N + row0 + l32_e] = l_tot > 0.f ? (m_run + fast_log2(l_tot)) * kLn2 : -INFINITY;
      constexpr int kSlice = 32 * D * (int)sizeof(OutT);
      constexpr int kTileBytes = BK * D * 2;
      const int off = gwave_u * kSlice;
      char* slice = off < kTileBytes ? (char*)Ks + off : (char*)Vs + (off - kTileBytes);
      store_rows_staged<D, OutT>(o, inv, slice, O + base + (int64_t)row0 * sn, sn, N - row0, lane_e);
    }
  } else if (has_item && part == 0 && row0 + l32_e < N) {
    if (half_e == 0)
      LSE[(int64_t)bh * N + row0 + l32_e] = l_tot > 0.f ? (m_run + fast_log2(l_tot)) * kLn2 : -INFINITY;
    OutT* orow = (O + base + (int64_t)row0 * sn) + (uint32_t)(l32_e * sn);
#pragma unroll
    for (int dg = 0; dg < D / 32; ++dg)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4)
        store_out4(orow + dg * 32 + 8 * r4 + 4 * half_e, o[dg][4 * r4 + 0] * inv,
                   o[dg][4 * r4 + 1] * inv, o[dg][4 * r4 + 2] * inv, o[dg][4 * r4 + 3] * inv);
  }
