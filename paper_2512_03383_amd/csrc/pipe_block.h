// What a block of the pipelined kernel does with one tile: the tokens m0 .. m0 + 16 AF - 1 and the BN rows of row tile rt of the linear a; `share`
// token tiles of the row tile run side by side, this one is the `mine`th.  Statements, for two places of pipe_kernel.h to include: the kernel, and the
// function that takes half a tile.  They stand in the kernel itself because as a function that is inlined there the same loops, to the instruction and
// the register, ran up to 1.12 times as long where segments keep part of a block (254 sizes of 4 bits at 24..333 tokens 1.014 in the mean, at worst
// 1.10, so 1.000 and 1.02; 4608 x 8192, 102 of 128 columns, bfloat16, 24 tokens 13.9 us, 15.7 as a function); what it waits for then is not known, it is
// not where the loops lie.
  constexpr int BM = S::BM, BN = S::BN, U = S::U, KS = S::KS, XM = S::XM, WM = S::WM;
  // A slab's activations land by the barrier before its use and not one earlier: its first fragments are then read behind that
  // barrier, but with three or four buffers the loads have a slab more of time.  Small tiles wait for them otherwise, and so do
  // segments in tiles of three buffers, whose movers still clear columns (two decoder layers at 48 tokens 140 -> 125 us a pass, the
  // attention block at 1000 tokens 106 -> 103), and 96 tokens with three buffers, i.e. codes of 8 and 6 bits (12185 x 4096 at 333 tokens
  // 67.5 -> 56.4 and 75.8 -> 65.3 us; 73.2 with 6 bits before units were placed by bank_key).  Prefixes in 96..112-token tiles of four
  // buffers and in 128-token ones go the other way (4 bits, 5120 x 4096 at 512 tokens 31.2 -> 33.2 us).
  // (16 x 32 tiles of up to 6 bits: early is up to 8 % better, rows of 14208 columns on segments above all; 8 bits: level)
  constexpr bool XLate = S::Small ? NX <= 4 && !(AF == 1 && BF == 1 && BITS != 8) : NX == 3 && (SEG || AF == 6);
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  const KeepMap& km = a.km;
  const int n0 = rt * BN;
  const int row_bytes = a.K_total / 8 * BITS, gpr = a.K_total / kGroup;
  const int ngroups = (km.k_span + kGroup - 1) / kGroup;
  const int nslab = (ngroups + G - 1) / G;
  // column segments: a power of two up to the group's 128 columns (the host checks), so every group has the same pattern
  const int seg_shift = SEG ? __builtin_ctz((unsigned)km.cs_stride) : 0;

  if (wave >= kPipeConsumers) {
    __builtin_amdgcn_s_setprio(3);
    typedef __attribute__((address_space(3))) unsigned char lds_byte;
    typedef __attribute__((address_space(3))) void lds_void;
    lds_byte* const lds = (lds_byte*)smem;
    // A mover's walk: slabs 0 .. N - 2 to begin with, then, one barrier per slab, the slab that takes the buffer which
    // everybody has left.  Before barrier `it` the slabs up to it + 1 have landed (codes, and activations unless XLate), or up to `it`
    // (`late`: activations with XLate).  Before barrier `extra_at` (the one that publishes the last slab, or -1 for none) the mover does
    // something more; with column segments it does `landed` for every slab's buffer before the barrier that publishes it.
    auto walk = [&](auto n, auto per, auto late, auto&& move, int extra_at, auto&& extra, auto&& landed) {
      constexpr int N = decltype(n)::value, PER = decltype(per)::value, AHEAD = decltype(late)::value ? 0 : 1;
#pragma unroll
      for (int p = 0; p < N - 1; ++p)
        if (p < nslab) move(p, p);
      int buf = N - 1, lbuf = AHEAD;                     // the buffers of slabs it + N - 1 and it + AHEAD
      for (int it = 0; it < nslab; ++it) {
        if (it + (N > 3 || !AHEAD ? N - 2 : 2) < nslab) {
          asm volatile("s_waitcnt vmcnt(%0)" ::"n"((N - 2 - AHEAD) * PER) : "memory");
        } else {
          // (the last slabs; `extra` is asked for here only: on the way from the wait to the barrier it costs 3 % at NX = 3)
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
          if (it == extra_at) extra();
        }
        if constexpr (SEG) {
          if (AHEAD && it == 0) landed(0);
          if (it + AHEAD < nslab) landed(lbuf);
          lbuf = lbuf + 1 == N ? 0 : lbuf + 1;
        }
        pipe_barrier();
        if (it + N - 1 < nslab) move(it + N - 1, buf);
        buf = buf + 1 == N ? 0 : buf + 1;
      }
      pipe_barrier();
    };
    if (wave < kPipeConsumers + XM) {
      // ---- activations
      auto move_activations = [&](auto movers, const int d) {   // (d: which of the movers)
        constexpr int XM = decltype(movers)::value, XPW = S::XI / XM;
        const int mt = a.M - m0 < BM ? a.M - m0 : BM;
        const int ldx2 = (int)a.ldx * 2;
        // rows past the last token lie beyond the resource and read as zero
        const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<half_t*>(a.x + (size_t)m0 * a.ldx), 0,
                                                                            (mt - 1) * ldx2 + km.k_keep * 2, kBufferWord3);
        // Byte offset of this lane's unit of load k in slab `slab`.  Segments divide the groups, so every group is alike: its
        // kept columns are `kpg` consecutive ones of x, a block's kept columns its first ones, contiguous.  A slab that lies
        // wholly in the row takes slab 0's offsets and a scalar (a load is then two instructions; a mover issues one
        // every 60 clocks otherwise).
        const int kpg = SEG ? (kGroup >> seg_shift) * km.cs_keep : kGroup;
        const int partial = SEG ? km.cs_keep & 7 : 0, seg_log = 7 - seg_shift;   // columns in a segment's last block (even), segments of a group
        auto unit = [&](int k, int slab) {
          constexpr int CH = 16 * G;                       // chunks per token
          const int v = (d + XM * k) * 64;
          const int tok = v / CH + (CH < 64 ? lane / CH : 0);
          const int c = (CH <= 64 ? lane % CH : v % CH + lane) ^ bank_key(tok);
          const int g = slab * G + c / 16, k0 = (c % 16) * 8;   // group, column in it
          int col = g * kpg + k0;
          bool there = g * kGroup + k0 < km.k_keep;        // a prefix: its last block comes with what lies behind it
          if constexpr (SEG) {
            const int off = k0 & (km.cs_stride - 1);
            col = g * kpg + (k0 >> seg_shift) * km.cs_keep + off;
            there = off < km.cs_keep && g < ngroups;
          }
          return there ? tok * ldx2 + col * 2 : kBeyond;
        };
        const int nwhole = SEG ? ngroups / G : km.k_keep / (G * kGroup);
        // The last block of a prefix whose columns are not whole blocks, in LDS: what lies behind the kept columns is cleared, and
        // an odd last column, whose word may lie partly past the resource and then reads as zero, is put in place from a load of
        // its own.  A lane per token, each mover the tokens that it has loaded itself.  (Added up in the epilogue, column after
        // column, they cost a chain of loads per fragment: 4096 x 9318 at 48 / 777 tokens 22.9 / 106 us, so 18.6 / 70.)
        const int tail = SEG ? 0 : km.k_keep & 7;
        constexpr int TI = (BM + 63) / 64;
        uint32_t odd[TI];
#pragma unroll
        for (int i = 0; i < TI; ++i) {
          const int t = lane + 64 * i;
          odd[i] = (tail & 1) && t < mt ? (uint32_t)__builtin_bit_cast(uint16_t, a.x[(size_t)(m0 + t) * a.ldx + km.k_keep - 1]) : 0u;
        }
        // Segments: the block that holds a segment's last kept columns arrives with the next segment's first ones (or the next
        // token's) behind them, which are cleared here, in the mover's own tokens (masked in the registers of the eight waves
        // that multiply, they were four vector instructions per activation fragment and step: 1000 x 4096 x 4096 in bfloat16, 108
        // of 128 columns, 62 -> 41 us, and 128 tokens a tile did not fit the registers).  Slabs are alike, so where those blocks lie is
        // worked out once, a lane's block of each turn: for every slab anew it was what a slab of short segments took (6 of 8
        // columns: 4096 x 8192 at 777 tokens in 112 x 128 tiles, 3 bits, 1.5 times as long, 32 x 32 tiles of 8 bits up to twice).  Lanes
        // without a block clear the last one again (a test of each costs 5 % with 32 x 32 tiles).
        const int blocks = (BM / XM * G) << seg_log, turns = partial ? (blocks + 63) / 64 : 0;
        int clear[SEG ? XPW : 1];                        // (segments of eight columns: as many turns as loads)
        if constexpr (SEG) {
          constexpr int TU = 4 / G;                      // tokens per load
#pragma unroll
          for (int k = 0; k < XPW; ++k) {
            const int i = lane + 64 * k < blocks ? lane + 64 * k : blocks - 1;
            const int sg = i & ((1 << seg_log) - 1), g = (i >> seg_log) % G, j = (i >> seg_log) / G;
            const int t = (j / TU * XM + d) * TU + j % TU, c = g * 16 + (sg << (seg_shift - 3)) + km.cs_keep / 8;
            clear[k] = (t * (16 * G) + (c ^ bank_key(t))) * 16;
          }
        }
        int first[XPW];                                 // (of use when there is a whole slab: then slab 0 is one)
#pragma unroll
        for (int k = 0; k < XPW; ++k) first[k] = unit(k, 0);
        walk(std::integral_constant<int, NX>(), std::integral_constant<int, XPW>(), std::integral_constant<bool, XLate>(), [&](int slab, int buf) {
          lds_byte* const to = lds + buf * S::XBytes + d * 1024;
          if (slab < nwhole) {
#pragma unroll
            for (int k = 0; k < XPW; ++k)
              __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_void*)(to + k * (XM * 1024)), 16, first[k], slab * (G * kpg * 2), 0, 0);
          } else {
#pragma unroll
            for (int k = 0; k < XPW; ++k)
              __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_void*)(to + k * (XM * 1024)), 16, unit(k, slab), 0, 0, 0);
          }
        }, tail == 0 ? -1 : nslab > 1 ? nslab - (XLate ? 1 : 2) : 0, [&]() {
          const int c = km.k_keep / 8 - (nslab - 1) * (16 * G), keep = tail & ~1;   // chunk in the slab, columns that stay
          auto m = [&](int i) { return keep > i ? ~0u : 0u; };
#pragma unroll
          for (int i = 0; i < TI; ++i) {
            const int t = lane + 64 * i;
            if (t >= BM || (t * G / 4) % XM != d) continue;
            uint4* p = reinterpret_cast<uint4*>(smem + (nslab - 1) % NX * S::XBytes) + t * (16 * G) + (c ^ bank_key(t));
            uint4 v = *p;
            v.x = (v.x & m(0)) | (tail == 1 ? odd[i] : 0u);
            v.y = (v.y & m(2)) | (tail == 3 ? odd[i] : 0u);
            v.z = (v.z & m(4)) | (tail == 5 ? odd[i] : 0u);
            v.w = tail == 7 ? odd[i] : 0u;
            *p = v;
          }
        }, [&](int buf) {
          if constexpr (SEG) {
            unsigned char* const to = smem + buf * S::XBytes;
            auto each = [&](auto&& put) {
#pragma unroll
              for (int k = 0; k < XPW; ++k) {
                if (k >= turns) return;
                put(reinterpret_cast<uint32_t*>(to + clear[k]));
              }
            };
            if (partial == 6) each([](uint32_t* p) { p[3] = 0u; });
            else if (partial == 4) each([](uint32_t* p) { *reinterpret_cast<u32x2_t*>(p + 2) = u32x2_t{0u, 0u}; });
            else each([](uint32_t* p) { p[1] = 0u; *reinterpret_cast<u32x2_t*>(p + 2) = u32x2_t{0u, 0u}; });
          }
        });
      };
      if (!S::TwoStandBy || nslab <= S::MostSlabsOfFour) move_activations(std::integral_constant<int, XM>(), wave - kPipeConsumers);
      else if (wave >= kPipeConsumers + XM / 2) move_activations(std::integral_constant<int, XM / 2>(), wave - kPipeConsumers - XM / 2);
      else for (int it = 0; it <= nslab; ++it) pipe_barrier();
      return;
    }
    if (wave < kPipeConsumers + XM + WM) {
      // ---- codes
      const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(a.qweight), 0, a.N_total * row_bytes, kBufferWord3);
      const int d = wave - kPipeConsumers - XM;
      int woff[S::WPW];                                  // byte offset of the lane's unit in slab 0
#pragma unroll
      for (int k = 0; k < S::WPW; ++k) {
        const int v = (d + WM * k) * 64 + lane, row = v / U, j = v - row * U;
        int js = j;
        if constexpr ((U & (U - 1)) == 0) js = j ^ (bank_key(row) / (U < 16 ? 16 / U : 1));
        int rc = n0 + row;
        rc = rc < km.n_keep ? rc : km.n_keep - 1;       // (rows past the last one: a valid, unused load)
        woff[k] = stored_row(km, rc) * row_bytes + js * 16;
      }
      walk(std::integral_constant<int, NW>(), std::integral_constant<int, S::WPW>(), std::false_type(), [&](int slab, int buf) {
        lds_byte* const to = lds + S::W0 + buf * S::WBytes + d * 1024;
        if ((slab + 1) * G <= gpr) {
#pragma unroll
          for (int k = 0; k < S::WPW; ++k)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_void*)(to + k * (WM * 1024)), 16, woff[k], slab * (U * 16), 0, 0);
        } else {
          // (a slab's groups past the row's end: the next row's codes, or nothing behind the matrix; their scale is zero)
#pragma unroll
          for (int k = 0; k < S::WPW; ++k)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_void*)(to + k * (WM * 1024)), 16, woff[k] + slab * (U * 16), 0, 0, 0);
        }
      }, -1, []() {}, [](int) {});
      return;
    }
    // ---- scales and zero points: row lane (+ 64 p) of the block, windows of eight groups, scale | zero << 16.  The window
    // never leaves the row (a load whose last word lies partly past the array comes back with that word zeroed): at the
    // row's end it starts `back` groups earlier and is shifted.  Groups past the last one get a zero scale.
    constexpr int P = (BN + 63) / 64, SPW = 8 / G;      // rows per lane, slabs per window
    uint32_t* szs = reinterpret_cast<uint32_t*>(smem + S::SZ0);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a.scales), 0, a.N_total * gpr * 2, kBufferWord3);
    const __amdgpu_buffer_rsrc_t rz = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(a.zeros), 0, a.zeros ? a.N_total * gpr : 0, kBufferWord3);
    const bool has_z = a.zeros != nullptr;
    int e0[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
      int rc = n0 + p * 64 + lane;
      rc = rc < km.n_keep ? rc : km.n_keep - 1;
      e0[p] = stored_row(km, rc) * gpr;
    }
    u32x4_t s[P];
    u32x2_t z[P];
    auto fetch = [&](int w) {
      const int g = 8 * w, back = g + 8 > gpr ? g + 8 - gpr : 0;
      const bool there = g < ngroups;
#pragma unroll
      for (int p = 0; p < P; ++p) {
        s[p] = __builtin_amdgcn_raw_buffer_load_b128(rs, there ? 2 * (e0[p] + g - back) : kBeyond, 0, 0);
        z[p] = __builtin_amdgcn_raw_buffer_load_b64(rz, there ? e0[p] + g - back : kBeyond, 0, 0);
      }
    };
    auto put = [&](int w) {
      const int g = 8 * w, back = g + 8 > gpr ? (g + 8 - gpr) & 7 : 0;
#pragma unroll
      for (int p = 0; p < P; ++p) {
        const unsigned __int128 sv = ((unsigned __int128)s[p].w << 96 | (unsigned __int128)s[p].z << 64 |
                                      (unsigned __int128)s[p].y << 32 | (unsigned __int128)s[p].x) >> (16 * back);
        const uint64_t zv = has_z ? (((uint64_t)z[p].y << 32) | z[p].x) >> (8 * back) : (uint64_t)(1u << (BITS - 1)) * 0x0101010101010101ull;
        uint32_t o[8];
#pragma unroll
        for (int j = 0; j < 8; ++j)
          o[j] = (g + j < ngroups ? (uint32_t)(sv >> (16 * j)) & 0xffffu : 0u) | ((uint32_t)(zv >> (8 * j)) & 0xffu) << 16;
        const int row = p * 64 + lane;
        uint4* dst = reinterpret_cast<uint4*>(szs + ((w & 1) * BN + row) * 8);
        if (BN % 64 == 0 || row < BN) {
          dst[0] = make_uint4(o[0], o[1], o[2], o[3]);
          dst[1] = make_uint4(o[4], o[5], o[6], o[7]);
        }
      }
    };
    // codes of window w, this block's share of the lines (asm: the compiler would have the stores of the scales wait for them; what they write
    // is not read)
    const bool touches = S::Touches && share == kPipeTokTilesPerPass;
    [[maybe_unused]] u32x4_t rt4 = {};
    [[maybe_unused]] const uint32_t spare = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem + S::Lds - kPipeTouch;
    if constexpr (S::Touches) {
      const uint64_t at = (uint64_t)a.qweight;
      rt4 = u32x4_t{(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)at), (uint32_t)__builtin_amdgcn_readfirstlane((int)((at >> 32) & 0xffffu)),
                    (uint32_t)__builtin_amdgcn_readfirstlane(a.N_total * row_bytes), kBufferWord3};
    }
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"   // (m0 is the compiler's own)
    auto touch = [&](int w) {
      if constexpr (S::Touches) {
        const int end = (w + 1) * 8 < ngroups ? (w + 1) * (128 * BITS) : ngroups * (16 * BITS);
        for (int b = w * (128 * BITS) + mine * 128; b < end; b += kPipeTokTilesPerPass * 128)
#pragma unroll
          for (int p = 0; p < P; ++p)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, %3 offen lds" ::"s"(spare), "v"(e0[p] * (16 * BITS)), "s"(rt4), "s"(b) : "memory", "m0");
      }
    };
#pragma clang diagnostic pop
    fetch(0);
    put(0);
    fetch(1);
    if (touches) {
      // (both windows before the first touches: the stores of a window wait for every load before them)
      put(1);
      fetch(2);
      touch(0);
      touch(1);
    }
    for (int it = 0; it < nslab; ++it) {
      pipe_barrier();
      if (it % SPW == 0 && (!touches || it > 0)) {
        const int w = it / SPW;
        put(w + 1);                       // into the window before the current one
        fetch(w + 2);
        if (touches) touch(w + 1);
      }
    }
    pipe_barrier();
    return;
  }

  // ---- consumers
  const int wn = wave % WN, wk = wave / WN, kg = wk / KQ, kq = wk % KQ;
  const int n = lane & 15, ks = lane >> 4;
  constexpr int SPW = 8 / G, T = S::T;
  float4_t acc[AF][BF];
#pragma unroll
  for (int f = 0; f < AF; ++f)
#pragma unroll
    for (int b = 0; b < BF; ++b) acc[f][b] = float4_t{0.f, 0.f, 0.f, 0.f};
  const CodeMagic mg = make_code_magic<BITS, BF16>();
  // LDS byte offsets inside a slab: activations of the wave's step t of its first group (token n), codes of its slots
  int xoff[T], wro[BF];
#pragma unroll
  for (int t = 0; t < T; ++t) xoff[t] = (n * (16 * G) + kg * 16 + ((ks * 4 + kq * T + t) ^ bank_key(n))) * 16;
#pragma unroll
  for (int b = 0; b < BF; ++b) {
    const int row = (wn * BF + b) * 16 + n, byte = kg * (16 * BITS) + ks * (4 * BITS);   // of the row's codes in the slab
    int o = byte;
    if constexpr ((U & (U - 1)) == 0) {
      // (8 bits: a slot is two units and the permutation may swap them, so the window's own unit is addressed)
      const int by = byte + (BITS == 8 ? kq * (T * BITS) : 0);
      const int sw = bank_key(row) / (U < 16 ? 16 / U : 1);
      o = (((by >> 4) ^ sw) << 4) | (by & 15);
    }
    wro[b] = S::W0 + row * U * 16 + o;
  }
  const uint32_t* szs = reinterpret_cast<const uint32_t*>(smem + S::SZ0) + (wn * BF * 16 + n) * 8 + kg;

  // A step multiplies one unpacked operand per row fragment with AF activation fragments.  Meanwhile the operands of the next
  // step are unpacked between the products -- two waves share a SIMD and run in phase, so a wave that unpacks, then
  // multiplies, leaves the matrix pipe idle while it unpacks -- and the fragments of the next step and the codes of the
  // group after that are read from LDS.
  typedef RawCodes<BITS, T> Raw;
  struct Group { Raw raw[BF]; uint32_t sz[BF]; };
  auto sz_at = [&](int it) { return ((it / SPW) & 1) * (BN * 8) + (it % SPW) * G; };   // of slab `it`, in words
  auto read_group = [&](const unsigned char* sl, int sz, Group& o) {   // sl: smem + offset of the slab's codes; sz: sz_at of it
#pragma unroll
    for (int b = 0; b < BF; ++b) {
      if constexpr (BITS == 8) {
        // a slot is two units of 16 bytes: both or one
#pragma unroll
        for (int h = 0; h < T / 2; ++h) {
          const uint4 v = *reinterpret_cast<const uint4*>(sl + (wro[b] ^ (16 * h)));
          o.raw[b].w[4 * h] = v.x; o.raw[b].w[4 * h + 1] = v.y; o.raw[b].w[4 * h + 2] = v.z; o.raw[b].w[4 * h + 3] = v.w;
        }
      } else {
        o.raw[b] = read_codes<BITS, T>(sl + wro[b], kq);
      }
      o.sz[b] = szs[sz + b * (16 * 8)];
    }
  };
  auto read_a = [&](const unsigned char* sl, int t, uint4 (&o)[AF]) {
#pragma unroll
    for (int f = 0; f < AF; ++f) o[f] = *reinterpret_cast<const uint4*>(sl + xoff[t] + f * (16 * 16 * G) * 16);
  };
  auto constants = [&](auto wide_form, const Group& r, CodeGroup<BITS, BF16> (&o)[BF]) {
#pragma unroll
    for (int b = 0; b < BF; ++b)
      o[b] = make_code_group<BITS, BF16, decltype(wide_form)::value>(r.sz[b] & 0xffffu, r.sz[b] >> 16);
  };
  auto unpack = [&](auto wide_form, int t, const Group& r, const CodeGroup<BITS, BF16> (&c)[BF], uint4 (&o)[BF]) {
#pragma unroll
    for (int b = 0; b < BF; ++b) o[b] = code_step<BITS, BF16, T, decltype(wide_form)::value>(r.raw[b], t, c[b], mg);
  };
  // bfloat16: whether a row of the group has a scale that asks for the wide unpack (codes.h), the same for the whole wave.  (Here
  // and not where the scales are staged: that wave is the last one at the barrier with small tiles, 8 bits at 8 tokens 10 %.)
  auto asks_wide = [&](const Group& r) {
    uint32_t largest = 0;
#pragma unroll
    for (int b = 0; b < BF; ++b) largest = max(largest, r.sz[b] << 17);   // magnitude of the scale
    return __builtin_amdgcn_ballot_w64(largest >= kScaleWide << 17) != 0;
  };
  // With many products a step its reads from LDS stand between them as well: eight waves that all read first wait in line for the LDS
  constexpr bool Spread = AF >= 6 && AF * BF >= 12;   // (64 tokens x 96 rows, 12 products a step of two groups a slab: 2 % slower with it)
  constexpr int kReads = 1 + (BITS == 8 ? T / 2 : BITS == 6 ? (T * BITS / 4 + 1) / 2 : BITS == 4 ? 1 : 2);   // of a row fragment's codes, scale and zero point
  // the group whose operands are being unpacked, and the next slab's
  Group cur, ahead;
  CodeGroup<BITS, BF16> gq[BF];
  uint4 av[2][AF], wf[2][BF];
  pipe_barrier();                         // slab 0 is in LDS, and slab 1 (with XLate only its codes)
  const unsigned char *xsl = smem, *wsl = smem;
  read_group(wsl, 0, cur);
  if (!XLate) read_a(xsl, 0, av[0]);
  int xb = 1, wb = 1, it = 0, sz = sz_at(1);
  const unsigned char *xnext = smem + S::XBytes, *wnext = smem + S::WBytes;
  // Slabs from `it` on.  The usual form of the bfloat16 unpack leaves at the first slab of which a scale asks for the wide form,
  // and the wide form, which is exact for every scale, goes on from there: one test a slab (a branch around the unpack of a
  // step costs 3 % of the whole kernel).
  auto slabs = [&](auto wide_form) {
    constants(wide_form, cur, gq);
    unpack(wide_form, 0, cur, gq, wf[0]);
    int end = nslab;
    while (it < end) {
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const int p = t & 1;
        if (XLate && t == 0) read_a(xsl, 0, av[0]);
        if (Spread && XLate && t == 0) __builtin_amdgcn_sched_barrier(0);   // (what the products of this step wait for)
        if (t + 1 < T || !XLate) read_a(t + 1 < T ? xsl : xnext, (t + 1) % T, av[p ^ 1]);
        if (!Spread) __builtin_amdgcn_sched_barrier(0);   // (activations first: the products wait for them)
        if (t == 0) read_group(wnext, sz, ahead);
        if (!Spread) __builtin_amdgcn_sched_barrier(0);   // (or the compiler moves the reads behind the products to save registers)
        if (t == T - 1) {
          // where the next slab's reads go, here and not behind the barrier (3 % with 64 x 64 tiles)
          xsl = xnext;
          wsl = wnext;
          xb = xb + 1 == NX ? 0 : xb + 1;
          wb = wb + 1 == NW ? 0 : wb + 1;
          xnext = smem + xb * S::XBytes;
          wnext = smem + wb * S::WBytes;
          sz = sz_at(++it + 1);
          cur = ahead;
          if constexpr (BF16 && !decltype(wide_form)::value) end = asks_wide(cur) ? 0 : nslab;
          constants(wide_form, cur, gq);
        }
        unpack(wide_form, (t + 1) % T, cur, gq, wf[p ^ 1]);
#pragma unroll
        for (int b = 0; b < BF; ++b)
#pragma unroll
          for (int f = 0; f < AF; ++f) acc[f][b] = mfma_16x16x32<BF16>(wf[p][b], av[p][f], acc[f][b]);
        // products and unpacking in turns
        constexpr int kVec = (BF * (BITS == 6 ? 20 : 17) + AF * BF - 1) / (AF * BF);
#pragma unroll
        for (int i = 0; i < AF * BF; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);      // matrix instruction
          __builtin_amdgcn_sched_group_barrier(0x002, kVec, 0);   // vector instructions
          if constexpr (Spread) {
            const int reads = (t + 1 < T || !XLate ? AF : 0) + (t == 0 ? BF * kReads : 0), n = (i + 1) * reads / (AF * BF) - i * reads / (AF * BF);
            if (n == 1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // LDS reads
            if (n >= 2) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (BF16 && !decltype(wide_form)::value) {
        // (used here: or the compiler moves the unpack of the next slab's first step behind the barrier and the test)
#pragma unroll
        for (int b = 0; b < BF; ++b) asm volatile("" : "+v"(wf[0][b].x), "+v"(wf[0][b].y), "+v"(wf[0][b].z), "+v"(wf[0][b].w));
        asm volatile("" : "+s"(end));     // (and the selection: 64 tokens x 64 rows, 5 % of the kernel)
      }
      pipe_barrier();                     // slab it + 1 is in LDS (with XLate only its codes, slab it whole), nobody reads slab it - 1 any more
    }
  };
  if (!BF16 || !asks_wide(cur)) slabs(std::false_type());
  if constexpr (BF16) {
    if (__builtin_expect(it < nslab, 0)) slabs(std::true_type());
  }

  // ---- output.  Lane l holds, for fragment (f, b): token l % 16, rows 4 (l / 16) + v.
  auto store = [&](int f, int b, float4_t s) {
    const int tok = m0 + f * 16 + n, rc = n0 + (wn * BF + b) * 16 + 4 * ks;
    if (tok >= a.M || rc >= km.n_keep) return;
    half_t* y = a.y + (size_t)tok * a.ldy + rc;
    uint16_t o[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) o[v] = __builtin_bit_cast(uint16_t, out16<BF16>(s[v]));
    if (rc + 4 <= km.n_keep) {
      typedef uint32_t u32x2_u2 __attribute__((ext_vector_type(2), aligned(2)));
      u32x2_u2 pk;
      pk.x = o[0] | ((uint32_t)o[1] << 16);
      pk.y = o[2] | ((uint32_t)o[3] << 16);
      *reinterpret_cast<u32x2_u2*>(y) = pk;
    } else {
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (rc + v < km.n_keep) y[v] = __builtin_bit_cast(half_t, o[v]);
    }
  };
  // partial sums through LDS (nobody reads or moves slabs any more): fragment q = f BF + b of a row position is added up
  // over the KS waves in order and stored by wave q % KS of them
  float4_t* red = reinterpret_cast<float4_t*>(smem);
#pragma unroll
  for (int f = 0; f < AF; ++f)
#pragma unroll
    for (int b = 0; b < BF; ++b) red[((wk * WN + wn) * AF * BF + f * BF + b) * 64 + lane] = acc[f][b];
  pipe_barrier();
  for (int q = wk; q < AF * BF; q += KS) {
    float4_t s = red[(wn * AF * BF + q) * 64 + lane];
#pragma unroll
    for (int k2 = 1; k2 < KS; ++k2) s += red[((k2 * WN + wn) * AF * BF + q) * 64 + lane];
    store(q / BF, q % BF, s);
  }
