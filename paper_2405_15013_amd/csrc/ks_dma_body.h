// Body of the batch-size-first LDS-DMA kernels (ks_dma.h), included inside
// ks_dma_kernel and ks_dma_klds_kernel, which define KLDS; not a header of its own.
  constexpr int S = sizeof(T);
  constexpr int CH = 4 * LP;  // values of l per stage
  constexpr int PE = STRIDED ? V : (LP * V * S < 16 ? LP * V : 16 / S);
  constexpr int NP = LP * V / PE;
  constexpr int PB = PE * S;
  static_assert(!KLDS || LP * S == 16, "K operands move through LDS as 64-byte rows");
  constexpr int KW = LP * S / 4;  // dwords of a lane's K operand
  using Piece = LdsVec<PB>;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, g = lane >> 4;
  kernarg_fetch(p, t);
  const STile st = dma_tile(t, blockIdx.x);
  const SItem si = dma_item(t, st, V, MT, w);
  DItem it;
  it.i = st.i;
  it.j0 = si.j0;
  it.k0 = si.k0;
  it.beta0 = si.beta0;
  const T* __restrict__ kv = static_cast<const T*>(p.kv);
  const int nst = p.c / CH;
  const int stage = t.stage;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;

  // DMA sources: instruction m of this wavefront fills physical units
  // (m*W + w)*64 + lane; the lane loads the logical unit stored there (rows
  // beyond the batch read the last row instead).
  const T* __restrict__ xi = static_cast<const T*>(p.x) + (int64_t)st.i * p.c * p.d;
  int soff[UD];
#pragma unroll
  for (int m = 0; m < UD; ++m) {
    int r, v;
    dma_unit_of_fast(t, dma_phys_unit(t, m, w, lane), &r, &v);
    int beta = st.bt * 16 * t.RS * NT + r;
    if (beta >= p.batch) beta = p.batch - 1;
    soff[m] = beta * p.N + v * (16 / S);
  }
  const int xstage = CH * p.d;  // X elements per stage along a row
  // DMA of the stage whose row runs start at xs, into stage buffer buf.
  auto dma = [&](const T* xs, int buf) {
    char* dst = smem + buf * stage + w * 1024;
#pragma unroll
    for (int m = 0; m < UD; ++m)
      __builtin_amdgcn_global_load_lds(static_cast<const void*>(xs + soff[m]),
                                       (lds_void_t*)(dst + m * t.W * 1024), 16, 0, 0);
  };

  // Operand pieces of this lane: LDS byte offsets within a stage buffer (row
  // group 0 of the wavefront; group u is 16*u rows further, and the swizzle
  // depends on the row modulo 16 only).
  uint32_t ooff[NP];
  const uint32_t ugroup = 16 * t.UR * 16;  // bytes of 16 stage rows
  {
    const int r = 16 * NT * si.rs + n;
#pragma unroll
    for (int q = 0; q < NP; ++q)
      ooff[q] = lds0 + dma_lds_byte(t, r, dma_op_byte(p, si, LP, V, STRIDED, PE, S, 0, g, q));
  }

  // K operands.  KLDS: DMA instruction (mt, e) moves operand (mt, e) of a
  // stage, the 64-byte runs of its 16 rows, into the wavefront's own LDS
  // buffer; lane i loads the unit that lands in slot i (four lanes per run).
  // Otherwise each lane loads its LP values straight into registers.
  const int64_t kmstride = (int64_t)16 * p.c, kestride = (int64_t)p.b * p.c;
  const T* kl = kv + (KLDS ? direct_k_base(p, it, LP, dma_k_row(lane), dma_k_piece(lane))
                           : direct_k_base(p, it, LP, n, g));
  const int kbuf = dma_stage_buffers(nst) * stage + w * (MT * V * 1024);
  const uint32_t kaddr = lds0 + kbuf + 16 * dma_k_slot(n, g);
  auto kdma = [&](int l) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int e = 0; e < V; ++e)
        __builtin_amdgcn_global_load_lds(static_cast<const void*>(kl + mt * kmstride + e * kestride + l),
                                         (lds_void_t*)(smem + kbuf + (mt * V + e) * 1024), 16, 0, 0);
  };

  f32x4 acc[NT][MT][V];
#pragma unroll
  for (int u = 0; u < NT; ++u)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int e = 0; e < V; ++e) acc[u][mt][e] = f32x4{0.f, 0.f, 0.f, 0.f};

  // One stage.  MODE 2: K of stage s+1 and DMA of stage s+2 (steady state);
  // MODE 1: K of stage s+1 only (stage nst-2); MODE 0: nothing (last stage).
  // The modes are separate straight-line code so that the compiler's own
  // wait before the MFMAs sees a fixed number of operations after each K load.
  // Stage s uses buffer cur = s % 3 (kept incrementally), the DMAs of stage
  // s+2 go to buffer (s+2) % 3 from the row runs at xnext.
  int cur = 0;
  const T* xnext = xi + 2 * xstage;
  u32x4 kf[MT * V];
  auto step = [&](auto mode, int s, DmaK<T, V, MT, LP>& kc, DmaK<T, V, MT, LP>& kn) {
    constexpr int MODE = decltype(mode)::value;
    // 1-2: stage s (and its K) complete in every wavefront; stage s-1 read.
    // (The scheduling barrier keeps the wait from being hoisted into the
    // previous stage's MFMAs.)
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (MODE == 0) wait_vmcnt<0>();
    else wait_vmcnt<UD>();
    dma_barrier();
    const uint32_t base = (uint32_t)(cur * stage);
    const int nbuf = cur == 0 ? 2 : cur - 1;
    cur = cur == 2 ? 0 : cur + 1;
    typename Piece::type pc[NP];
    // 3: K of stage s+1, then the DMAs of stage s+2 (this order is what the
    // count of step 1 relies on).  KLDS: stage s's K operands and the first
    // row group's X operands leave LDS first, because K of stage s+1 goes into
    // the same buffer.
    if constexpr (KLDS) {
#pragma unroll
      for (int f = 0; f < MT * V; ++f) kf[f] = LdsVec<16>::read(kaddr + f * 1024);
#pragma unroll
      for (int q = 0; q < NP; ++q) pc[q] = Piece::read(ooff[q] + base);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
      for (int f = 0; f < MT * V; ++f) {
        asm volatile("" : "+v"(kf[f]));  // ordered after the wait above
#pragma unroll
        for (int w2 = 0; w2 < KW; ++w2) kc.kw[f / V][f % V][w2] = kf[f][w2];
      }
      if constexpr (MODE >= 1) kdma((s + 1) * CH);
    } else {
      if constexpr (MODE >= 1) kn.load(kl, kmstride, kestride, (s + 1) * CH);
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (MODE == 2) {
      dma(xnext, nbuf);
      xnext += xstage;
    }
    __builtin_amdgcn_sched_barrier(0);
    // 4: per row group, operands from LDS, then the MFMAs (the K operands
    // serve all NT groups).
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      if (!KLDS || u > 0) {
#pragma unroll
        for (int q = 0; q < NP; ++q) pc[q] = Piece::read(ooff[q] + base + u * ugroup);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      }
      uint32_t xw[LP * V * S / 4];
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        asm volatile("" : "+v"(pc[q]));  // ordered after the wait above
#pragma unroll
        for (int w2 = 0; w2 < PB / 4; ++w2) xw[q * (PB / 4) + w2] = pc[q][w2];
      }
      direct_mma<T, BSF, V, MT, LP>(xw, kc.kw, acc[u]);
    }
  };
  using M0 = std::integral_constant<int, 0>;
  using M1 = std::integral_constant<int, 1>;
  using M2 = std::integral_constant<int, 2>;

  DmaK<T, V, MT, LP> ka, kb;
  if constexpr (KLDS) kdma(0);
  else ka.load(kl, kmstride, kestride, 0);
  __builtin_amdgcn_sched_barrier(0);
  dma(xi, 0);
  if (nst > 1) dma(xi + xstage, 1);
  __builtin_amdgcn_sched_barrier(0);
  int s = 0;
  for (; s + 3 < nst; s += 2) {  // both steps are steady-state steps
    step(M2(), s, ka, kb);
    step(M2(), s + 1, kb, ka);
  }
  // The last 1-3 stages (s even, so ka holds K of stage s).
  const int left = nst - s;
  if (left == 3) {
    step(M2(), s, ka, kb);
    step(M1(), s + 1, kb, ka);
    step(M0(), s + 2, ka, kb);
  } else if (left == 2) {
    step(M1(), s, ka, kb);
    step(M0(), s + 1, kb, ka);
  } else {
    step(M0(), s, ka, kb);
  }

  // Structured epilogue: accumulators -> LDS output tile -> contiguous runs.
  // Bias of output feature (mt, e, r4) = row k0 + 16 mt + 4 g + r4 of block
  // (i, j0 + e), shared by the NT row groups; loads issued before the wait
  // for the last MFMA results.
  const bool has_bias = p.bias != nullptr;
  float bv[MT][V][4];
  if (has_bias) {
    const T* bb = static_cast<const T*>(p.bias) + (int64_t)(st.i * p.b + it.k0 + 4 * g) * p.d + it.j0;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4)
#pragma unroll
        for (int e = 0; e < V; ++e) bv[mt][e][r4] = to_f32(bb[(16 * mt + r4) * p.d + e]);
  }
  mfma_results_settle();
  if (has_bias) {
#pragma unroll
    for (int u = 0; u < NT; ++u)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int e = 0; e < V; ++e)
#pragma unroll
          for (int r4 = 0; r4 < 4; ++r4) acc[u][mt][e][r4] += bv[mt][e][r4];
  }
  if (epilogue_gelu(p)) {
#pragma unroll
    for (int u = 0; u < NT; ++u)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int e = 0; e < V; ++e)
#pragma unroll
          for (int r4 = 0; r4 < 4; ++r4) acc[u][mt][e][r4] = gelu_f32<T>(acc[u][mt][e][r4]);
  }
  __syncthreads();  // every wavefront is done with the stage buffers
  char* ycell0 = smem + dma_y_lds_lane(p, t, si, MT, S, n, g);
#pragma unroll
  for (int u = 0; u < NT; ++u)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        // V consecutive j of output row k = k0 + 16*mt + 4*g + r4
        char* cell = ycell0 + u * 16 * t.ypitch + (16 * mt + r4) * p.d * S;
        if constexpr (V == 4) {
          if constexpr (S == 4) {
            *reinterpret_cast<f32x4*>(cell) =
                f32x4{acc[u][mt][0][r4], acc[u][mt][1][r4], acc[u][mt][2][r4], acc[u][mt][3][r4]};
          } else {
            uint32_t wv[2];
#pragma unroll
            for (int e = 0; e < V; e += 2) {
              wv[e / 2] = pack2_f32<T>(acc[u][mt][e][r4], acc[u][mt][e + 1][r4]);
            }
            *reinterpret_cast<u32x2*>(cell) = u32x2{wv[0], wv[1]};
          }
        } else {
#pragma unroll
          for (int e = 0; e < V; ++e) reinterpret_cast<T*>(cell)[e] = from_f32<T>(acc[u][mt][e][r4]);
        }
      }
  __syncthreads();
  // 16-byte units of the output tile (uy = 2^lUY per row): rows beyond the
  // batch are not stored.
  const int nunits = (16 * t.RS * NT) << t.lUY;
  const int rows_valid = p.batch - st.bt * 16 * t.RS * NT;
  T* __restrict__ ytile = static_cast<T*>(p.y) + dma_y_tile_base(p, t, st, MT);
  for (int u = tid; u < nunits; u += 64 * t.W) {
    const int row = u >> t.lUY, v = u & ((1 << t.lUY) - 1);
    if (row >= rows_valid) continue;
    const u32x4 val = *reinterpret_cast<const u32x4*>(smem + row * t.ypitch + v * 16);
    __builtin_nontemporal_store(val, reinterpret_cast<u32x4*>(ytile + dma_y_row(p, row, v, S)));
  }
