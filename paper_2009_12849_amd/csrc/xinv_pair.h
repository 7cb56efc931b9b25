  // The inverse transform of the row pair `pair` by its threads q, with its part of
  // the LDS at lds (part: false only takes part in the barriers). Included by the
  // kernel and by the level kernel: as a function of its own the compiler orders
  // its loads otherwise and the FP64 kernel at 512 or 2048 is 7-10 % slower.
  const long long r0 = 2 * pair, r1 = 2 * pair + 1;
  const bool v0 = part && r0 < d.nrow, v1 = part && r1 < d.nrow;
  const cx<T>* S = reinterpret_cast<const cx<T>*>(io.spec);
  auto li = [](int i) { return xpad<T, N>(i); };
  if (sizeof(T) == 4 && d.sbw >= 2) {
    // FP32 with column blocks at least 2 wide: bins m, m+1 (m even) of a row
    // are adjacent and 16-byte aligned in memory, so a lane loads both with
    // one access (half the load instructions). Pairs m = 0, 2, .. up to nx/2
    // over NT threads. Where nx/2 is even the slot after bin nx/2 is read and
    // dropped (nx/2 + 1 is then odd and the padded row length a multiple of 8,
    // so it is a padding slot of the row's last block). Loads first and
    // unconditional, as below.
    typedef T t4 __attribute__((ext_vector_type(4)));
    constexpr int NP = N / 4 + 1;  // pairs (m even, m <= N/2)
    constexpr int RND2 = (NP + NT - 1) / NT;
    const long long so0 = spec_row(d, v0 ? r0 : 0), so1 = spec_row(d, v1 ? r1 : 0);
    t4 ya[RND2], yb[RND2];
#pragma unroll
    for (int t = 0; t < RND2; ++t) {
      const int m = 2 * (q + t * NT);
      const bool in = m <= N / 2;
      const long long cm = spec_col(d, in ? m : 0);
      const t4 a = *reinterpret_cast<const t4*>(S + so0 + cm), b = *reinterpret_cast<const t4*>(S + so1 + cm);
      ya[t] = (in && v0) ? a : (t4)(T)0;
      yb[t] = (in && v1) ? b : (t4)(T)0;
    }
#pragma unroll
    for (int t = 0; t < RND2; ++t) {
      const int m = 2 * (q + t * NT);
      if (m <= N / 2) {
        pack_bins<T>(lds, li, cx<T>{ya[t][0], ya[t][1]}, cx<T>{yb[t][0], yb[t][1]}, N, m);
        if (m + 1 <= N / 2) pack_bins<T>(lds, li, cx<T>{ya[t][2], ya[t][3]}, cx<T>{yb[t][2], yb[t][3]}, N, m + 1);
      }
    }
  } else {
    // nx/2 + 1 bins over NT threads: N/(2 NT) + 1 rounds, loads issued first
    // and unconditional (clamped bin; a missing row reads row 0), selected after
    constexpr int RND = N / (2 * NT) + 1;
    const long long so0 = spec_row(d, v0 ? r0 : 0), so1 = spec_row(d, v1 ? r1 : 0);
    cx<T> xa[RND], xb[RND];
#pragma unroll
    for (int t = 0; t < RND; ++t) {
      const int m = q + t * NT;
      const bool in = m <= N / 2;
      const long long cm = spec_col(d, in ? m : N / 2);
      const cx<T> a = S[so0 + cm], b = S[so1 + cm];
      xa[t] = (in && v0) ? a : cx<T>{0, 0};
      xb[t] = (in && v1) ? b : cx<T>{0, 0};
    }
#pragma unroll
    for (int t = 0; t < RND; ++t) {
      const int m = q + t * NT;
      if (m <= N / 2) pack_bins<T>(lds, li, xa[t], xb[t], N, m);
    }
  }
  __syncthreads();
  cx<T> v[F::VMAX];
#pragma unroll
  for (int t = 0; t < F::BT0; ++t) {
    const int b = q + t * NT;
    if (F::valid_first(b)) {
#pragma unroll
      for (int r = 0; r < F::R0; ++r) v[t * F::R0 + r] = lds[xpad<T, N>(b + r * F::NB0)];
    }
  }
  __syncthreads();
  F::run(v, lds, li, q, reinterpret_cast<const cx<T>*>(d.twx));
#pragma unroll
  for (int t = 0; t < F::BTL; ++t) {
    const int b = q + t * NT;
    if (F::valid_last(b)) {
#pragma unroll
      for (int r = 0; r < F::RL; ++r) lds[xpad<T, N>(F::out_index(q, t, r))] = v[t * F::RL + r];
    }
  }
  __syncthreads();
  // vector phase: chunks of V points of both rows
  constexpr int V = x_chunk(N, sizeof(T)), NCH = N / V;
  using vt = typename Vec<T, V>::type;
  auto p = reinterpret_cast<__attribute__((address_space(1))) vt*>(xinv_dest<T, MODE>(io));
  double dz0 = 0.0, dz1 = 0.0, rz = 0.0, zq = 0.0;  // MODE 3
  if constexpr (MODE == 3) {
    dz0 = ldg(d.dz + row_level(d, v0 ? (int)r0 : 0));
    dz1 = ldg(d.dz + row_level(d, v1 ? (int)r1 : 0));
  }
#pragma unroll
  for (int t = 0; t < (NCH + NT - 1) / NT; ++t) {
    const int ch = q + t * NT;
    if (NCH % NT == 0 || ch < NCH) {
      vt a0, a1;
#pragma unroll
      for (int e = 0; e < V; ++e) {
        const cx<T> z = lds[xpad<T, N>(ch * V + e)];
        a0[e] = z.x;
        a1[e] = z.y;
      }
      if (v0) p[r0 * NCH + ch] = a0;
      if (v1) p[r1 * NCH + ch] = a1;
      if constexpr (MODE == 3) {
        if (v0) dots_vec<T, V>(io, r0 * N + ch * V, reinterpret_cast<const T*>(&a0), dz0, rz, zq);
        if (v1) dots_vec<T, V>(io, r1 * N + ch * V, reinterpret_cast<const T*>(&a1), dz1, rz, zq);
      }
    }
  }
