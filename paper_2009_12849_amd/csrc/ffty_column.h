  // The transform of column m of level k by its threads q (part: false only takes
  // part in the barriers); column c of mt in LDS. Included by the kernel and by
  // the level kernels: as a function of its own the compiler orders its loads
  // otherwise and the FP64 kernel at 2048 or the FP32 one at 432 is 5 % slower.
  const bool valid = part && m < d.nxh;
  cx<T>* S = reinterpret_cast<cx<T>*>(io.spec) + (long long)k * d.plane + spec_col(d, valid ? m : 0);
  const int rs = d.sbw;  // row stride inside a column block
  cx<T> v[F::VMAX];
  // FP32: unconditional loads (an invalid column reads column 0), zeroed
  // after; FP64 keeps the guarded loads, which measure faster there
#pragma unroll
  for (int t = 0; t < F::BT0; ++t) {
    const int b = q + t * NT;
    if (F::valid_first(b)) {
#pragma unroll
      for (int r = 0; r < F::R0; ++r) {
        if constexpr (sizeof(T) == 4) {
          const cx<T> x = S[(b + r * F::NB0) * rs];
          v[t * F::R0 + r] = valid ? x : cx<T>{0, 0};
        } else {
          v[t * F::R0 + r] = valid ? S[(b + r * F::NB0) * rs] : cx<T>{0, 0};
        }
      }
    }
  }
  auto li = [mt, c](int i) { return i * mt + c; };
  F::run(v, lds, li, q, reinterpret_cast<const cx<T>*>(d.twy));
  if (valid) {
#pragma unroll
    for (int t = 0; t < F::BTL; ++t) {
      const int b = q + t * NT;
      if (F::valid_last(b)) {
#pragma unroll
        for (int r = 0; r < F::RL; ++r) S[F::out_index(q, t, r) * rs] = v[t * F::RL + r];
      }
    }
  }
