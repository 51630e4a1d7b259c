// Column kernels for grids with few columns: tiles of CT columns kept whole in LDS.
//
// The streaming column kernels (one thread per column) are bound by the latency of one exposed memory
// access per row step: below about two waves per SIMD a step takes ~0.7 us, whatever it computes.  Here a
// block of 8 waves brings all rows of its CT columns to LDS at once (loads straight to LDS, all in flight
// together), one wave runs the sweeps there, the other waves stream the factors of A(k) to LDS ahead of
// it, and all waves evaluate the banded products at tau in parallel over the rows.  The intermediates of
// the sweeps never leave the CU.
//
// Lanes.  A lane owns a real column: every operator of the sweeps is real, so the real and imaginary parts
// of a column are two lanes.  S[row][lane] has RS = 2 CT lanes per row.  Flat tiles hold CT consecutive
// columns; pair tiles (A(k) solves) hold CT/2 pairs (l, +-n), lanes 0 .. CT-1 the columns +n, lanes
// CT .. 2 CT-1 the columns -n.  With RS < 64 a wave works on 64 / RS rows at once outside the sweeps.
//
// Tables.  The banded rows of a sweep or product are the same for all lanes.  Lane n of every 16 holds the
// entries of row n of a block of 16 rows, read with a few wide loads per block; v_fmac_f64 takes them from
// there with a row broadcast (DPP row_newbcast), so a table entry costs neither an LDS read nor a scalar
// load per row.  Measured (129 rows, one wave): a step of the L sweep takes 64 cycles against 106 with the
// rows read from LDS, 36-50 of them the dependent chain.
#pragma once

constexpr int kTileWaves = 8, kTileThreads = 64 * kTileWaves;
// a += sum_k t_k(lane N of the lane's 16) x_k.  Wait states: the table registers may have been written by a
// vector instruction just before.  The sums of these blocks are written before the last operand is read, so they are
// early-clobber: else one may share its register with an operand of the same value (two zeros, say).
#define LMVD_FB(a, t, x) "v_fmac_f64_dpp " a ", " t ", " x " row_newbcast:%[n] row_mask:0xf bank_mask:0xf\n\t"
template <int N>
__device__ __forceinline__ void fb8(double& a, const double* t, const double* x) {
  asm("s_nop 1\n\t" LMVD_FB("%0", "%8", "%16") LMVD_FB("%0", "%7", "%15") LMVD_FB("%0", "%6", "%14")
      LMVD_FB("%0", "%5", "%13") LMVD_FB("%0", "%4", "%12") LMVD_FB("%0", "%3", "%11") LMVD_FB("%0", "%2", "%10")
      LMVD_FB("%0", "%1", "%9")
      : "+&v"(a)
      : "v"(t[0]), "v"(t[1]), "v"(t[2]), "v"(t[3]), "v"(t[4]), "v"(t[5]), "v"(t[6]), "v"(t[7]), "v"(x[0]), "v"(x[1]),
        "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]), "v"(x[6]), "v"(x[7]), [n] "n"(N));
}
template <int N>
__device__ __forceinline__ void fb12(double& a, const double* t, const double* x) {
  asm("s_nop 1\n\t" LMVD_FB("%0", "%1", "%13") LMVD_FB("%0", "%2", "%14") LMVD_FB("%0", "%3", "%15")
      LMVD_FB("%0", "%4", "%16") LMVD_FB("%0", "%5", "%17") LMVD_FB("%0", "%6", "%18") LMVD_FB("%0", "%7", "%19")
      LMVD_FB("%0", "%8", "%20") LMVD_FB("%0", "%9", "%21") LMVD_FB("%0", "%10", "%22") LMVD_FB("%0", "%11", "%23")
      LMVD_FB("%0", "%12", "%24")
      : "+&v"(a)
      : "v"(t[0]), "v"(t[1]), "v"(t[2]), "v"(t[3]), "v"(t[4]), "v"(t[5]), "v"(t[6]), "v"(t[7]), "v"(t[8]), "v"(t[9]),
        "v"(t[10]), "v"(t[11]), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]), "v"(x[6]), "v"(x[7]),
        "v"(x[8]), "v"(x[9]), "v"(x[10]), "v"(x[11]), [n] "n"(N));
}
// two and three sums over the same 4 (5) values, interleaved
template <int N>
__device__ __forceinline__ void fb2x4(double& a, double& b, const double* t, const double* u, const double* x) {
  asm("s_nop 1\n\t" LMVD_FB("%0", "%2", "%10") LMVD_FB("%1", "%6", "%10") LMVD_FB("%0", "%3", "%11")
      LMVD_FB("%1", "%7", "%11") LMVD_FB("%0", "%4", "%12") LMVD_FB("%1", "%8", "%12") LMVD_FB("%0", "%5", "%13")
      LMVD_FB("%1", "%9", "%13")
      : "+&v"(a), "+&v"(b)
      : "v"(t[0]), "v"(t[1]), "v"(t[2]), "v"(t[3]), "v"(u[0]), "v"(u[1]), "v"(u[2]), "v"(u[3]), "v"(x[0]), "v"(x[1]),
        "v"(x[2]), "v"(x[3]), [n] "n"(N));
}
template <int N>
__device__ __forceinline__ void fb3x4(double& a, double& b, double& c, const double* t, const double* u,
                                      const double* v, const double* x) {
  asm("s_nop 1\n\t" LMVD_FB("%0", "%3", "%15") LMVD_FB("%1", "%7", "%15") LMVD_FB("%2", "%11", "%15")
      LMVD_FB("%0", "%4", "%16") LMVD_FB("%1", "%8", "%16") LMVD_FB("%2", "%12", "%16")
      LMVD_FB("%0", "%5", "%17") LMVD_FB("%1", "%9", "%17") LMVD_FB("%2", "%13", "%17")
      LMVD_FB("%0", "%6", "%18") LMVD_FB("%1", "%10", "%18") LMVD_FB("%2", "%14", "%18")
      : "+&v"(a), "+&v"(b), "+&v"(c)
      : "v"(t[0]), "v"(t[1]), "v"(t[2]), "v"(t[3]), "v"(u[0]), "v"(u[1]), "v"(u[2]), "v"(u[3]), "v"(v[0]), "v"(v[1]),
        "v"(v[2]), "v"(v[3]), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), [n] "n"(N));
}
template <int N>
__device__ __forceinline__ void fb2x5(double& a, double& b, const double* t, const double* u, const double* x) {
  asm("s_nop 1\n\t" LMVD_FB("%0", "%2", "%12") LMVD_FB("%1", "%7", "%12") LMVD_FB("%0", "%3", "%13")
      LMVD_FB("%1", "%8", "%13") LMVD_FB("%0", "%4", "%14") LMVD_FB("%1", "%9", "%14") LMVD_FB("%0", "%5", "%15")
      LMVD_FB("%1", "%10", "%15") LMVD_FB("%0", "%6", "%16") LMVD_FB("%1", "%11", "%16")
      : "+&v"(a), "+&v"(b)
      : "v"(t[0]), "v"(t[1]), "v"(t[2]), "v"(t[3]), "v"(t[4]), "v"(u[0]), "v"(u[1]), "v"(u[2]), "v"(u[3]), "v"(u[4]),
        "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), [n] "n"(N));
}
// Four rows N .. N+3 of an L sweep (v: their right-hand sides, then their solutions; y: the six before them,
// the newest first): v_fmac_f64 issues every five cycles and its result is there for the next, so the chain
// costs nothing over the issue.
template <int N>
__device__ __forceinline__ void fb_l4(double* v, const double* t, const double* y) {
  asm("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %9, %15 row_newbcast:%[n0] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %8, %14 row_newbcast:%[n0] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %7, %13 row_newbcast:%[n0] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %6, %12 row_newbcast:%[n0] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %5, %11 row_newbcast:%[n0] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %4, %10 row_newbcast:%[n0] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %9, %14 row_newbcast:%[n1] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %8, %13 row_newbcast:%[n1] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %7, %12 row_newbcast:%[n1] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %6, %11 row_newbcast:%[n1] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %5, %10 row_newbcast:%[n1] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %4, %0 row_newbcast:%[n1] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %9, %13 row_newbcast:%[n2] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %8, %12 row_newbcast:%[n2] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %7, %11 row_newbcast:%[n2] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %6, %10 row_newbcast:%[n2] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %5, %0 row_newbcast:%[n2] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %4, %1 row_newbcast:%[n2] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %9, %12 row_newbcast:%[n3] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %8, %11 row_newbcast:%[n3] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %7, %10 row_newbcast:%[n3] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %6, %0 row_newbcast:%[n3] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %5, %1 row_newbcast:%[n3] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %4, %2 row_newbcast:%[n3] row_mask:0xf bank_mask:0xf\n\t"
      : "+&v"(v[0]), "+&v"(v[1]), "+&v"(v[2]), "+&v"(v[3])
      : "v"(t[0]), "v"(t[1]), "v"(t[2]), "v"(t[3]), "v"(t[4]), "v"(t[5]),
        "v"(y[0]), "v"(y[1]), "v"(y[2]), "v"(y[3]), "v"(y[4]), "v"(y[5]),
        [n0] "n"(N), [n1] "n"(N + 1), [n2] "n"(N + 2), [n3] "n"(N + 3));
}
// four rows N, N-1, N-2, N-3 of a U sweep: z = v times the inverse pivot t[6]
template <int N>
__device__ __forceinline__ void fb_u4(double* v, double* z, const double* t, const double* x) {
  asm("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %13, %20 row_newbcast:%[n0] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %12, %19 row_newbcast:%[n0] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %11, %18 row_newbcast:%[n0] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %10, %17 row_newbcast:%[n0] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %9, %16 row_newbcast:%[n0] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %8, %15 row_newbcast:%[n0] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %4, %14, %0 row_newbcast:%[n0] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %13, %19 row_newbcast:%[n1] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %12, %18 row_newbcast:%[n1] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %11, %17 row_newbcast:%[n1] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %10, %16 row_newbcast:%[n1] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %9, %15 row_newbcast:%[n1] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %8, %4 row_newbcast:%[n1] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %5, %14, %1 row_newbcast:%[n1] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %13, %18 row_newbcast:%[n2] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %12, %17 row_newbcast:%[n2] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %11, %16 row_newbcast:%[n2] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %10, %15 row_newbcast:%[n2] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %9, %4 row_newbcast:%[n2] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %8, %5 row_newbcast:%[n2] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %6, %14, %2 row_newbcast:%[n2] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %13, %17 row_newbcast:%[n3] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %12, %16 row_newbcast:%[n3] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %11, %15 row_newbcast:%[n3] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %10, %4 row_newbcast:%[n3] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %9, %5 row_newbcast:%[n3] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %8, %6 row_newbcast:%[n3] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %7, %14, %3 row_newbcast:%[n3] row_mask:0xf bank_mask:0xf\n\t"
      : "+&v"(v[0]), "+&v"(v[1]), "+&v"(v[2]), "+&v"(v[3]), "+&v"(z[0]), "+&v"(z[1]), "+&v"(z[2]), "+&v"(z[3])
      : "v"(t[0]), "v"(t[1]), "v"(t[2]), "v"(t[3]), "v"(t[4]), "v"(t[5]), "v"(t[6]),
        "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]),
        [n0] "n"(N), [n1] "n"(N - 1), [n2] "n"(N - 2), [n3] "n"(N - 3));
}
template <int I, int E, class F>
__device__ __forceinline__ void unrolled(F&& f) {
  if constexpr (I < E) {
    f(std::integral_constant<int, I>{});
    unrolled<I + 1, E>(f);
  }
}

__device__ __forceinline__ double swap_ri(double v) {  // the other part of the lane's complex column
  union { double d; int i[2]; } a;
  a.d = v;
  a.i[0] = __builtin_amdgcn_mov_dpp(a.i[0], 0xB1, 0xf, 0xf, true);
  a.i[1] = __builtin_amdgcn_mov_dpp(a.i[1], 0xB1, 0xf, 0xf, true);
  return a.d;
}
// the lane's part of i z
__device__ __forceinline__ double times_i_lane(double v, int c) {
  const double o = swap_ri(v);
  return c ? o : -o;
}
// lane N of the lane's 16
template <int N>
__device__ __forceinline__ int bcast16(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x150 + N, 0xf, 0xf, false);
}
__device__ __forceinline__ int tile_wave() { return __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6); }

// Byte offsets are 32-bit: a plan with tiles has fields below 2^32 bytes.
struct TileLane {
  bool act;      // the lane owns a column
  bool mean;     // ... the plane mean
  int c;         // 0 real, 1 imaginary part
  unsigned off;  // of its element in a row
  unsigned rs;   // bytes per row of a spectral field
  unsigned doff; // offset of the column that the lane fetches for the tile
  double k1, k3;
};
template <int CT, bool PAIR>
__device__ __forceinline__ TileLane tile_lane(const DevPlan& P, unsigned tile, int lane) {
  TileLane L;
  const unsigned nl = P.nl, nn = P.nn, ncol = nn * nl;
  // column j of the tile: whether there is one, and its number
  auto column = [&](unsigned j, unsigned& col) {
    if constexpr (PAIR) {
      const unsigned npairs = nl * ((nn + 1) / 2), side = j / (CT / 2), pr = tile * (CT / 2) + j % (CT / 2), pp = pr / nl;
      col = (side ? nn - pp : pp) * nl + (pr - pp * nl);
      return pr < npairs && !(side == 1 && pp == 0);
    } else {
      col = tile * CT + j;
      return col < ncol;
    }
  };
  unsigned col, dcol;
  L.act = column((lane >> 1) & (CT - 1), col);
  if (!column(lane & (CT - 1), dcol)) dcol = 0;
  if (!L.act) col = 0;
  L.c = lane & 1;
  L.off = 16 * col + 8 * L.c;
  L.rs = 16 * ncol;
  L.doff = 16 * dcol;
  const unsigned n = col / nl;
  L.k1 = P.k1[col - n * nl];
  L.k3 = P.k3[n];
  L.mean = L.act && col == 0;
  return L;
}
// A field as a buffer: loads past its end give 0 and stores there are dropped, so that a store needs no branch
// around it.  (Behind a branch the compiler cannot count the stores in flight and waits for all of them to
// complete before it uses the next load: ~2 us for every group of rows.)
struct TileBuf {
  __amdgpu_buffer_rsrc_t r;
};
constexpr unsigned kNoStore = 0xfffffff0u;
__device__ __forceinline__ TileBuf tile_buf(const void* p, unsigned bytes) {
  return {__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, p ? bytes : 0u, 0x00020000)};
}
typedef int tile_v2i __attribute__((ext_vector_type(2)));
__device__ __forceinline__ double gld(const TileBuf& b, unsigned byte) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(b.r, byte, 0, 0));
}
__device__ __forceinline__ void gst(const TileBuf& b, unsigned byte, double v) {
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(tile_v2i, v), b.r, byte, 0, 0);
}

__device__ __forceinline__ void lds_fetch16(const void* g, double* l) {  // 16 bytes per lane to l + 2 lane
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                   (__attribute__((address_space(3))) void*)l, 16, 0, 0);
}
__device__ __forceinline__ void lds_fetched() {  // all fetches of the block have arrived
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
}
// barrier for LDS traffic only: fetches in flight stay in flight (__syncthreads would wait for them)
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
// rows 0 .. rows-1 of the tile's columns -> S, up to the padded row count with copies of the last row (asynchronous:
// lds_fetched).  The U sweep passes through the padding rows, and 0 times what is not finite there would reach every
// row: REPLACED, where the last row may be a wall value that the projection replaces, they are copies of the row before.
template <int CT, bool REPLACED = false>
__device__ __forceinline__ void tile_fetch(double* S, const double* src, const TileLane& L, int rows, int w, int lane) {
  constexpr int RPI = 64 / CT;  // rows of one instruction
  const int padded = pad16(rows);
  const unsigned last = L.doff + unsigned(rows - 1) * L.rs, step = kTileWaves * RPI * L.rs;
  unsigned o = L.doff + unsigned(w * RPI + lane / CT) * L.rs;
  int r = w * RPI;
  auto fetch = [&](unsigned at) { lds_fetch16(reinterpret_cast<const char*>(src) + at, S + r * (2 * CT)); };
  if (REPLACED)
    for (; r + RPI <= rows; r += kTileWaves * RPI, o += step) fetch(o);
  for (; r < padded; r += kTileWaves * RPI, o += step) fetch(REPLACED && o > last ? last - L.rs : min(o, last));
}

// The rows that a lane works on outside the sweeps: slot w * 64 / RS + lane / RS of SLOTS owns R rows from r0
// on.  They are worked on four at a time, without branches inside, so that the LDS reads and the chains of
// four rows overlap; rows past the slot's are computed and not stored.
template <int CT>
struct TileRows {
  static constexpr int RS = 2 * CT, SLOTS = kTileWaves * (64 / RS);
  int n, R, r0;
  unsigned o0, last;  // byte offset of the first row's element and of the last row's
  unsigned rs;
  bool act;
  __device__ __forceinline__ TileRows(int n_, const TileLane& L, int w, int lane) : n(n_), R((n_ + SLOTS - 1) / SLOTS) {
    r0 = (w * (64 / RS) + lane / RS) * R;
    rs = L.rs;
    act = L.act;
    o0 = L.off + unsigned(r0) * rs;
    last = L.off + unsigned(n - 1) * rs;
  }
  __device__ __forceinline__ unsigned at(int k) const { return min(o0 + unsigned(k) * rs, last); }
  __device__ __forceinline__ bool own(int k) const { return k < R && r0 + k < n; }
  __device__ __forceinline__ unsigned st(int k) const { return act && own(k) ? o0 + unsigned(k) * rs : kNoStore; }
  // row r0 + k of a column in LDS to write to; rows that the slot does not own go to a spare row (behind a branch the
  // rows of a group would be worked on one after the other)
  __device__ __forceinline__ double* put(double* s, int k, double* spare) const {
    return own(k) ? s + (r0 + k) * RS : spare;
  }
  // row of the table that the lane holds for rows k .. k+M-1
  template <int M>
  __device__ __forceinline__ int tab(int k, int lane) const { return min(r0 + k + (lane & (M - 1)), n - 1); }
};
// groups of four rows: work(k, d) with d = load(k) read one group ahead
template <class Load, class Work>
__device__ __forceinline__ void tile_groups(int R, Load&& load, Work&& work) {
  auto cur = load(0);
  for (int k = 0; k < R; k += 4) {
    const auto nxt = load(k + 4 < R ? k + 4 : k);
    work(k, cur);
    cur = nxt;
  }
}
template <int K>
__device__ __forceinline__ void load_row(double (&t)[K], const double* p) {
#pragma unroll
  for (int q = 0; q < K; q += 2) {
    const double2 v = *reinterpret_cast<const double2*>(p + q);
    t[q] = v.x;
    if (q + 1 < K) t[q + 1] = v.y;
  }
}
// a row of a table in global memory (in its address space: through a generic pointer, as one read from a plan in
// memory is, it would be a flat load, which waits with the LDS traffic)
template <int K>
__device__ __forceinline__ void load_row(double (&t)[K], cptr<double> p) {
  using v2 = double __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int q = 0; q < K; q += 2) {
    const v2 v = *(const __attribute__((address_space(4))) v2*)(p + q);
    t[q] = v.x;
    if (q + 1 < K) t[q + 1] = v.y;
  }
}
// taps of a row of 16 in the lane's slot, from the row number that lane N holds
template <int N, int K, int RS>
__device__ __forceinline__ void tile_taps(double (&v)[K], const double* s, int lo) {
  const double* p = s + bcast16<N>(lo) * RS;
#pragma unroll
  for (int q = 0; q < K; ++q) v[q] = p[q * RS];
}

// The projection tables of a kind in LDS: L rows [kTLRow], then U rows [kTURow], pad16(n2) of each
__host__ __device__ constexpr size_t tile_tab_bytes(int n2) {
  return (size_t(pad16(n2)) * (kTLRow + kTURow) * 8 + 1023) / 1024 * 1024;
}
__device__ __forceinline__ void tile_fetch_tables(const TileTab& T, int kind, double* tab, int n2, int w, int lane) {
  const char* src = reinterpret_cast<const char*>(T.lu[kind]);
  for (unsigned o = 1024 * w; o < tile_tab_bytes(n2); o += 1024 * kTileWaves)
    lds_fetch16(src + o + 16 * lane, tab + o / 8);
}
// L sweep of a column in LDS (s: its row 0) over pad16(n2) rows, in place
template <int RS>
__device__ __forceinline__ void tile_lsweep(double* s, const double* tab, int n2, int lane) {
  double y[kTB], nt[kTLRow];
#pragma unroll
  for (int m = 0; m < kTB; ++m) y[m] = 0.0;
  const int blocks = pad16(n2) / 16;
  tab += (lane & 15) * kTLRow;
  load_row(nt, tab);
  for (int b = 0; b < blocks; ++b) {
    double t[kTLRow];
#pragma unroll
    for (int m = 0; m < kTLRow; ++m) t[m] = nt[m];
    double v[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = s[r * RS];
    if (b + 1 < blocks) tab += 16 * kTLRow;
    load_row(nt, tab);
    unrolled<0, 4>([&](auto nc) __attribute__((always_inline)) {
      constexpr int N = 4 * decltype(nc)::value;
      fb_l4<N>(v + N, t, y);
      y[5] = y[1];
      y[4] = y[0];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        y[3 - r] = v[N + r];
        s[(N + r) * RS] = v[N + r];
      }
    });
    s += 16 * RS;
  }
}
// U sweep, rows pad16(n2)-1 .. 0 in place (the padding rows have inverse pivot 0)
template <int RS>
__device__ __forceinline__ void tile_usweep(double* s, const double* tab, int n2, int lane) {
  double x[kTB], nt[kTURow];
#pragma unroll
  for (int m = 0; m < kTB; ++m) x[m] = 0.0;
  const int blocks = pad16(n2) / 16;
  tab += ((blocks - 1) * 16 + (lane & 15)) * kTURow;
  load_row(nt, tab);
  s += (blocks - 1) * 16 * RS;
  for (int b = blocks - 1; b >= 0; --b) {
    double t[kTURow];
#pragma unroll
    for (int m = 0; m < kTURow; ++m) t[m] = nt[m];
    double v[16];  // descending
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = s[(15 - r) * RS];
    if (b > 0) tab -= 16 * kTURow;
    load_row(nt, tab);
    unrolled<0, 4>([&](auto nc) __attribute__((always_inline)) {
      constexpr int M = 4 * decltype(nc)::value, N = 15 - M;
      double z[4] = {0.0, 0.0, 0.0, 0.0};
      fb_u4<N>(v + M, z, t, x);
      x[5] = x[1];
      x[4] = x[0];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        x[3 - r] = z[r];
        s[(N - r) * RS] = z[r];
      }
    });
    s -= 16 * RS;
  }
}
// both, of the columns whose row 0 is s
template <int RS>
__device__ __forceinline__ void tile_solve(double* s, const double* tab, int n2, int lane) {
  tile_lsweep<RS>(s, tab, n2, lane);
  tile_usweep<RS>(s, tab + pad16(n2) * kTLRow, n2, lane);
}

// ---------------------------------------------------------------------------
// A(k) c = r of a pair tile in LDS: bottom-up forward sweep (rows n2-1 .. 0; row n2 is given), ascending
// back substitution, by wave 0.  The other waves stream the packed factors to LDS, one chunk ahead.  Entries of a
// row: kTIn multipliers (forward) or kTIn entries and the inverse pivot (back) where no more are nonzero, else 8.
// Bound by the dependent chain of the two sweeps and their LDS reads: ~150 cycles per row and sweep pair of 129
// rows 39.8k of the 97k cycles of an m^c tile.
template <int CT>
struct TileSolveA {
  static constexpr int RS = 2 * CT, TP = CT / 2;
  static constexpr int LPS = TP / 2;                       // lanes that fetch a slot
  static constexpr int SPI = 64 / LPS;                     // slots of one instruction
  static constexpr int FPW = ((kTChunk + SPI - 1) / SPI + kTileWaves - 2) / (kTileWaves - 1);  // fetches of a wave per chunk
  static constexpr int BUF = (kTChunk + SPI - 1) / SPI * SPI * TP;  // doubles
  static constexpr size_t LDS = size_t(kTBufs) * BUF * 8;
  double* buf;
  const double* src;  // the lane's place in the tile's factors
  int h;              // helper wave, -1: sweeping
  __device__ __forceinline__ void init(const TileTab& T, double* lds, unsigned tile, int w, int lane) {
    buf = lds;
    h = w - 1;
    const int per = kTGroup / TP;  // tiles of a group
    src = T.fac + (size_t(tile / per) * T.slots + h * SPI + lane / LPS) * kTGroup + (tile % per) * TP + (lane % LPS) * 2;
  }
  __device__ __forceinline__ void fetch(const TileTab& T, int q) const {
    if (q >= T.nchunk) return;
    const double* g = src + size_t(T.chunk[4 * q + 3]) * kTGroup;
    double* l = buf + (q % kTBufs) * BUF;
#pragma unroll
    for (int u = 0; u < FPW; ++u) {
      const int s = (h + u * (kTileWaves - 1)) * SPI;
      if (s < kTChunk) lds_fetch16(g + size_t(u) * (kTileWaves - 1) * SPI * kTGroup, l + s * TP);
    }
  }
  __device__ __forceinline__ void start(const TileTab& T) const {  // before the first barrier that run() needs
    if (h >= 0) fetch(T, 0);
  }
  // NROW rows: values and factors to registers first (the compiler cannot tell the factor buffers from S, so
  // loads would wait behind the stores of earlier rows), then the chain
  template <int K, int NROW>
  struct Rows {
    double v[NROW], f[NROW * K];
  };
  template <int K, bool FWD, int NROW>
  static __device__ __forceinline__ void load(Rows<K, NROW>& r, const double* p, const double* f) {
    constexpr int ST = FWD ? -RS : RS;
#pragma unroll
    for (int t = 0; t < NROW; ++t) {
      r.v[t] = p[t * ST];
#pragma unroll
      for (int m = 0; m < K; ++m) r.f[t * K + m] = f[(t * K + m) * TP];
    }
  }
  template <int K, bool FWD, int NROW>
  static __device__ __forceinline__ void solve(Rows<K, NROW>& r, double* p, double (&y)[kTA]) {
    constexpr int M = FWD ? (K == 8 ? kTA : K) : K - 1, ST = FWD ? -RS : RS;
#pragma unroll
    for (int t = 0; t < NROW; ++t) {
      double v = r.v[t];
#pragma unroll
      for (int m = M - 1; m >= 0; --m) v = fma(r.f[t * K + m], y[m], v);
      if (!FWD) v *= r.f[t * K + K - 1];
#pragma unroll
      for (int m = kTA - 1; m > 0; --m) y[m] = y[m - 1];
      y[0] = v;
      p[t * ST] = v;
    }
  }
  // cnt rows: pairs of units, the next unit read while one is worked on, then the rest row by row
  template <int K, bool FWD>
  static __device__ __forceinline__ void chunk(double* p, const double* f, int cnt, double (&y)[kTA]) {
    constexpr int U = 4, ST = FWD ? -RS : RS;
    if constexpr (K != 8) {
      if (cnt >= 2 * U) {
        Rows<K, U> a, b;
        load<K, FWD, U>(a, p, f);
        do {
          load<K, FWD, U>(b, p + U * ST, f + U * K * TP);
          solve<K, FWD, U>(a, p, y);
          cnt -= 2 * U;
          const int nx = cnt >= 2 * U ? 2 * U : 0;  // the first unit again where there is no other
          load<K, FWD, U>(a, p + nx * ST, f + nx * K * TP);
          solve<K, FWD, U>(b, p + U * ST, y);
          p += 2 * U * ST;
          f += 2 * U * K * TP;
        } while (cnt >= 2 * U);
      }
    }
    for (; cnt > 0; --cnt, p += ST, f += K * TP) {
      Rows<K, 1> a;
      load<K, FWD, 1>(a, p, f);
      solve<K, FWD, 1>(a, p, y);
    }
  }
  // all waves, after start(); S complete before the call's first barrier, the solution visible after
  __device__ __forceinline__ void run(const TileTab& T, double* S, int lane) const {
    double y[kTA];
    const int lp = (lane & (CT - 1)) >> 1;
    lds_fetched();
    int nrow = T.chunk[0], ncnt = T.chunk[1], nk = T.chunk[2];
    for (int q = 0; q < T.nchunk; ++q) {
      if (h < 0) {
        const int row = nrow, cnt = ncnt, K = nk;
        nrow = T.chunk[4 * q + 4];  // the next chunk's, read while this one is worked on
        ncnt = T.chunk[4 * q + 5];
        nk = T.chunk[4 * q + 6];
        if (q == 0 || q == T.nfwd) {
#pragma unroll
          for (int m = 0; m < kTA; ++m) y[m] = 0.0;
        }
        const double* f = buf + (q % kTBufs) * BUF + lp;
        double* p = S + size_t(row) * RS + lane;
        if (lane < RS) {
          if (q < T.nfwd) {
            if (K == kTIn) chunk<kTIn, true>(p, f, cnt, y);
            else chunk<8, true>(p, f, cnt, y);
          } else {
            if (K == kTIn + 1) chunk<kTIn + 1, false>(p, f, cnt, y);
            else chunk<8, false>(p, f, cnt, y);
          }
        }
      } else {
        fetch(T, q + 1);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      }
      lds_barrier();
    }
  }

  // A(k)^T psi = b: the same rows of factors in the reverse order.  A row's entries, which the solve above gathers
  // with, scatter here: acc[0] is the row's own value with all that has reached it, acc[m + 1] that of the row
  // m + 1 further on.  Rows up to 8 past either end are read (not used): S has as many spare rows there.
  static constexpr int SPARE = kTA + 1;
  template <int K, bool FWD, int NROW>
  static __device__ __forceinline__ void load_t(Rows<K, NROW>& r, const double* p, const double* f) {
    constexpr int ST = FWD ? RS : -RS;
#pragma unroll
    for (int t = 0; t < NROW; ++t) {
      r.v[t] = p[(t + SPARE) * ST];
#pragma unroll
      for (int m = 0; m < K; ++m) r.f[t * K + m] = f[(m - t * K) * TP];
    }
  }
  template <int K, bool FWD, int NROW>
  static __device__ __forceinline__ void solve_t(Rows<K, NROW>& r, double* p, double (&acc)[SPARE]) {
    constexpr int M = FWD ? (K == 8 ? kTA : K) : K - 1, ST = FWD ? RS : -RS;
#pragma unroll
    for (int t = 0; t < NROW; ++t) {
      const double w = FWD ? acc[0] : acc[0] * r.f[t * K + K - 1];
#pragma unroll
      for (int m = 0; m < kTA; ++m) acc[m] = m < M ? fma(r.f[t * K + m], w, acc[m + 1]) : acc[m + 1];
      acc[kTA] = r.v[t];
      p[t * ST] = w;
    }
  }
  template <int K, bool FWD>
  static __device__ __forceinline__ void chunk_t(double* p, const double* f, int cnt, double (&acc)[SPARE]) {
    constexpr int U = 4, ST = FWD ? RS : -RS;
    if constexpr (K != 8) {
      if (cnt >= 2 * U) {
        Rows<K, U> a, b;
        load_t<K, FWD, U>(a, p, f);
        do {
          load_t<K, FWD, U>(b, p + U * ST, f - U * K * TP);
          solve_t<K, FWD, U>(a, p, acc);
          cnt -= 2 * U;
          const int nx = cnt >= 2 * U ? 2 * U : 0;
          load_t<K, FWD, U>(a, p + nx * ST, f - nx * K * TP);
          solve_t<K, FWD, U>(b, p + U * ST, acc);
          p += 2 * U * ST;
          f -= 2 * U * K * TP;
        } while (cnt >= 2 * U);
      }
    }
    for (; cnt > 0; --cnt, p += ST, f -= K * TP) {
      Rows<K, 1> a;
      load_t<K, FWD, 1>(a, p, f);
      solve_t<K, FWD, 1>(a, p, acc);
    }
  }
  __device__ __forceinline__ void start_t(const TileTab& T) const {
    if (h >= 0) fetch(T, T.nchunk - 1);
  }
  __device__ __forceinline__ void run_t(const TileTab& T, double* S, int n2, int lane) const {
    double acc[SPARE];
    const int lp = (lane & (CT - 1)) >> 1;
    double* s = S + (lane & (RS - 1));
    lds_fetched();
    for (int q = T.nchunk - 1; q >= 0; --q) {
      if (h < 0) {
        const int row = T.chunk[4 * q], cnt = T.chunk[4 * q + 1], K = T.chunk[4 * q + 2];
        const bool up = q < T.nfwd;  // rows ascending
        if (q == T.nchunk - 1 || q == T.nfwd - 1) {
#pragma unroll
          for (int m = 0; m < SPARE; ++m) acc[m] = s[(up ? m : n2 - m) * RS];
        }
        const double* f = buf + (q % kTBufs) * BUF + lp + (cnt - 1) * K * TP;
        double* p = s + (up ? row - (cnt - 1) : row + cnt - 1) * RS;
        if (lane < RS) {
          if (up) {
            if (K == kTIn) chunk_t<kTIn, true>(p, f, cnt, acc);
            else chunk_t<8, true>(p, f, cnt, acc);
          } else {
            if (K == kTIn + 1) chunk_t<kTIn + 1, false>(p, f, cnt, acc);
            else chunk_t<8, false>(p, f, cnt, acc);
          }
          if (q == 0) s[n2 * RS] = acc[0];
        }
      } else {
        if (q > 0) fetch(T, q - 1);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      }
      lds_barrier();
    }
  }
};


// ---------------------------------------------------------------------------
// fused m^c (the sweeps of mc_body).  Bound by its serial sweeps (LU 20k cycles, A(k) 40k of 97k at 129 rows) and
// by the LDS reads and field latency of the values (25k).  One tile per compute unit takes 45.9 us at
// 64 x 129 x 64 and 52.4 us at 128 x 129 x 128; the streaming kernel took 251 and 290 us.
struct McTileArgs {
  const double *vals, *d1, *d2, *d3;
  double *V1, *V2, *V3, *rhoc, *c2, *mparc;
};
constexpr int kTMostRows = 24;  // rows of a lane in kernels that hold them in registers
template <int CT>
constexpr bool tile_rows_fit(int n2, int most) {
  return (n2 + TileRows<CT>::SLOTS - 1) / TileRows<CT>::SLOTS <= most;
}
template <int CT>
struct McTileLds {
  static size_t bytes(int n2) {
    return !tile_rows_fit<CT>(n2 + 1, kTMostRows) ? SIZE_MAX
           : size_t(pad16(n2 + 1)) * 2 * CT * 8 + TileSolveA<CT>::LDS + tile_tab_bytes(n2) + size_t(n2 + 1) * 16;
  }
};
// Tables of the G rows (0 at the Robin rows) that a lane's 16 hold: rows 0 .. 15 and 16 .. 23 of its slot
template <int CT>
struct TileG {
  double t[2][kTGRow];
  int lo[2];
  __device__ __forceinline__ TileG(const TileTab& T, int d, const TileRows<CT>& rows, int lane) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int tr = rows.template tab<16>(16 * h, lane);
      load_row(t[h], T.g[d] + size_t(tr) * kTGRow);
      lo[h] = T.glo[d][tr];
    }
  }
  // r = G x from the n2 rows of a column in LDS
  __device__ __forceinline__ void rows(double (&r)[kTMostRows], const double* x, const TileRows<CT>& rw) const {
    unrolled<0, kTMostRows / 4>([&](auto gc) __attribute__((always_inline)) {
      constexpr int G = 4 * decltype(gc)::value, H = G / 16;
      if (G < rw.R) {
        double v[4][kTW];
        unrolled<0, 4>([&](auto uc) __attribute__((always_inline)) { tile_taps<(G + decltype(uc)::value) % 16, kTW, 2 * CT>(v[decltype(uc)::value], x, lo[H]); });
        unrolled<0, 4>([&](auto uc) __attribute__((always_inline)) {
          constexpr int U = decltype(uc)::value;
          r[G + U] = 0.0;
          fb8<(G + U) % 16>(r[G + U], t[H], v[U]);
        });
      }
    });
  }
};
template <int CT>
__device__ __forceinline__ void tile_put_rows(double* s, const double (&r)[kTMostRows], const TileRows<CT>& rows) {
  unrolled<0, kTMostRows>([&](auto nc) __attribute__((always_inline)) {
    constexpr int N = decltype(nc)::value;
    if (N < rows.R && rows.own(N)) s[(rows.r0 + N) * (2 * CT)] = r[N];
  });
}
// plane mean of S's column 0: c_j = c_{j+1} + x_j / dstar_j, c_{n2} = 0
template <int RS>
__device__ __forceinline__ void mc_tile_mean(const DevPlan& P, const double* S, double* mean) {
  const int n2 = P.n2;
  for (int e = threadIdx.x; e < 2 * n2; e += kTileThreads) mean[e] = S[(e >> 1) * RS + (e & 1)] / P.dstar[e >> 1];
  __syncthreads();
  if (threadIdx.x < 2) {
    double acc = 0.0;
    mean[2 * n2 + threadIdx.x] = 0.0;
#pragma unroll 8
    for (int j = n2 - 1; j >= 0; --j) {
      acc += mean[2 * j + threadIdx.x];
      mean[2 * j + threadIdx.x] = acc;
    }
  }
}
template <int CT>
__device__ __forceinline__ void mc_tile_body(const DevPlan& P, unsigned tile, const McTileArgs& A) {
  constexpr int RS = 2 * CT;
  extern __shared__ double lds_d[];
  const TileTab& T = P.tt;
  const int n2 = P.n2, w = tile_wave(), lane = threadIdx.x & 63;
  double* S = lds_d;
  double* s = S + (lane & (RS - 1));
  const TileLane L = tile_lane<CT, true>(P, tile, lane);
  const unsigned bytes = unsigned(n2) * L.rs;
  const TileBuf vals = tile_buf(A.vals, bytes), d1 = tile_buf(A.d1, bytes), d2 = tile_buf(A.d2, bytes),
                d3 = tile_buf(A.d3, bytes), V1 = tile_buf(A.V1, bytes), V2 = tile_buf(A.V2, bytes),
                V3 = tile_buf(A.V3, bytes);
  double* tab = S + size_t(pad16(n2 + 1)) * RS;
  double* fbuf = tab + tile_tab_bytes(n2) / 8;
  double* mean = fbuf + TileSolveA<CT>::LDS / 8;
  tile_fetch<CT>(S, A.vals, L, n2, w, lane);
  tile_fetch_tables(T, 0, tab, n2, w, lane);
  TileSolveA<CT> sa;
  sa.init(T, fbuf, tile, w, lane);
  sa.start(T);
  const TileRows<CT> rows(n2, L, w, lane), rows1(n2 + 1, L, w, lane);
  const TileG<CT> G(T, 1, rows1, lane);
  lds_fetched();
  const double ksq = L.k1 * L.k1 + L.k3 * L.k3;
  const double ik = ksq == 0.0 ? 0.0 : 1.0 / sqrt(ksq);
  const bool tile_mean = tile == 0;
  if (w == 0 && lane < RS) tile_solve<RS>(S + lane, tab, n2, lane);
  lds_barrier();
  if (A.rhoc) {
    const TileBuf rhoc = tile_buf(A.rhoc, bytes);
    for (int k = 0; k < rows.R; ++k) gst(rhoc, rows.st(k), s[min(rows.r0 + k, n2 - 1) * RS]);
  }
  // the plane mean's solution is kept aside during the sweeps of A(k)
  if (tile_mean) mc_tile_mean<RS>(P, S, mean);
  {  // r = -G1 rho_t takes the place of rho_t
    double r[kTMostRows];
    G.rows(r, s, rows1);
    lds_barrier();
    tile_put_rows<CT>(s, r, rows1);
  }
  sa.run(T, S, lane);
  if (tile_mean) {
    for (int e = threadIdx.x; e < 2 * (n2 + 1); e += kTileThreads) S[(e >> 1) * RS + (e & 1)] = mean[e];
    __syncthreads();
  }
  // coefficients (where asked for)
  if (A.c2) {
    const TileBuf rhoc = tile_buf(A.rhoc, bytes), c2 = tile_buf(A.c2, bytes + L.rs), mp = tile_buf(A.mparc, bytes);
    for (int k = 0; k < rows1.R; ++k) {
      const int i = min(rows1.r0 + k, n2), j = max(i - 1, 0);
      const double x = s[i * RS], d = P.dstar[j] * (x - s[j * RS]);
      const unsigned o = L.off + unsigned(j) * L.rs;
      const double m = times_i_lane(gld(rhoc, o) + d, L.c) * ik;
      gst(c2, rows1.st(k), x);
      gst(mp, rows1.own(k) && L.act && i > 0 ? o : kNoStore, L.mean ? 0.0 : m);
    }
  }
  // values at tau
  struct Group {
    double f[kTFRow], ev[4], e1[4], e2[4], e3[4];
    int lo;
  };
  tile_groups(
      rows.R,
      [&](int k) __attribute__((always_inline)) {
        Group g;
        const int tr = rows.template tab<4>(k, lane);
        load_row(g.f, T.f + size_t(tr) * kTFRow);
        g.lo = T.flo[tr];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const unsigned o = rows.at(k + u);
          g.ev[u] = gld(vals, o);
          g.e1[u] = gld(d1, o);  // 0 where there is no m^d
          g.e2[u] = gld(d2, o);
          g.e3[u] = gld(d3, o);
        }
        return g;
      },
      [&](int k, const Group& g) __attribute__((always_inline)) {
        double v[4][kMaxW];
        unrolled<0, 4>([&](auto uc) __attribute__((always_inline)) { tile_taps<decltype(uc)::value, kMaxW, RS>(v[decltype(uc)::value], s, g.lo); });
        unrolled<0, 4>([&](auto uc) __attribute__((always_inline)) {
          constexpr int U = decltype(uc)::value;
          double m2 = 0.0, f1 = 0.0;
          fb2x5<U>(m2, f1, g.f, g.f + kMaxW, v[U]);
          fb2x5<U>(m2, f1, g.f + 5, g.f + kMaxW + 5, v[U] + 5);
          const double sum = L.mean ? 0.0 : g.ev[U] + f1;  // rho_t + F1 c
          // m1, m3, or for the iterates before the last psi (see mc_body)
          const double mp = times_i_lane(sum, L.c) * ik, psi = sum * (ik * ik);
          const unsigned o = rows.st(k + U);
          gst(V1, o, (A.V3 ? mp * (L.k1 * ik) : psi) + g.e1[U]);
          gst(V2, o, m2 + g.e2[U]);
          gst(V3, o, mp * (L.k3 * ik) + g.e3[U]);
        });
      });
}
template <int CT>
__global__ void __launch_bounds__(kTileThreads) k_mc_tile(DevPlan P, McTileArgs A) {
  mc_tile_body<CT>(P, blockIdx.x, A);
}

// E0 values of a column in LDS
template <int CT>
__device__ __forceinline__ void tile_values0(const TileTab& T, const double* s, const TileRows<CT>& rows, int lane,
                                             const TileBuf& out) {
  struct Group {
    double t[kTW];
    int lo;
  };
  tile_groups(
      rows.R,
      [&](int k) __attribute__((always_inline)) {
        Group g;
        const int tr = rows.template tab<4>(k, lane);
        load_row(g.t, T.e + size_t(tr) * kTERow);
        g.lo = T.elo[tr];
        return g;
      },
      [&](int k, const Group& g) __attribute__((always_inline)) {
        double v[4][kTW];
        unrolled<0, 4>([&](auto uc) __attribute__((always_inline)) { tile_taps<decltype(uc)::value, kTW, 2 * CT>(v[decltype(uc)::value], s, g.lo); });
        unrolled<0, 4>([&](auto uc) __attribute__((always_inline)) {
          constexpr int U = decltype(uc)::value;
          double e0 = 0.0;
          fb8<U>(e0, g.t, v[U]);
          gst(out, rows.st(k + U), e0);
        });
      });
}

// ---------------------------------------------------------------------------
// m^c of rho_t coefficients: the m1, m2, m3 coefficients (operator entry point).  Bound by the sweeps of A(k).
// 64 x 65 x 64: 328 -> 18.2 us (the streaming kernel forms the LU as it goes).
struct McCoefTileArgs {
  const double* rho;
  double *m1, *m2, *m3;
};
template <int CT>
struct McCoefTileLds {
  static size_t bytes(int n2) {
    return !tile_rows_fit<CT>(n2 + 1, kTMostRows) ? SIZE_MAX
           : size_t(pad16(n2 + 1)) * 2 * CT * 8 + TileSolveA<CT>::LDS + size_t(n2 + 1) * 16;
  }
};
template <int CT>
__global__ void __launch_bounds__(kTileThreads) k_mc_coef_tile(DevPlan P, McCoefTileArgs A) {
  constexpr int RS = 2 * CT;
  extern __shared__ double lds_d[];
  const TileTab& T = P.tt;
  const int n2 = P.n2, w = tile_wave(), lane = threadIdx.x & 63;
  double* S = lds_d;
  double* s = S + (lane & (RS - 1));
  const TileLane L = tile_lane<CT, true>(P, blockIdx.x, lane);
  double* fbuf = S + size_t(pad16(n2 + 1)) * RS;
  double* mean = fbuf + TileSolveA<CT>::LDS / 8;
  tile_fetch<CT>(S, A.rho, L, n2, w, lane);
  TileSolveA<CT> sa;
  sa.init(T, fbuf, blockIdx.x, w, lane);
  sa.start(T);
  const TileRows<CT> rows1(n2 + 1, L, w, lane);
  const TileG<CT> G(T, 1, rows1, lane);
  lds_fetched();
  const double ksq = L.k1 * L.k1 + L.k3 * L.k3, ik = ksq == 0.0 ? 0.0 : 1.0 / sqrt(ksq);
  if (blockIdx.x == 0) mc_tile_mean<RS>(P, S, mean);
  {
    double r[kTMostRows];
    G.rows(r, s, rows1);
    lds_barrier();
    tile_put_rows<CT>(s, r, rows1);
  }
  sa.run(T, S, lane);
  if (blockIdx.x == 0) {
    for (int e = threadIdx.x; e < 2 * (n2 + 1); e += kTileThreads) S[(e >> 1) * RS + (e & 1)] = mean[e];
    __syncthreads();
  }
  const unsigned bytes = unsigned(n2) * L.rs;
  const TileBuf rho = tile_buf(A.rho, bytes), m1 = tile_buf(A.m1, bytes), m2 = tile_buf(A.m2, bytes + L.rs),
                m3 = tile_buf(A.m3, bytes);
  struct Group {  // row i and the row i - 1 of m1, m3
    double r[4], d[4];
  };
  tile_groups(
      rows1.R,
      [&](int k) __attribute__((always_inline)) {
        Group g;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int j = max(min(rows1.r0 + k + u, n2) - 1, 0);
          g.r[u] = gld(rho, L.off + unsigned(j) * L.rs);
          g.d[u] = P.dstar[j];
        }
        return g;
      },
      [&](int k, const Group& g) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int i = min(rows1.r0 + k + u, n2), j = max(i - 1, 0);
          const double x = s[i * RS], sum = L.mean ? 0.0 : g.r[u] + g.d[u] * (x - s[j * RS]);
          const double mp = times_i_lane(sum, L.c) * ik;
          const unsigned o = rows1.own(k + u) && L.act && i > 0 ? L.off + unsigned(j) * L.rs : kNoStore;
          gst(m2, rows1.st(k + u), x);
          gst(m1, o, mp * (L.k1 * ik));
          gst(m3, o, mp * (L.k3 * ik));
        }
      });
}

// ---------------------------------------------------------------------------
// Transposes of the m^d and m^c maps (what k_md_t, k_mc_t do): with D = -i (k1 m1 + k3 m3) / k^2 and
// b = m2 + D*^T D, psi = A(k)^-T b; m^d: phi2 = G0^T psi, Omega2 = i (k3 m1 - k1 m3) / k^2; m^c: rho_t = D - G1^T psi.
// Bound by the two sweeps of A(k)^T.  m^c 64 x 65 x 64: 175 -> 23.2 us, 96 x 97 x 96:
// 288 -> 32.8 us; m^d 155 -> 22.1 and 277 -> 31.5 us.
struct SolveTTileArgs {
  const double *m1, *m2, *m3;
  double *out, *om, *m1bar, *m3bar;  // om, m1bar, m3bar: m^d
};
template <int CT>
struct SolveTTileLds {
  static constexpr size_t rows(int n2) { return 2 * size_t(pad16(n2 + 1)) + 2 * TileSolveA<CT>::SPARE; }
  static size_t bytes(int n2) {
    return (rows(n2) + 1) * 2 * CT * 8 + TileSolveA<CT>::LDS + size_t(n2 + 1) * 16;
  }
};
template <int CT, bool MC>
__global__ void __launch_bounds__(kTileThreads) k_solve_t_tile(DevPlan P, SolveTTileArgs A) {
  constexpr int RS = 2 * CT, SP = TileSolveA<CT>::SPARE;
  extern __shared__ double lds_d[];
  const TileTab& T = P.tt;
  const int n2 = P.n2, w = tile_wave(), lane = threadIdx.x & 63, l = lane & (RS - 1);
  double* S = lds_d + SP * RS;                         // n2 + 1 rows of b, then psi
  double* X = S + size_t(pad16(n2 + 1) + SP) * RS;     // n2 + 1 rows of D
  double* s = S + l;
  double* x = X + l;
  double* spare = X + size_t(pad16(n2 + 1)) * RS + l;
  double* fbuf = X + size_t(pad16(n2 + 1) + 1) * RS;
  double* mean = fbuf + TileSolveA<CT>::LDS / 8;
  const TileLane L = tile_lane<CT, true>(P, blockIdx.x, lane);
  TileSolveA<CT> sa;
  sa.init(T, fbuf, blockIdx.x, w, lane);
  sa.start_t(T);
  const TileRows<CT> rows(n2, L, w, lane), rows1(n2 + 1, L, w, lane);
  const double ksq = L.k1 * L.k1 + L.k3 * L.k3, iksq = ksq == 0.0 ? 0.0 : 1.0 / ksq;
  const unsigned bytes = unsigned(n2) * L.rs;
  {
    const TileBuf m1 = tile_buf(A.m1, bytes), m2 = tile_buf(A.m2, bytes + L.rs), m3 = tile_buf(A.m3, bytes),
                  om = tile_buf(MC ? nullptr : A.om, bytes), b1 = tile_buf(MC ? nullptr : A.m1bar, 8 * n2),
                  b3 = tile_buf(MC ? nullptr : A.m3bar, 8 * n2);
    struct Group {
      double a[4], b[4], c[4];
    };
    tile_groups(
        rows1.R,
        [&](int k) __attribute__((always_inline)) {
          Group g;
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const unsigned o = rows1.at(k + u);
            g.a[u] = gld(m1, o);  // 0 at row n2
            g.b[u] = gld(m2, o);
            g.c[u] = gld(m3, o);
          }
          return g;
        },
        [&](int k, const Group& g) __attribute__((always_inline)) {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            // (of the plane mean neither enters, whatever it holds)
            const double D = -times_i_lane(L.k1 * g.a[u] + L.k3 * g.c[u], L.c) * iksq;
            *rows1.put(x, k + u, spare) = L.mean ? 0.0 : D;
            *rows1.put(s, k + u, spare) = g.b[u];
            if constexpr (!MC) {
              const double O = times_i_lane(L.k3 * g.a[u] - L.k1 * g.c[u], L.c) * iksq;
              gst(om, rows1.st(k + u), L.mean ? 0.0 : O);
              // the plane mean's m1, m3 (row n2 is past the end)
              const unsigned o = L.mean && L.c == 0 && rows1.own(k + u) ? 8 * unsigned(rows1.r0 + k + u) : kNoStore;
              gst(b1, o, g.a[u]);
              gst(b3, o, g.c[u]);
            }
          }
        });
  }
  lds_barrier();
  for (int k = 0; k < rows1.R; k += 4) {  // b += D*^T D
    double v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int r = min(rows1.r0 + k + u, n2), q = max(r - 1, 0);
      const double up = r > 0 ? P.dstar[q] * x[q * RS] : 0.0;
      v[u] = s[r * RS] + (up - P.dstar[min(r, n2 - 1)] * x[r * RS]);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) *rows1.put(s, k + u, spare) = v[u];
  }
  if (MC && blockIdx.x == 0) {  // plane mean: sums of b from the bottom, over dstar
    lds_barrier();
    if (threadIdx.x < 2) {
      double acc = 0.0;
#pragma unroll 8
      for (int j = 0; j < n2; ++j) {
        acc += S[j * RS + threadIdx.x];
        mean[2 * j + threadIdx.x] = acc / P.dstar[j];
      }
    }
  }
  sa.run_t(T, S, n2, lane);
  const TileBuf out = tile_buf(A.out, bytes);
  struct Group {
    double t[kTGTRow];
    int lo;
  };
  tile_groups(
      rows.R,
      [&](int k) __attribute__((always_inline)) {
        Group g;
        const int tr = rows.template tab<4>(k, lane);
        load_row(g.t, T.gt[MC] + size_t(tr) * kTGTRow);
        g.lo = T.gtlo[MC][tr];
        return g;
      },
      [&](int k, const Group& g) __attribute__((always_inline)) {
        unrolled<0, 4>([&](auto uc) __attribute__((always_inline)) {
          constexpr int U = decltype(uc)::value;
          const int r = min(rows.r0 + k + U, n2 - 1);
          double v[kTGTRow], a = MC ? x[r * RS] : 0.0;
          tile_taps<U, kTGTRow, RS>(v, s, g.lo);
          fb12<U>(a, g.t, v);
          if (L.mean) a = MC ? mean[2 * r + L.c] : 0.0;
          gst(out, rows.st(k + U), a);
        });
      });
}

// ---------------------------------------------------------------------------
// projections (the sweeps and epilogues of proj_body).  Bound by the LU sweeps (20k cycles at 129 rows).  Final
// projection with the z update and values at 64 x 129 x 64: 151 -> 23.7 us, 128 x 129 x 128: 169 -> 35.3 us.
// Kinds 3 .. 5 are the transposes of kinds 0 .. 2, R A^-T: with U = D V, A^T = V^T (D L^T) has the same form (tables
// of V^T and D L^T), and what is 0 at the end rows is the result.  96 x 97 x 96: 77.4 -> 13.5 us (streaming,
// tile).
constexpr int kProjTileFields = 8;
struct ProjTileArgs {
  int kind, stage;
  const double* in[kProjTileFields];
  double* out[kProjTileFields];         // EPI_STORE: one per blockIdx.y
  const double *add, *z, *zt_prev;
  double *z_out, *vals_out;
};
template <int CT>
struct ProjTileLds {
  static size_t bytes(int n2) { return (size_t(pad16(n2)) + 1) * 2 * CT * 8 + tile_tab_bytes(n2); }
};
template <int CT, int EPI>
__device__ __forceinline__ void proj_tile_body(const DevPlan& P, unsigned tile, unsigned field, const ProjTileArgs& A) {
  constexpr int RS = 2 * CT;
  extern __shared__ double lds_d[];
  const TileTab& T = P.tt;
  const int n2 = P.n2, w = tile_wave(), lane = threadIdx.x & 63;
  double* S = lds_d;
  const TileLane L = tile_lane<CT, false>(P, tile, lane);
  double* spare = S + size_t(pad16(n2)) * RS + (lane & (RS - 1));
  double* tab = S + size_t(pad16(n2) + 1) * RS;
  tile_fetch<CT, true>(S, A.in[field], L, n2, w, lane);
  tile_fetch_tables(T, A.kind, tab, n2, w, lane);
  lds_fetched();
  if (w == 0 && lane < RS) {
    if (A.kind == 1 || A.kind == 2) S[lane] = S[(n2 - 1) * RS + lane] = 0.0;
    tile_solve<RS>(S + lane, tab, n2, lane);
    if (A.kind > 3) S[lane] = S[(n2 - 1) * RS + lane] = 0.0;
  }
  lds_barrier();
  double* s = S + (lane & (RS - 1));
  const unsigned bytes = unsigned(n2) * L.rs;
  // a fixed-point iterate before the last is used only through its values
  const TileBuf out = tile_buf(EPI == EPI_ADD ? nullptr : A.out[field], bytes), add = tile_buf(A.add, bytes),
                z = tile_buf(A.z, bytes), zp = tile_buf(A.stage != 0 ? A.zt_prev : nullptr, bytes),
                zo = tile_buf(A.z_out, bytes);
  const TileRows<CT> rows(n2, L, w, lane);
  struct Group {
    double a[4], z0[4], zp[4];
  };
  tile_groups(
      rows.R,
      [&](int k) __attribute__((always_inline)) {
        Group g;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const unsigned o = rows.at(k + u);
          g.a[u] = EPI != EPI_STORE ? gld(add, o) : 0.0;
          g.z0[u] = EPI == EPI_ADD_ZUPDATE ? gld(z, o) : 0.0;
          g.zp[u] = EPI == EPI_ADD_ZUPDATE ? gld(zp, o) : 0.0;
        }
        return g;
      },
      [&](int k, const Group& g) __attribute__((always_inline)) {
        double x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = s[min(rows.r0 + k + u, n2 - 1) * RS];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (EPI != EPI_STORE) {
            x[u] += g.a[u];
            *rows.put(s, k + u, spare) = x[u];
          }
          const unsigned o = rows.st(k + u);
          if (EPI != EPI_ADD) gst(out, o, x[u]);
          if (EPI == EPI_ADD_ZUPDATE)
            gst(zo, o, A.stage == 0 ? fma(0.5 * P.dt, x[u], g.z0[u]) : fma(P.dt, x[u] - 0.5 * g.zp[u], g.z0[u]));
        }
      });
  if (!A.vals_out) return;
  lds_barrier();
  tile_values0<CT>(T, s, rows, lane, tile_buf(A.vals_out, bytes));
}
template <int CT, int EPI>
__global__ void __launch_bounds__(kTileThreads) k_proj_tile(DevPlan P, ProjTileArgs A) {
  proj_tile_body<CT, EPI>(P, blockIdx.x, blockIdx.y, A);
}

// ---------------------------------------------------------------------------
// prologue: m^d and its values (job 0, pair tiles), values of z (job 1) and the guess (job 2), flat tiles.  Bound
// by the sweeps of m^d (42k of its 70k cycles at 129 rows).  64 x 129 x 64: 426 -> 35.1 us, 128 x 129 x 128:
// 464 -> 95 us.
constexpr size_t kTileLdsMax = 160 * 1024;  // LDS of one workgroup
// m^d has Omega2 in rows of its own beside phi2's where both fit: it is there before the sweeps, and V1 and V3 are
// written once.  Else it follows when the values of c are done, with parts of V1 and V3 written and read back
// meanwhile, which keeps the wide tiles up to 191 rows (128 x 129 x 128: 117 -> 95 us,
// 256 x 129 x 256: 460 -> 377 us)
template <int CT>
struct PrologueTileLds {
  __host__ __device__ static constexpr size_t rows(int n2, bool both) {
    return (size_t(pad16(n2 + 1)) + (both ? pad16(n2) : 0)) * 2 * CT * 8;
  }
  __host__ __device__ static constexpr bool both(int n2) { return rows(n2, true) + TileSolveA<CT>::LDS <= kTileLdsMax; }
  static size_t bytes(int n2) {
    return !tile_rows_fit<CT>(n2 + 1, kTMostRows) ? SIZE_MAX : rows(n2, both(n2)) + TileSolveA<CT>::LDS;
  }
};
template <int CT>
__device__ __forceinline__ void md_tile_body(const DevPlan& P, unsigned tile, const MdArgs& A) {
  constexpr int RS = 2 * CT;
  extern __shared__ double lds_d[];
  const TileTab& T = P.tt;
  const int n2 = P.n2, w = tile_wave(), lane = threadIdx.x & 63;
  if (int(tile) * (CT / 2) >= P.nl * ((P.nn + 1) / 2)) return;
  const bool both = PrologueTileLds<CT>::both(n2);
  double* S = lds_d;                                              // c
  double* X = both ? S + size_t(pad16(n2 + 1)) * RS : S;          // phi2, then Omega2
  const TileLane L = tile_lane<CT, true>(P, tile, lane);
  const double ksq = L.k1 * L.k1 + L.k3 * L.k3, iksq = ksq == 0.0 ? 0.0 : 1.0 / ksq;
  tile_fetch<CT>(X, reinterpret_cast<const double*>(A.phi), L, n2, w, lane);
  TileSolveA<CT> sa;
  sa.init(T, lds_d + PrologueTileLds<CT>::rows(n2, both) / 8, tile, w, lane);
  sa.start(T);
  const TileRows<CT> rows(n2, L, w, lane), rows1(n2 + 1, L, w, lane);
  const TileG<CT> G(T, 0, rows1, lane);
  lds_fetched();
  const double* x = X + (lane & (RS - 1));
  double* s = S + (lane & (RS - 1));
  {
    double r[kTMostRows];
    G.rows(r, x, rows1);
    if (!both) lds_barrier();
    tile_put_rows<CT>(s, r, rows1);
  }
  lds_barrier();
  if (both) tile_fetch<CT>(X, reinterpret_cast<const double*>(A.om), L, n2, w, lane);
  sa.run(T, S, lane);
  lds_fetched();
  const unsigned bytes = unsigned(n2) * L.rs;
  const TileBuf V1 = tile_buf(A.V1, bytes), V2 = tile_buf(A.V2, bytes), V3 = tile_buf(A.V3, bytes);
  if (A.c2o) {
    const TileBuf c2o = tile_buf(A.c2o, bytes + L.rs), m1o = tile_buf(A.m1o, bytes), m3o = tile_buf(A.m3o, bytes),
                  om = tile_buf(A.om, bytes);
    for (int k = 0; k < rows1.R; ++k) {
      const int i = min(rows1.r0 + k, n2), j = max(i - 1, 0);
      const double c = s[i * RS], D = P.dstar[j] * (c - s[j * RS]), O = gld(om, L.off + unsigned(j) * L.rs);
      double m1 = times_i_lane(L.k1 * D - L.k3 * O, L.c) * iksq;
      double m3 = times_i_lane(L.k3 * D + L.k1 * O, L.c) * iksq;
      if (L.mean) {
        m1 = L.c ? 0.0 : A.m1bar[j];
        m3 = L.c ? 0.0 : A.m3bar[j];
      }
      const unsigned o = rows1.own(k) && L.act && i > 0 ? L.off + unsigned(j) * L.rs : kNoStore;
      gst(c2o, rows1.st(k), L.mean ? 0.0 : c);
      gst(m1o, o, m1);
      gst(m3o, o, m3);
    }
  }
  if (!A.V1) return;  // coefficients only
  // V2 = F0 c, and with f1 = F1 c, oe = E0 Omega2: V1 = i (k1 f1 - k3 oe) / k^2, V3 = i (k3 f1 + k1 oe) / k^2.
  // Without rows of its own for Omega2, k1 f1 and k3 f1 wait in V1 and V3 (each element its own lane's).
  struct GroupF {
    double f[kTFRow];
    int lo;
  };
  struct GroupE {
    double t[kTW], p1[4], p3[4];
    int lo;
  };
  auto load_f = [&](int k) __attribute__((always_inline)) {
    GroupF g;
    const int tr = rows.template tab<4>(k, lane);
    load_row(g.f, T.f + size_t(tr) * kTFRow);
    g.lo = T.flo[tr];
    return g;
  };
  auto load_e = [&](int k, bool part) __attribute__((always_inline)) {
    GroupE g;
    const int tr = rows.template tab<4>(k, lane);
    load_row(g.t, T.e + size_t(tr) * kTERow);
    g.lo = T.elo[tr];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      g.p1[u] = part ? gld(V1, rows.at(k + u)) : 0.0;
      g.p3[u] = part ? gld(V3, rows.at(k + u)) : 0.0;
    }
    return g;
  };
  auto work_f = [&](int k, const GroupF& g, double (&p1)[4], double (&p3)[4]) __attribute__((always_inline)) {
    unrolled<0, 4>([&](auto uc) __attribute__((always_inline)) {
      constexpr int U = decltype(uc)::value;
      double v[kMaxW], f0 = 0.0, f1 = 0.0;
      tile_taps<U, kMaxW, RS>(v, s, g.lo);
      fb2x5<U>(f0, f1, g.f, g.f + kMaxW, v);
      fb2x5<U>(f0, f1, g.f + 5, g.f + kMaxW + 5, v + 5);
      gst(V2, L.mean ? kNoStore : rows.st(k + U), f0);
      p1[U] = L.k1 * f1;
      p3[U] = L.k3 * f1;
    });
  };
  auto work_e = [&](int k, const GroupE& g, const double (&p1)[4], const double (&p3)[4]) __attribute__((always_inline)) {
    unrolled<0, 4>([&](auto uc) __attribute__((always_inline)) {
      constexpr int U = decltype(uc)::value;
      double u[kTW], oe = 0.0;
      tile_taps<U, kTW, RS>(u, x, g.lo);
      fb8<U>(oe, g.t, u);
      const unsigned o = L.mean ? kNoStore : rows.st(k + U);
      gst(V1, o, times_i_lane(fma(-L.k3, oe, p1[U]), L.c) * iksq);
      gst(V3, o, times_i_lane(fma(L.k1, oe, p3[U]), L.c) * iksq);
    });
  };
  if (both) {
    struct Group {
      GroupF f;
      GroupE e;
    };
    tile_groups(
        rows.R, [&](int k) __attribute__((always_inline)) { return Group{load_f(k), load_e(k, false)}; },
        [&](int k, const Group& g) __attribute__((always_inline)) {
          double p1[4], p3[4];
          work_f(k, g.f, p1, p3);
          work_e(k, g.e, p1, p3);
        });
  } else {
    tile_groups(rows.R, load_f, [&](int k, const GroupF& g) __attribute__((always_inline)) {
      double p1[4], p3[4];
      work_f(k, g, p1, p3);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const unsigned o = L.mean ? kNoStore : rows.st(k + u);
        gst(V1, o, p1[u]);
        gst(V3, o, p3[u]);
      }
    });
    lds_barrier();
    tile_fetch<CT>(X, reinterpret_cast<const double*>(A.om), L, n2, w, lane);
    lds_fetched();
    tile_groups(
        rows.R, [&](int k) __attribute__((always_inline)) { return load_e(k, true); },
        [&](int k, const GroupE& g) __attribute__((always_inline)) { work_e(k, g, g.p1, g.p3); });
  }
  if (tile == 0)  // plane mean: (<m>1, 0, <m>3)
    for (int e = threadIdx.x; e < 2 * n2; e += kTileThreads) {
      const int row = e >> 1, lo = T.elo[row];
      const cptr<double> wt = T.e + size_t(row) * kTERow;
      double a1 = 0.0, a3 = 0.0;
      if (!(e & 1)) {
#pragma unroll
        for (int q = 0; q < kTW; ++q) {
          a1 = fma(wt[q], A.m1bar[lo + q], a1);
          a3 = fma(wt[q], A.m3bar[lo + q], a3);
        }
      }
      const unsigned o = unsigned(row) * L.rs + 8 * (e & 1);
      gst(V1, o, a1);
      gst(V2, o, 0.0);
      gst(V3, o, a3);
    }
}
template <int CT>
__device__ __forceinline__ void values_z_tile_body(const DevPlan& P, unsigned tile, const ValuesZArgs& A) {
  constexpr int RS = 2 * CT;
  extern __shared__ double lds_d[];
  const TileTab& T = P.tt;
  const int n2 = P.n2, w = tile_wave(), lane = threadIdx.x & 63;
  if (tile * CT >= unsigned(P.nn) * P.nl) return;
  const TileLane L = tile_lane<CT, false>(P, tile, lane);
  const double ksq = L.k1 * L.k1 + L.k3 * L.k3;
  tile_fetch<CT>(lds_d, reinterpret_cast<const double*>(A.z), L, n2, w, lane);
  lds_fetched();
  const double* s = lds_d + (lane & (RS - 1));
  const TileRows<CT> rows(n2, L, w, lane);
  const unsigned bytes = unsigned(n2) * L.rs;
  const TileBuf V0 = tile_buf(A.V0, bytes), V1 = tile_buf(A.V1, bytes), VL = tile_buf(A.VL, bytes), V3 = tile_buf(A.V3, bytes);
  struct Group {
    double t[kTERow];
    int lo;
  };
  tile_groups(
      rows.R,
      [&](int k) __attribute__((always_inline)) {
        Group g;
        const int tr = rows.template tab<4>(k, lane);
        load_row(g.t, T.e + size_t(tr) * kTERow);
        g.lo = T.elo[tr];
        return g;
      },
      [&](int k, const Group& g) __attribute__((always_inline)) {
        unrolled<0, 4>([&](auto uc) __attribute__((always_inline)) {
          constexpr int U = decltype(uc)::value;
          double v[kTW], e0 = 0.0, e1 = 0.0, e2 = 0.0;
          tile_taps<U, kTW, RS>(v, s, g.lo);
          fb3x4<U>(e0, e1, e2, g.t, g.t + kTW, g.t + 2 * kTW, v);
          fb3x4<U>(e0, e1, e2, g.t + 4, g.t + kTW + 4, g.t + 2 * kTW + 4, v + 4);
          const double v3 = times_i_lane(e0 * L.k3, L.c);
          const unsigned o = rows.st(k + U);
          gst(V0, o, e0);
          gst(V1, o, e1);
          gst(VL, o, e2 - ksq * e0);
          gst(V3, o, v3);
        });
      });
}
template <int CT>
__device__ __forceinline__ void guess_tile_body(const DevPlan& P, unsigned tile, const GuessArgs& G) {
  constexpr int RS = 2 * CT;
  extern __shared__ double lds_d[];
  const TileTab& T = P.tt;
  const int n2 = P.n2, w = tile_wave(), lane = threadIdx.x & 63;
  if (tile * CT >= unsigned(P.nn) * P.nl) return;
  const TileLane L = tile_lane<CT, false>(P, tile, lane);
  const unsigned bytes = unsigned(n2) * L.rs;
  // (the zero guess reads nothing)
  const TileBuf z = tile_buf(G.zero ? nullptr : G.z, bytes), h1 = tile_buf(G.zero ? nullptr : G.h1, bytes),
                h2 = tile_buf(G.zero ? nullptr : G.h2, bytes), h3 = tile_buf(G.zero ? nullptr : G.h3, bytes),
                zt = tile_buf(G.zt, bytes);
  double* s = lds_d + (lane & (RS - 1));
  double* spare = s + size_t(pad16(n2)) * RS;
  const TileRows<CT> rows(n2, L, w, lane);
  struct Group {
    double a[4], b[4], c[4], d[4];
  };
  tile_groups(
      rows.R,
      [&](int k) __attribute__((always_inline)) {
        Group g;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const unsigned o = rows.at(k + u);
          g.a[u] = gld(z, o);
          g.b[u] = gld(h1, o);
          g.c[u] = gld(h2, o);
          g.d[u] = gld(h3, o);
        }
        return g;
      },
      [&](int k, const Group& g) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const double v = G.zero ? 0.0 : (G.a1 * g.a[u] + G.a2 * g.b[u] + G.a3 * g.c[u] + G.a4 * g.d[u]) / G.dt;
          *rows.put(s, k + u, spare) = v;
          gst(zt, rows.st(k + u), v);
        }
      });
  lds_barrier();
  tile_values0<CT>(T, s, rows, lane, tile_buf(G.V, bytes));
}
template <int CT>
__device__ __forceinline__ void prologue_tile_body(const DevPlan& P, unsigned tile, unsigned job, const MdArgs& M,
                                                   const ValuesZArgs& Z, const GuessArgs& G) {
  if (job == 0) md_tile_body<CT>(P, tile, M);
  else if (job == 1) values_z_tile_body<CT>(P, tile, Z);
  else guess_tile_body<CT>(P, tile, G);
}
template <int CT>
__global__ void __launch_bounds__(kTileThreads) k_prologue_tile(DevPlan P, MdArgs M, ValuesZArgs Z, GuessArgs G) {
  prologue_tile_body<CT>(P, blockIdx.x, blockIdx.y, M, Z, G);
}

// ---------------------------------------------------------------------------
// S_ij values from the velocity coefficients (strain_body).  Bound by LDS reads.  48 x 65 x 96: 83.9 -> 13.7 us.
template <int CT>
struct StrainTileLds {
  static size_t bytes(int n2) { return size_t(pad16(n2)) * 3 * 2 * CT * 8; }
};
struct StrainTileArgs {
  const double* u[3];
  double* S[6];
};
template <int CT>
__device__ __forceinline__ void strain_tile_body(const DevPlan& P, unsigned tile, const StrainTileArgs& A) {
  constexpr int RS = 2 * CT;
  extern __shared__ double lds_d[];
  const TileTab& T = P.tt;
  const int n2 = P.n2, w = tile_wave(), lane = threadIdx.x & 63;
  const size_t fld = size_t(pad16(n2)) * RS;
  const TileLane L = tile_lane<CT, false>(P, tile, lane);
#pragma unroll
  for (int f = 0; f < 3; ++f) tile_fetch<CT>(lds_d + f * fld, A.u[f], L, n2, w, lane);
  lds_fetched();
  const double* x = lds_d + (lane & (RS - 1));
  const TileRows<CT> rows(n2, L, w, lane);
  const unsigned bytes = unsigned(n2) * L.rs;
  const TileBuf S[6] = {tile_buf(A.S[0], bytes), tile_buf(A.S[1], bytes), tile_buf(A.S[2], bytes),
                        tile_buf(A.S[3], bytes), tile_buf(A.S[4], bytes), tile_buf(A.S[5], bytes)};
  struct Group {
    double t[2 * kTW];
    int lo;
  };
  tile_groups(
      rows.R,
      [&](int k) __attribute__((always_inline)) {
        Group g;
        const int tr = rows.template tab<4>(k, lane);
        load_row(g.t, T.e + size_t(tr) * kTERow);
        g.lo = T.elo[tr];
        return g;
      },
      [&](int k, const Group& g) __attribute__((always_inline)) {
        unrolled<0, 4>([&](auto uc) __attribute__((always_inline)) {
          constexpr int U = decltype(uc)::value;
          double i0[3], e1[3];
#pragma unroll
          for (int f = 0; f < 3; ++f) {
            double v[kTW], a = 0.0, b = 0.0;
            tile_taps<U, kTW, RS>(v, x + f * fld, g.lo);
            fb2x4<U>(a, b, g.t, g.t + kTW, v);
            fb2x4<U>(a, b, g.t + 4, g.t + kTW + 4, v + 4);
            i0[f] = times_i_lane(a, L.c);
            e1[f] = b;
          }
          const double d11 = L.k1 * i0[0], d33 = L.k3 * i0[2], th = (2.0 / 3.0) * ((d11 + e1[1]) + d33);
          const unsigned o = rows.st(k + U);
          gst(S[0], o, 2.0 * d11 - th);
          gst(S[1], o, fma(L.k1, i0[1], e1[0]));
          gst(S[2], o, L.k3 * i0[0] + L.k1 * i0[2]);
          gst(S[3], o, 2.0 * e1[1] - th);
          gst(S[4], o, fma(L.k3, i0[1], e1[2]));
          gst(S[5], o, 2.0 * d33 - th);
        });
      });
}
template <int CT>
__global__ void __launch_bounds__(kTileThreads) k_strain_tile(DevPlan P, StrainTileArgs A) {
  strain_tile_body<CT>(P, blockIdx.x, A);
}

// ---------------------------------------------------------------------------
// Momentum right-hand sides and the RK2 update from C_ij, u_hat and rho (what flux_body, rhs_fluct_body and
// rhs_mean_body do together).  With N_i = i k1 T_i1 + d/dy T_i2 + i k3 T_i3 the right-hand sides are
//   Omega2: E0 P a0 + E1 P a1,   phi2: E1 P b1 + (k^2 E0 + E2) P b2 + k^2 g rho
// of four sums of the values of T_ij = C_ij + tau_ij at tau (P the interpolation),
//   a0 = -k1 k3 T11 + (k1^2 - k3^2) T13 + k1 k3 T33,        a1 = i (k3 T12 - k1 T23),
//   b1 = k1^2 T11 + 2 k1 k3 T13 - k^2 T22 + k3^2 T33,       b2 = -i (k1 T12 + k3 T23),
// so four columns are interpolated instead of six and no T_ij goes through memory.  With constant mu the
// viscous parts are (the bulk terms cancel)
//   a0: i mu k^2 (k1 E0 u3 - k3 E0 u1),          a1: i mu (k3 E1 u1 - k1 E1 u3),
//   b1: 2 mu k^2 (i k1 E0 u1 + i k3 E0 u3 - E1 u2),   b2: -i mu (k1 E1 u1 + k3 E1 u3) + mu k^2 E0 u2.
// blockIdx.y 0 is Omega2, 1 phi2; the block after the last tile does the plane means.
// Bound by the two LU solves in turn (42k of 80k cycles at 129 rows) and by the latency of the six fields (16k).
// The six fields are loaded before the taps of their group and the four rows of a group stored together: loaded a
// group ahead they took 234 registers and 106k cycles.  64 x 129 x 64: ~50 us for what took 867 us in four kernels.
struct MomentumTileArgs {
  const double *C[6], *tau[6], *u[3];  // tau: tau_ij values (variable mu)
  const double* rho;
  const double *phi, *om, *rphi_prev, *rom_prev;
  double *phi_out, *om_out, *rphi_out, *rom_out;
  const double *m1, *m3, *r1p, *r3p;
  double *m1o, *m3o, *r1o, *r3o;
  int stage;
  unsigned tiles;
};
// rows of its four columns with the spare one: the fourth's padding (u3 is fetched once, before any write to it; so
// 129 rows of 16 columns just fit), else one more
__host__ __device__ constexpr int momentum_tile_rows(int n2) { return 4 * pad16(n2) + (n2 % 16 == 0); }
template <int CT>
struct MomentumTileLds {
  static size_t bytes(int n2) { return size_t(momentum_tile_rows(n2)) * 2 * CT * 8 + tile_tab_bytes(n2); }
};
// RHS of <m>1 and <m>3: P_N of d/dy <T12>, d/dy <T32>
template <bool VARMU>
__device__ __forceinline__ void momentum_mean_tile(const DevPlan& P, const MomentumTileArgs& A) {
  extern __shared__ double lds_d[];
  const TileTab& T = P.tt;
  const int n2 = P.n2, np = pad16(n2), w = tile_wave(), lane = threadIdx.x & 63;
  double* y = lds_d;  // [np][2]
  double* z = y + 2 * np;
  double* tab = z + 2 * np;
  const size_t rs = 2 * size_t(P.nn) * P.nl;
  tile_fetch_tables(T, 0, tab, n2, w, lane);
  for (int t = threadIdx.x; t < 2 * np; t += kTileThreads) {
    const int i = t >> 1, ij = (t & 1) ? 4 : 1;
    double v = 0.0;
    if (i < n2) {
      v = A.C[ij][size_t(i) * rs];
      if constexpr (VARMU) {
        v += A.tau[ij][size_t(i) * rs];
      } else {
        const double* u = A.u[(t & 1) ? 2 : 0];
        const cptr<double> w1 = T.e + size_t(i) * kTERow + kTW;
        const int lo = T.elo[i];
        double d = 0.0;
#pragma unroll
        for (int q = 0; q < kTW; ++q) d = fma(w1[q], u[size_t(lo + q) * rs], d);
        v = fma(P.mu, d, v);
      }
    }
    y[t] = v;
  }
#pragma unroll 1
  for (int pass = 0; pass < 2; ++pass) {
    lds_fetched();
    if (threadIdx.x < 16)  // a full row of lanes for the broadcasts, two of them columns
      tile_solve<2>((pass ? z : y) + (threadIdx.x & 1), tab, n2, threadIdx.x);
    lds_barrier();
    if (pass) break;
    tile_fetch_tables(T, 2, tab, n2, w, lane);
    for (int t = threadIdx.x; t < 2 * np; t += kTileThreads) {
      const int i = t >> 1;
      double b = 0.0;
      if (i > 0 && i < n2 - 1) {
        const cptr<double> w1 = T.e + size_t(i) * kTERow + kTW;
        const int lo = T.elo[i];
#pragma unroll
        for (int q = 0; q < kTW; ++q) b = fma(w1[q], y[2 * (lo + q) + (t & 1)], b);
      }
      z[t] = b;
    }
  }
  for (int t = threadIdx.x; t < 2 * n2; t += kTileThreads) {
    const int i = t >> 1;
    const bool b = t & 1;
    const double x = z[t];
    double* ro = b ? A.r3o : A.r1o;
    if (ro) ro[i] = x;
    if (A.stage > 1) continue;
    const double m = (b ? A.m3 : A.m1)[i];
    (b ? A.m3o : A.m1o)[i] = A.stage == 0 ? m + 0.5 * P.dt * x : m + P.dt * (x - 0.5 * (b ? A.r3p : A.r1p)[i]);
  }
}
template <int CT, bool VARMU>
__device__ __forceinline__ void momentum_tile_body(const DevPlan& P, unsigned tile, unsigned part, const MomentumTileArgs& A) {
  constexpr int RS = 2 * CT;
  extern __shared__ double lds_d[];
  if (tile == A.tiles) {
    if (part == 0) momentum_mean_tile<VARMU>(P, A);
    return;
  }
  const TileTab& T = P.tt;
  const int n2 = P.n2, w = tile_wave(), lane = threadIdx.x & 63;
  const bool om = part == 0;
  const size_t fld = size_t(pad16(n2)) * RS;
  double* S = lds_d;                       // x0, x1: the sums; u1 (u2, the result), u3
  double* s = S + (lane & (RS - 1));
  double* u1 = s + 2 * fld;
  double* u3 = s + 3 * fld;
  double* spare = s + size_t(momentum_tile_rows(n2) - 1) * RS;
  double* tab = S + size_t(momentum_tile_rows(n2)) * RS;
  const TileLane L = tile_lane<CT, false>(P, tile, lane);
  const TileRows<CT> rows(n2, L, w, lane);
  const double k1 = L.k1, k3 = L.k3, ksq = k1 * k1 + k3 * k3, mu = P.mu;
  const unsigned bytes = unsigned(n2) * L.rs;
  if constexpr (!VARMU) {
    tile_fetch<CT>(S + 2 * fld, A.u[0], L, n2, w, lane);
    tile_fetch<CT>(S + 3 * fld, A.u[2], L, n2, w, lane);
  }
  tile_fetch_tables(T, 0, tab, n2, w, lane);
  {  // rows past the last one: zeros
    if (rows.r0 < n2 && rows.r0 + rows.R >= n2)
      for (int r = n2; r < pad16(n2); ++r) s[r * RS] = s[fld + r * RS] = 0.0;
  }
  lds_fetched();
  {  // x0 = a0 or b1, x1 = a1 or b2 (but for u2)
    const double c11 = om ? -k1 * k3 : k1 * k1, c13 = om ? k1 * k1 - k3 * k3 : 2.0 * k1 * k3, c22 = om ? 0.0 : -ksq,
                 c33 = om ? k1 * k3 : k3 * k3, sg = om ? 1.0 : -1.0, c12 = sg * (om ? k3 : k1), c23 = sg * (om ? -k1 : k3);
    const double f1 = om ? -mu * ksq * k3 : 2.0 * mu * ksq * k1, f3 = om ? mu * ksq * k1 : 2.0 * mu * ksq * k3;
    const TileBuf C[6] = {tile_buf(A.C[0], bytes), tile_buf(A.C[1], bytes), tile_buf(A.C[2], bytes),
                          tile_buf(om ? nullptr : A.C[3], bytes), tile_buf(A.C[4], bytes), tile_buf(A.C[5], bytes)};
    const TileBuf V[6] = {tile_buf(A.tau[0], bytes), tile_buf(A.tau[1], bytes), tile_buf(A.tau[2], bytes),
                          tile_buf(om ? nullptr : A.tau[3], bytes), tile_buf(A.tau[4], bytes), tile_buf(A.tau[5], bytes)};
    // the tables are read a group ahead, the six fields before the taps of their group
    struct Group {
      double t[VARMU ? 2 : 2 * kTW];
      int lo;
    };
    tile_groups(
        rows.R,
        [&](int k) __attribute__((always_inline)) {
          Group g;
          if constexpr (!VARMU) {
            const int tr = rows.template tab<4>(k, lane);
            load_row(g.t, T.e + size_t(tr) * kTERow);
            g.lo = T.elo[tr];
          }
          return g;
        },
        [&](int k, const Group& g) __attribute__((always_inline)) {
          double c[6][4], va[4], vb[4];
#pragma unroll
          for (int q = 0; q < 6; ++q)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              c[q][u] = gld(C[q], rows.at(k + u));
              if (VARMU) c[q][u] += gld(V[q], rows.at(k + u));
            }
          unrolled<0, 4>([&](auto uc) __attribute__((always_inline)) {
            constexpr int U = decltype(uc)::value;
            va[U] = vb[U] = 0.0;
            if constexpr (!VARMU) {
              double v[kTW], q[kTW], v0 = 0.0, v1 = 0.0, q0 = 0.0, q1 = 0.0;
              tile_taps<U, kTW, RS>(v, u1, g.lo);
              tile_taps<U, kTW, RS>(q, u3, g.lo);
              fb2x4<U>(v0, v1, g.t, g.t + kTW, v);
              fb2x4<U>(v0, v1, g.t + 4, g.t + kTW + 4, v + 4);
              fb2x4<U>(q0, q1, g.t, g.t + kTW, q);
              fb2x4<U>(q0, q1, g.t + 4, g.t + kTW + 4, q + 4);
              va[U] = times_i_lane(fma(f3, q0, f1 * v0), L.c);
              vb[U] = fma(mu * c23, q1, mu * c12 * v1);
            }
          });
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const double a = fma(c33, c[5][u], fma(c22, c[3][u], fma(c13, c[2][u], c11 * c[0][u]))) + va[u];
            const double b = times_i_lane(fma(c23, c[4][u], fma(c12, c[1][u], vb[u])), L.c);
            double* x = rows.put(s, k + u, spare);
            *x = a;
            *(x == spare ? spare : x + fld) = b;
          }
        });
  }
  lds_barrier();
  if constexpr (!VARMU) {
    if (!om) {  // u2 enters phi2 only
      tile_fetch<CT>(S + 2 * fld, A.u[1], L, n2, w, lane);
      lds_fetched();
      struct Group {
        double t[2 * kTW];
        int lo;
      };
      tile_groups(
          rows.R,
          [&](int k) __attribute__((always_inline)) {
            Group g;
            const int tr = rows.template tab<4>(k, lane);
            load_row(g.t, T.e + size_t(tr) * kTERow);
            g.lo = T.elo[tr];
            return g;
          },
          [&](int k, const Group& g) __attribute__((always_inline)) {
            double z[4][2];
            unrolled<0, 4>([&](auto uc) __attribute__((always_inline)) {
              constexpr int U = decltype(uc)::value;
              double v[kTW], e0 = 0.0, e1 = 0.0;
              tile_taps<U, kTW, RS>(v, u1, g.lo);
              fb2x4<U>(e0, e1, g.t, g.t + kTW, v);
              fb2x4<U>(e0, e1, g.t + 4, g.t + kTW + 4, v + 4);
              const double* x = rows.put(s, k + U, spare);
              z[U][0] = fma(-2.0 * mu * ksq, e1, x[0]);
              z[U][1] = fma(mu * ksq, e0, *(x == spare ? spare : x + fld));
            });
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              double* x = rows.put(s, k + u, spare);
              *x = z[u][0];
              *(x == spare ? spare : x + fld) = z[u][1];
            }
          });
      lds_barrier();
    }
  }
  if (w < 2 && lane < RS) tile_solve<RS>(S + w * fld + lane, tab, n2, lane);
  lds_barrier();
  tile_fetch_tables(T, 1, tab, n2, w, lane);
  {  // the right-hand side at tau, 0 at the Dirichlet rows
    const TileBuf rho = tile_buf(om ? nullptr : A.rho, bytes);
    const double gk = ksq * P.g;
    struct Group {
      double t[kTERow], r[4];
      int lo;
    };
    tile_groups(
        rows.R,
        [&](int k) __attribute__((always_inline)) {
          Group g;
          const int tr = rows.template tab<4>(k, lane);
          load_row(g.t, T.e + size_t(tr) * kTERow);
          g.lo = T.elo[tr];
#pragma unroll
          for (int u = 0; u < 4; ++u) g.r[u] = gld(rho, rows.at(k + u));
          return g;
        },
        [&](int k, const Group& g) __attribute__((always_inline)) {
          double z[4];
          unrolled<0, 4>([&](auto uc) __attribute__((always_inline)) {
            constexpr int U = decltype(uc)::value;
            double v[kTW], q[kTW], p0 = 0.0, p1 = 0.0, q0 = 0.0, q1 = 0.0, q2 = 0.0;
            tile_taps<U, kTW, RS>(v, s, g.lo);
            tile_taps<U, kTW, RS>(q, s + fld, g.lo);
            fb2x4<U>(p0, p1, g.t, g.t + kTW, v);
            fb2x4<U>(p0, p1, g.t + 4, g.t + kTW + 4, v + 4);
            fb3x4<U>(q0, q1, q2, g.t, g.t + kTW, g.t + 2 * kTW, q);
            fb3x4<U>(q0, q1, q2, g.t + 4, g.t + kTW + 4, g.t + 2 * kTW + 4, q + 4);
            const int row = rows.r0 + k + U;
            z[U] = om ? p0 + q1 : fma(gk, g.r[U], fma(ksq, q0, q2) + p1);
            if (row == 0 || row == n2 - 1) z[U] = 0.0;
          });
#pragma unroll
          for (int u = 0; u < 4; ++u) *rows.put(u1, k + u, spare) = z[u];
        });
    if (rows.r0 < n2 && rows.r0 + rows.R >= n2)
      for (int r = n2; r < pad16(n2); ++r) u1[r * RS] = 0.0;
  }
  lds_fetched();
  if (w == 0 && lane < RS) tile_solve<RS>(S + 2 * fld + lane, tab, n2, lane);
  lds_barrier();
  const bool upd = A.stage <= 1;
  const TileBuf in = tile_buf(upd ? (om ? A.om : A.phi) : nullptr, bytes),
                prev = tile_buf(A.stage == 1 ? (om ? A.rom_prev : A.rphi_prev) : nullptr, bytes),
                out = tile_buf(upd ? (om ? A.om_out : A.phi_out) : nullptr, bytes),
                rout = tile_buf(om ? A.rom_out : A.rphi_out, bytes);
  struct Group {
    double a[4], b[4];
  };
  tile_groups(
      rows.R,
      [&](int k) __attribute__((always_inline)) {
        Group g;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          g.a[u] = gld(in, rows.at(k + u));
          g.b[u] = gld(prev, rows.at(k + u));
        }
        return g;
      },
      [&](int k, const Group& g) __attribute__((always_inline)) {
        double z[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) z[u] = u1[min(rows.r0 + k + u, n2 - 1) * RS];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const unsigned o = rows.st(k + u);
          gst(rout, o, z[u]);
          gst(out, o, A.stage == 0 ? fma(0.5 * P.dt, z[u], g.a[u]) : fma(P.dt, z[u] - 0.5 * g.b[u], g.a[u]));
        }
      });
}
template <int CT, bool VARMU>
__global__ void __launch_bounds__(kTileThreads) k_momentum_tile(DevPlan P, MomentumTileArgs A) {
  momentum_tile_body<CT, VARMU>(P, blockIdx.x, blockIdx.y, A);
}

// ---------------------------------------------------------------------------
// jobs of the tile kernels (single launches and grouped ones)
struct TileJob {
  static constexpr int kBound = kTileThreads, kBlock = kTileThreads, kMinBlocks = 0;
};
template <int CT>
struct JobMcTile : TileJob {
  using Args = McTileArgs;
  __device__ static void run(const DevPlan& P, unsigned bx, unsigned, unsigned, const Args& A) { mc_tile_body<CT>(P, bx, A); }
  static void launch(dim3 g, size_t lds, hipStream_t s, const DevPlan& P, const Args& A) {
    hipLaunchKernelGGL(k_mc_tile<CT>, g, dim3(kTileThreads), lds, s, P, A);
  }
};
template <int CT, int EPI>
struct JobProjTile : TileJob {
  using Args = ProjTileArgs;
  __device__ static void run(const DevPlan& P, unsigned bx, unsigned by, unsigned, const Args& A) {
    proj_tile_body<CT, EPI>(P, bx, by, A);
  }
  static void launch(dim3 g, size_t lds, hipStream_t s, const DevPlan& P, const Args& A) {
    hipLaunchKernelGGL((k_proj_tile<CT, EPI>), g, dim3(kTileThreads), lds, s, P, A);
  }
};
template <int CT>
struct JobPrologueTile : TileJob {
  struct Args {
    MdArgs M;
    ValuesZArgs Z;
    GuessArgs G;
  };
  __device__ static void run(const DevPlan& P, unsigned bx, unsigned by, unsigned, const Args& A) {
    prologue_tile_body<CT>(P, bx, by, A.M, A.Z, A.G);
  }
  static void launch(dim3 g, size_t lds, hipStream_t s, const DevPlan& P, const Args& A) {
    hipLaunchKernelGGL(k_prologue_tile<CT>, g, dim3(kTileThreads), lds, s, P, A.M, A.Z, A.G);
  }
};
template <int CT, bool VARMU>
struct JobMomentumTile : TileJob {
  using Args = MomentumTileArgs;
  __device__ static void run(const DevPlan& P, unsigned bx, unsigned by, unsigned, const Args& A) {
    momentum_tile_body<CT, VARMU>(P, bx, by, A);
  }
  static void launch(dim3 g, size_t lds, hipStream_t s, const DevPlan& P, const Args& A) {
    hipLaunchKernelGGL((k_momentum_tile<CT, VARMU>), g, dim3(kTileThreads), lds, s, P, A);
  }
};
template <int CT>
struct JobStrainTile : TileJob {
  using Args = StrainTileArgs;
  __device__ static void run(const DevPlan& P, unsigned bx, unsigned, unsigned, const Args& A) { strain_tile_body<CT>(P, bx, A); }
  static void launch(dim3 g, size_t lds, hipStream_t s, const DevPlan& P, const Args& A) {
    hipLaunchKernelGGL(k_strain_tile<CT>, g, dim3(kTileThreads), lds, s, P, A);
  }
};

