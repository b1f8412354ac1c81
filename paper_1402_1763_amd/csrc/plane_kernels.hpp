// The two-pass sweep of grid sides up to 128 (gfx950).
//
// Up to N = 128 the (kz, iy) plane of one ix fits the LDS of a CU (70 KB of
// 160 KB in FP32, 147 KB in FP64 at 128), so the y transforms join the z-pass
// in one kernel and a sweep is two launches instead of four, with half the
// spectrum traffic:
//   plane  : inverse y-DFT, inverse z-DFT (-> s), messenger draw, forward
//            z-DFT, forward y-DFT of one (kz, iy) plane; the P(k) draw of the
//            sweep before in extra workgroups
//   column : forward x-DFT (-> t^), signal draw, shell sums, inverse x-DFT
// n sweeps run plane without its inverse y-DFT, column, then (plane, column)
// n - 1 times, and last the inverse y-DFT alone with the last P(k) draw, so
// the state between calls is the four-pass schedule's (transformed along z
// only).  The plane kernel's parts are template switches of one piece of code:
// joined or launched one by one they compute the same values bit for bit.
//
// The planes kz = 0 and kz = N/2 are real before the y-DFT, and run as one
// complex row F_0 + i F_{N/2}: a plane is N/2 rows, as many as it has pairs of
// z pencils.
#pragma once

#include <type_traits>

#include "sweep_kernels.hpp"

namespace mf {

template <int N>
__host__ __device__ constexpr bool has_planes() { return N <= 128; }

// Radix schedule of the plane path.  A stage's butterflies are dealt to the
// threads one by one (no thread keeps a fixed set of elements), so a stage may
// leave threads idle and radices need no common multiple.  FP32 takes few
// large stages (each costs an LDS round trip and two barriers); FP64 small
// ones, because the last z and x stages also draw: a thread draws one or two
// normals of FP64 log and sincos per element, in series.  The last radix is a
// multiple of 4 (a Philox call serves n, n + N/4, n + N/2, n + 3N/4).
template <int N, bool FP64>
struct PlaneRadices;
//
// nt threads run a plane where there are no more planes than CUs: as many as
// the last stage has butterflies, since a lone workgroup's time is its longest
// chain.  ntb threads where planes queue: fewer, so that a CU overlaps the
// barriers and memory waits of several workgroups.  At 128 in FP64 that leaves
// 128 registers a thread, and 25 to 59 are spilled: 64.3 us a sweep; with 512
// threads none is, but it takes 69.2, with 768 68.5.
#define MF_RADICES(NN, D, COUNT, A, B, C, NT_, NTB_)                                       \
  template <> struct PlaneRadices<NN, D> {                                                 \
    static constexpr int n = COUNT, nt = NT_, ntb = NTB_;                                  \
    static constexpr int r[3] = {A, B, C};                                                 \
  };
MF_RADICES(8, false, 2, 2, 4, 1, 64, 64)
MF_RADICES(16, false, 2, 4, 4, 1, 64, 64)
MF_RADICES(32, false, 2, 8, 4, 1, 128, 128)
MF_RADICES(48, false, 3, 3, 4, 4, 320, 320)
MF_RADICES(64, false, 2, 8, 8, 1, 256, 256)
MF_RADICES(80, false, 3, 5, 4, 4, 832, 448)
MF_RADICES(96, false, 3, 6, 4, 4, 1024, 1024)
MF_RADICES(128, false, 2, 16, 8, 1, 1024, 512)
MF_RADICES(8, true, 2, 2, 4, 1, 64, 64)
MF_RADICES(16, true, 2, 4, 4, 1, 64, 64)
MF_RADICES(32, true, 2, 8, 4, 1, 128, 128)
MF_RADICES(48, true, 3, 3, 4, 4, 320, 320)
MF_RADICES(64, true, 3, 4, 4, 4, 512, 512)
MF_RADICES(80, true, 3, 5, 4, 4, 832, 832)
MF_RADICES(96, true, 3, 6, 4, 4, 576, 576)
MF_RADICES(128, true, 3, 8, 4, 4, 1024, 1024)
#undef MF_RADICES

__host__ __device__ constexpr int round_up(int n, int m) { return (n + m - 1) / m * m; }

// The LDS that transforms pass their elements through: p, in one buffer or in
// two by turns.  With one, every thread must be done reading it (drain) before
// it is written again; with two, the barrier between writing the other one and
// reading it says so, too, and half of the barriers go.
template <class T, int SIZE, bool TWO>
struct Exchange {
  T* p;
  T* other;
  __device__ __forceinline__ explicit Exchange(T* lds) : p(lds), other(TWO ? lds + SIZE : lds) {}
  __device__ __forceinline__ void drain() const {
    if (!TWO) __syncthreads();
  }
  __device__ __forceinline__ void turn() {   // before each write
    T* t = p;
    p = other;
    other = t;
  }
};

// One batch of NPEN transforms of length N by NT threads, its stages in the
// schedule's order or (REV) backwards.  PENFAST: neighbouring lanes take
// neighbouring pencils, else neighbouring butterflies of one pencil.
template <typename R, int N, class Sch, int NPEN, int NT_, bool PENFAST>
struct Batch {
  static constexpr int NT = NT_;
  static constexpr int STAGES = Sch::n;
  template <bool REV>
  __host__ __device__ static constexpr int radix(int s) { return Sch::r[REV ? STAGES - 1 - s : s]; }
  template <bool REV>
  __host__ __device__ static constexpr int span(int s) {   // product of the earlier radices
    int ns = 1;
    for (int t = 0; t < s; ++t) ns *= radix<REV>(t);
    return ns;
  }
  __host__ __device__ static constexpr int slots(int rad) {
    return (NPEN * (N / rad) + NT - 1) / NT;
  }
  __host__ __device__ static constexpr int regs() {   // complex registers of the widest stage
    int m = 0;
    for (int s = 0; s < STAGES; ++s)
      m = slots(Sch::r[s]) * Sch::r[s] > m ? slots(Sch::r[s]) * Sch::r[s] : m;
    return m;
  }
  static constexpr int REGS = regs();
  // Butterfly of slot i in a stage of radix RAD: false past the last one.
  template <int RAD>
  __device__ __forceinline__ static bool at(int i, int& pen, int& q) {
    constexpr int BPP = N / RAD, TOT = NPEN * BPP;
    const int bf = threadIdx.x + i * NT;
    if (PENFAST) {
      pen = bf % NPEN;
      q = bf / NPEN;
    } else {
      pen = bf / BPP;
      q = bf % BPP;
    }
    if (TOT % NT != 0 && bf >= TOT) return false;
    __builtin_assume(pen >= 0 && pen < NPEN && q >= 0 && q < BPP);
    return true;
  }
  // Stage S: read(pen, pos) gives the inputs; fix(pen, q, BPP, x) may then
  // replace some of a butterfly's inputs x[r], which sit at q + r BPP (one
  // branch per butterfly instead of one per input: loads under a condition of
  // their own would go out one by one).
  struct NoFix {
    template <class Step>
    __device__ __forceinline__ void operator()(int, int, Step, const cx<R>*) const {}
  };
  template <int K>
  using Int = std::integral_constant<int, K>;
  template <int S, bool INV, bool REV, class Read, class Fix = NoFix>
  __device__ __forceinline__ static void in(cx<R>* v, const cx<R>* tw, Read read, Fix fix = Fix()) {
    constexpr int RAD = radix<REV>(S), NS = span<REV>(S), BPP = N / RAD;
#pragma unroll
    for (int i = 0; i < slots(RAD); ++i) {
      int pen = 0, q = 0;
      if (!at<RAD>(i, pen, q)) continue;
      cx<R>* x = v + i * RAD;
#pragma unroll
      for (int r = 0; r < RAD; ++r) x[r] = read(pen, q + r * BPP);
      fix(pen, q, Int<BPP>(), x);
      if (NS > 1) {
        const int k = q % NS;
#pragma unroll
        for (int r = 1; r < RAD; ++r) {
          const cx<R> w = tw[r * k * (N / (NS * RAD))];
          x[r] = INV ? cmulc(x[r], w) : cmul(x[r], w);
        }
      }
      dft<R, RAD, INV>(x);
    }
  }
  // Stage S's outputs through write(pen, pos, value), then fix(pen, pos0, step,
  // x) for a butterfly's outputs x[r] at pos0 + r step.
  template <int S, bool REV, class Write, class Fix = NoFix>
  __device__ __forceinline__ static void out(const cx<R>* v, Write write, Fix fix = Fix()) {
    constexpr int RAD = radix<REV>(S), NS = span<REV>(S);
#pragma unroll
    for (int i = 0; i < slots(RAD); ++i) {
      int pen = 0, q = 0;
      if (!at<RAD>(i, pen, q)) continue;
      const int base = (q / NS) * NS * RAD + q % NS;
#pragma unroll
      for (int r = 0; r < RAD; ++r) write(pen, base + r * NS, v[i * RAD + r]);
      fix(pen, base, Int<NS>(), v + i * RAD);
    }
  }
  // The stages after the first, whose results sit in v: through LDS at
  // idx(pen, pos), which must be free with one buffer; the last stage's results
  // stay in v.  Other threads may still read the LDS on return.
  template <bool INV, bool REV, class Lds, class Idx>
  __device__ __forceinline__ static void rest(cx<R>* v, const cx<R>* tw, Lds& lds, Idx idx) {
    auto rd = [&](int pen, int pos) { return lds.p[idx(pen, pos)]; };
    auto wr = [&](int pen, int pos, cx<R> z) { lds.p[idx(pen, pos)] = z; };
    if constexpr (STAGES > 1) {
      lds.turn();
      out<0, REV>(v, wr);
      __syncthreads();
      in<1, INV, REV>(v, tw, rd);
    }
    if constexpr (STAGES > 2) {
      lds.drain();
      lds.turn();
      out<1, REV>(v, wr);
      __syncthreads();
      in<2, INV, REV>(v, tw, rd);
    }
  }
};

// ---------------------------------------------------------------- plane
template <typename R, int N, bool MANY = false>
struct PlaneTile {
  static constexpr int H = N / 2;
  using Sch = PlaneRadices<N, sizeof(R) == 8>;
  static constexpr int RL = Sch::r[Sch::n - 1];       // radix of the draw's stage
  static constexpr int NT = MANY ? Sch::ntb : Sch::nt;
  // waves per SIMD that fit two workgroups of a CU's LDS, where that is all
  static constexpr int WAVES = MANY && NT == 512 ? 4 : 1;
  static constexpr int PADS = pow2<Sch::r[0]>() ? ilog2(Sch::r[0]) : 2;
  static constexpr int YSTR = N + (N >> PADS), ZSTR = N + 1;
  static constexpr int FIELD = H * (YSTR > ZSTR ? YSTR : ZSTR);
  static constexpr int LDS = FIELD > NT ? FIELD : NT;   // NT: the P(k) sums' reduction
  // Two exchange buffers where planes do not queue and both fit: us per sweep
  // with one : two, one chain, 80^3 FP64 29.5 : 28.5, 96^3 FP32 22.4 : 21.4, 128^3
  // FP32 28.7 : 28.2 (8 chains of 96^3, which lose a CU's second workgroup,
  // 60.4 : 60.9).
  static constexpr bool TWO = !MANY && (2 * LDS + 2 * N) * sizeof(cx<R>) <= 160 * 1024;
  // queues of planes have a kernel of their own: other threads, or two buffers
  // would leave a CU one workgroup
  static constexpr bool QUEUES =
      Sch::nt != Sch::ntb || (TWO && 4 * LDS * sizeof(cx<R>) > 160 * 1024);
  using Y = Batch<R, N, Sch, H, NT, false>;
  using Z = Batch<R, N, Sch, H, NT, true>;
  static constexpr int REGS = Y::REGS > Z::REGS ? Y::REGS : Z::REGS;
  __device__ __forceinline__ static int yidx(int row, int i) { return row * YSTR + i + (i >> PADS); }
  __device__ __forceinline__ static int zidx(int pen, int k) { return pen * ZSTR + k; }
};

// Index of the coefficient entry (z-pass order) of the voxels (ix, 2 p, n) and
// (ix, 2 p + 1, n): the inverse of zpass_coef_voxel, with the z tile and the
// element in it.
template <typename R, int N>
__host__ __device__ __forceinline__ int coef_entry(int ix, int p, int n, int& tile, int& e) {
  using T = ZTile<R, N>;
  constexpr int RZ = radix_at<N, false>(Radices<N>::n - 1), NSL = N / RZ;
  const int iya = 2 * p;
  tile = (ix / T::IXB) * (N / T::P) + iya / T::P;
  const int bf = (ix % T::IXB) * T::NPAIR + (iya % T::P) / 2 + T::NPEN * (n % NSL);
  e = bf / T::NT * RZ + n / NSL;
  return (tile * T::EPT + e) * T::NT + bf % T::NT;
}

enum : int { kNoZ = -1 };   // ZMODE of a plane kernel without its z part
// What a plane kernel does besides its plane: gamma variates of the P draws in
// extra workgroups, the update of the recorded moments.
enum : int { kWithGammas = 1, kWithMoments = 2 };

// One (kz, iy) plane of one ix: the parts YI (inverse y-DFT), ZMODE (inverse
// z-DFT, messenger step kZSweep or kZDet, forward z-DFT) and YF (forward
// y-DFT), reading a.spec_in and writing a.spec.  With YI the first nb
// workgroups of a chain finish the P(k) step of the sweep before (pk_mode).
//
// The gamma variates of those steps take 116 registers and some 3 us of one
// thread, but depend on the bin, the sweep and the chain alone.  Only the first
// launch of a run and every kGammaAhead-th one have them (X & kWithGammas):
// a.gam_wgs more workgroups per chain compute those of this sweep and the
// following ones, a.gam_sweeps in all, one per thread.  Only launches of recorded
// sweeps update the moments (X & kWithMoments); the others keep the registers
// of the transforms.  us per recorded sweep with the gamma variates in all of
// them : without, FP32, 16 chains of 48^3 39.9 : 29.3, 8 of 80^3 61.5 : 60.1.
// With NORM the messenger's normals come from a.nrm, where the column kernel
// before put them (column_kernel, AHEAD).
template <typename R, int N, bool YI, int ZMODE, bool YF, int X = 0, bool MANY = false,
          bool NORM = false>
__global__ void __launch_bounds__((PlaneTile<R, N, MANY>::NT), (PlaneTile<R, N, MANY>::WAVES))
plane_kernel(SweepArgs<R> a) {
  using T = PlaneTile<R, N, MANY>;
  using Y = typename T::Y;
  using Z = typename T::Z;
  constexpr int H = N / 2, NT = T::NT;
  constexpr bool ZP = ZMODE != kNoZ;
  __shared__ cx<R> field[T::TWO ? 2 * T::LDS : T::LDS];
  __shared__ cx<R> tw[N];
  __shared__ cx<R> row0[N];
  static_assert(T::LDS * sizeof(cx<R>) >= NT * sizeof(double), "reduction space");
  Exchange<cx<R>, T::LDS, T::TWO> lds(field);
  const int tid = threadIdx.x, c = blockIdx.z;
  int ix = blockIdx.x;
  if (X & kWithGammas) {
    if (ix < a.gam_wgs) {
      const uint32_t first = a.ctr[0];
      for (int it = ix * NT + tid; it < a.gam_sweeps * a.nb; it += a.gam_wgs * NT) {
        const uint32_t n = first + it / a.nb;
        const int b = it % a.nb;
        a.gam[(static_cast<size_t>(n % kGammaSlots) * a.gam_chains + c) * a.nb + b] =
            a.counts[b] > 0.0 ? gamma_mt(0.5 * a.counts[b] + a.prior_a, static_cast<uint32_t>(b), n,
                                         a.chain0 + c, a.key0, a.key1) : 0.0;
      }
      return;
    }
    ix -= a.gam_wgs;
  }
  if (YI) {
    if (ix < a.nb) {
      // with the z part, slot 0 of the counter already counts this sweep
      pk_draw_block<R, NT, true>(a, ix, c, reinterpret_cast<double*>(field), ZP ? a.ctr[0] - 1u : a.ctr[1]);
      return;
    }
    ix -= pk_blocks(a.nb);
    if (ix < 0) return;
  }
  const cx<R>* src = a.spec_in + static_cast<size_t>(c) * a.spec_stride + static_cast<size_t>(ix) * N;
  cx<R>* dst = a.spec + static_cast<size_t>(c) * a.spec_stride + static_cast<size_t>(ix) * N;
  constexpr uint32_t ROW = N * N;   // from one kz to the next
  load_twiddles(tw, a.tw, N, NT);
  cx<R> v[T::REGS];
  auto ylds = [&](int row, int i) { return T::yidx(row, i); };
  auto zlds = [&](int pen, int k) { return T::zidx(pen, k); };

  if (YI) {
    Y::template in<0, true, false>(
        v, tw, [&](int row, int i) { return src[static_cast<uint32_t>(row * N * N + i)]; },
        [&](int row, int q, auto bpp, cx<R>* x) {
          if (row != 0) return;
#pragma unroll
          for (int r = 0; r < Y::template radix<false>(0); ++r) {
            const cx<R> w = src[H * ROW + q + r * bpp];
            x[r] = cx<R>{x[r].x - w.y, x[r].y + w.x};
          }
        });
    Y::template rest<true, false>(v, tw, lds, ylds);
    if (!ZP) {
      Y::template out<Y::STAGES - 1, false>(
          v, [&](int row, int i, cx<R> y) { dst[static_cast<uint32_t>(row * N * N + i)] = y; },
          [&](int row, int i0, auto step, const cx<R>* x) {
            if (row != 0) return;
#pragma unroll
            for (int r = 0; r < T::RL; ++r) {
              dst[i0 + r * step] = cx<R>{x[r].x, R(0)};
              dst[H * ROW + i0 + r * step] = cx<R>{x[r].y, R(0)};
            }
          });
    } else {
      lds.drain();
      lds.turn();
      Y::template out<Y::STAGES - 1, false>(v, [&](int row, int i, cx<R> y) { lds.p[T::yidx(row, i)] = y; });
      __syncthreads();
    }
  }

  if constexpr (ZP) {
    const uint32_t sweep = a.ctr[0];
    if (ZMODE == kZSweep && ix == 0 && c == 0 && tid == 0) a.ctr[1] = sweep;
    // Z_k = A_k + i B_k of the pencils iy = 2 p and 2 p + 1
    auto pack = [](int k, cx<R> A, cx<R> B) {
      return k < H ? cx<R>{A.x - B.y, A.y + B.x} : cx<R>{A.x + B.y, B.x - A.y};
    };
    if (YI) {
      Z::template in<0, true, false>(
          v, tw, [&](int p, int k) {
            const int row = k <= H ? k % H : N - k;
            return pack(k, lds.p[T::yidx(row, 2 * p)], lds.p[T::yidx(row, 2 * p + 1)]);
          },
          [&](int p, int q, auto bpp, cx<R>* x) {   // k = 0 and k = H share row 0
            const cx<R> A = lds.p[T::yidx(0, 2 * p)], B = lds.p[T::yidx(0, 2 * p + 1)];
            if (q == 0) x[0] = cx<R>{A.x, B.x};
            if (q == H % bpp) x[H / bpp] = cx<R>{A.y, B.y};
          });
    } else {
      Z::template in<0, true, false>(v, tw, [&](int p, int k) {
        cx<R> A, B;
        ld2(src + static_cast<uint32_t>((k <= H ? k : N - k) * N * N + 2 * p), A, B);
        if (k == 0 || k == H) A.y = B.y = R(0);
        return pack(k, A, B);
      });
    }
    lds.drain();   // the rows are read
    Z::template rest<true, false>(v, tw, lds, zlds);

    constexpr int RL = T::RL, NSL = N / RL;
    constexpr bool kXor3 = sizeof(R) == 4;
    // a wave loads an element's coefficients where any of its lanes' tiles has an
    // observed voxel in it; they are (1, 0) elsewhere, stored or not
    const uint32_t* obs = a.tile_obs + static_cast<size_t>(c) * a.ztiles;
    const R* coef = a.coef + static_cast<size_t>(c) * 2 * a.m;
    const int rec = (X & kWithMoments) && ZMODE == kZSweep && a.mom != nullptr ? recorded(a, sweep) : -1;
#pragma unroll
    for (int i = 0; i < Z::slots(RL); ++i) {
      int p = 0, q = 0;
      if (!Z::template at<RL>(i, p, q)) continue;
      cx<R>* s = v + i * RL;
      if ((X & kWithMoments) && rec >= 0) {   // Welford update with the (rec + 1)-th sample
        const double inv_k = 1.0 / (rec + 1.0);
        double* mean = a.mom + static_cast<size_t>(c) * 2 * a.m;
        double* m2 = mean + a.m;
#pragma unroll
        for (int r = 0; r < RL; ++r) {
          int tile = 0, e = 0;
          const size_t j = static_cast<size_t>(coef_entry<R, N>(ix, p, q + r * NSL, tile, e)) * 2;
          const double x0 = s[r].x, x1 = s[r].y;
          const double u0 = mean[j], u1 = mean[j + 1];
          const double n0 = u0 + (x0 - u0) * inv_k, n1 = u1 + (x1 - u1) * inv_k;
          mean[j] = n0;
          mean[j + 1] = n1;
          m2[j] += (x0 - u0) * (x0 - n0);
          m2[j + 1] += (x1 - u1) * (x1 - n1);
        }
      }
      if (ZMODE == kZDet) {
        R* acc = a.acc == nullptr ? nullptr : a.acc + static_cast<size_t>(c) * a.m;
        const R cb = a.cb_over_tau ? static_cast<R>(static_cast<double>(a.cb) / a.tau[c]) : a.cb;
#pragma unroll
        for (int r = 0; r < RL; ++r) {
          int tile = 0, e = 0;
          const int j = coef_entry<R, N>(ix, p, q + r * NSL, tile, e);
          R cf[4] = {R(1), R(1), R(0), R(0)};
          if (__any(obs[tile] >> e & 1u)) ld4(coef + static_cast<uint32_t>(j) * 4, cf);
          if (acc != nullptr) {
            acc[static_cast<size_t>(j) * 2] += s[r].x;
            acc[static_cast<size_t>(j) * 2 + 1] += s[r].y;
          }
          s[r] = cx<R>{a.cs * cf[0] * s[r].x + cb * cf[2], a.cs * cf[1] * s[r].y + cb * cf[3]};
        }
      } else if (NORM) {
        const R tau = static_cast<R>(a.tau[c]);
        const cx<R>* nrm = a.nrm + static_cast<size_t>(c) * (a.m / 2);
#pragma unroll
        for (int r = 0; r < RL; ++r) {
          int tile = 0, e = 0;
          const int j = coef_entry<R, N>(ix, p, q + r * NSL, tile, e);
          R cf[4] = {R(1), R(1), R(0), R(0)};
          if (__any(obs[tile] >> e & 1u)) ld4(coef + static_cast<uint32_t>(j) * 4, cf);
          const cx<R> g = nrm[static_cast<uint32_t>(j)];
          s[r] = cx<R>{cf[0] * s[r].x + cf[2] + noise_amp(tau * cf[0]) * g.x,
                       cf[1] * s[r].y + cf[3] + noise_amp(tau * cf[1]) * g.y};
        }
      } else {
        const R tau = static_cast<R>(a.tau[c]);
        const uint32_t chain = a.chain0 + c;
        const uint32_t wa = static_cast<uint32_t>((ix * N + 2 * p) * (N / 4) + q);
#pragma unroll
        for (int cq = 0; cq < RL / 4; ++cq) {
          R ga[4], gb[4];
          {
            const Words4 w = philox4x32_10<kXor3>(wa + NSL * cq, sweep, kPhaseMessenger, chain, a.key0, a.key1);
            box_muller(w.x0, w.x1, ga[0], ga[1]);
            box_muller(w.x2, w.x3, ga[2], ga[3]);
          }
          {
            const Words4 w = philox4x32_10<kXor3>(wa + N / 4 + NSL * cq, sweep, kPhaseMessenger, chain,
                                           a.key0, a.key1);
            box_muller(w.x0, w.x1, gb[0], gb[1]);
            box_muller(w.x2, w.x3, gb[2], gb[3]);
          }
#pragma unroll
          for (int j4 = 0; j4 < 4; ++j4) {
            const int r = cq + j4 * (RL / 4);
            int tile = 0, e = 0;
            const int j = coef_entry<R, N>(ix, p, q + r * NSL, tile, e);
            R cf[4] = {R(1), R(1), R(0), R(0)};
            if (__any(obs[tile] >> e & 1u)) ld4(coef + static_cast<uint32_t>(j) * 4, cf);
            s[r] = cx<R>{cf[0] * s[r].x + cf[2] + noise_amp(tau * cf[0]) * ga[j4],
                         cf[1] * s[r].y + cf[3] + noise_amp(tau * cf[1]) * gb[j4]};
          }
        }
      }
      // the forward transform's first stage works on the same registers
      dft<R, RL, false>(s);
      __builtin_amdgcn_sched_barrier(0);   // one slot's draws at a time: fewer registers
    }
    lds.drain();   // the inverse transform's reads
    Z::template rest<false, true>(v, tw, lds, zlds);
    if constexpr (Z::STAGES > 1) lds.drain();
    lds.turn();
    Z::template out<Z::STAGES - 1, true>(v, [&](int p, int k, cx<R> w) { lds.p[T::zidx(p, k)] = w; });
    __syncthreads();
    if (!YF) {
      for (int it = tid; it < (H + 1) * H; it += NT) {
        const int k = it / H, p = it % H;
        const cx<R> u = lds.p[T::zidx(p, k)], w = lds.p[T::zidx(p, (N - k) % N)];
        st2(dst + k * ROW + 2 * p, cx<R>{R(0.5) * (u.x + w.x), R(0.5) * (u.y - w.y)},
            cx<R>{R(0.5) * (u.y + w.y), R(0.5) * (w.x - u.x)});
      }
    }
  }

  if constexpr (YF) {
    if (ZP) {
      // row k: A_k = (W_k + conj W_{N-k}) / 2 at even i, B_k = (W_k - conj
      // W_{N-k}) / (2 i) at odd i; row 0: the real F_0 and F_{N/2}
      Y::template in<0, false, true>(
          v, tw, [&](int row, int i) {
            const cx<R> u = lds.p[T::zidx(i / 2, row)], w = lds.p[T::zidx(i / 2, N - row)];
            const bool odd = i % 2 != 0;
            const R a0 = odd ? u.y : u.x, a1 = odd ? w.y : w.x;
            const R b0 = odd ? w.x : u.y, b1 = odd ? u.x : w.y;
            return cx<R>{R(0.5) * (a0 + a1), R(0.5) * (b0 - b1)};
          },
          [&](int row, int q, auto bpp, cx<R>* x) {
            if (row != 0) return;
#pragma unroll
            for (int r = 0; r < Y::template radix<true>(0); ++r) {
              const int i = q + r * bpp;
              const cx<R> u = lds.p[T::zidx(i / 2, 0)], w = lds.p[T::zidx(i / 2, H)];
              x[r] = i % 2 != 0 ? cx<R>{u.y, w.y} : cx<R>{u.x, w.x};
            }
          });
      lds.drain();
    } else {
      Y::template in<0, false, true>(
          v, tw, [&](int row, int i) { return src[static_cast<uint32_t>(row * N * N + i)]; },
          [&](int row, int q, auto bpp, cx<R>* x) {
            if (row != 0) return;
#pragma unroll
            for (int r = 0; r < Y::template radix<true>(0); ++r) x[r].y = src[H * ROW + q + r * bpp].x;
          });
    }
    Y::template rest<false, true>(v, tw, lds, ylds);
    // row 0 goes out as it is, too, and is written again below
    Y::template out<Y::STAGES - 1, true>(
        v, [&](int row, int i, cx<R> y) { dst[static_cast<uint32_t>(row * N * N + i)] = y; },
        [&](int row, int i0, auto step, const cx<R>* x) {
          if (row != 0) return;
#pragma unroll
          for (int r = 0; r < Y::template radix<true>(Y::STAGES - 1); ++r) row0[i0 + r * step] = x[r];
        });
    __syncthreads();
    for (int i = tid; i < N; i += NT) {
      const cx<R> u = row0[i], w = row0[(N - i) % N];
      dst[i] = cx<R>{R(0.5) * (u.x + w.x), R(0.5) * (u.y - w.y)};
      dst[H * ROW + i] = cx<R>{R(0.5) * (u.y + w.y), R(0.5) * (w.x - u.x)};
    }
  }
}

// ---------------------------------------------------------------- column
// P neighbouring iy columns of one kz plane: runs of 128 bytes in FP32, 256 in
// FP64, where N allows.  FP32 takes no radix above 8 at 128 (66 VGPRs: {8, 4, 4}
// 35.8 us for 8 chains, {16, 8} 44 with 32 columns, 36 with 16; 8 columns 45);
// the smallest FP64 grids end on radix 2, so that a thread draws two modes
// instead of four (16^3 7.3 -> 6.1 us, 32^3 8.2 -> 6.5).  One exchange buffer:
// several workgroups share a CU and cover each other's barriers (two buffers:
// one chain of 96^3 21.3 against 21.4 us a sweep, 8 of them 61.7 against 60.9).
template <int N, bool FP64>
struct ColRadices;
#define MF_RADICES(NN, D, COUNT, A, B, C, P_, NT_)                                         \
  template <> struct ColRadices<NN, D> {                                                   \
    static constexpr int n = COUNT, p = P_, nt = NT_;                                      \
    static constexpr int r[3] = {A, B, C};                                                 \
  };
MF_RADICES(8, false, 2, 2, 4, 1, 8, 64)
MF_RADICES(16, false, 2, 4, 4, 1, 16, 64)
MF_RADICES(32, false, 2, 8, 4, 1, 8, 64)
MF_RADICES(48, false, 3, 3, 4, 4, 16, 192)
MF_RADICES(64, false, 3, 4, 4, 4, 16, 256)
MF_RADICES(80, false, 3, 5, 4, 4, 16, 320)
MF_RADICES(96, false, 3, 6, 4, 4, 16, 384)
MF_RADICES(128, false, 3, 8, 4, 4, 16, 256)
MF_RADICES(8, true, 2, 2, 4, 1, 8, 64)
MF_RADICES(16, true, 3, 2, 4, 2, 16, 128)
MF_RADICES(32, true, 3, 4, 4, 2, 8, 128)
MF_RADICES(48, true, 3, 3, 4, 4, 16, 192)
MF_RADICES(64, true, 3, 4, 4, 4, 16, 256)
MF_RADICES(80, true, 3, 5, 4, 4, 16, 320)
MF_RADICES(96, true, 3, 6, 4, 4, 16, 384)
MF_RADICES(128, true, 3, 8, 4, 4, 16, 512)
#undef MF_RADICES

template <typename R, int N>
struct ColTile {
  using Sch = ColRadices<N, sizeof(R) == 8>;
  static constexpr int RL = Sch::r[Sch::n - 1];
  static constexpr int P = Sch::p, NT = Sch::nt;
  static constexpr int NWAVES = NT / 64;
  static constexpr int STR = N + 1;
  using X = Batch<R, N, Sch, P, NT, true>;
};

// LDS shell histograms of a column workgroup: 8 copies per wave (by lane)
// where they take at most 32 KB, else 4, 2 or 1.
template <typename R, int N>
__host__ __device__ constexpr int column_hist_copies(int nb) {
  int hg = 8;
  while (hg > 1 && ColTile<R, N>::NWAVES * hg * hist_stride(nb) * 8 > 32768) hg /= 2;
  return ColTile<R, N>::NWAVES * hg;
}

// With AHEAD, rows of workgroups after the planes compute the next sweep's
// messenger normals into a.nrm, a voxel pair's quads per thread.  A plane kernel
// of few planes leaves half of the CUs idle and is bound by the vector
// instructions on the others (10.6 of 20.8 us at 80^3 FP64), of which the draws
// are the larger part and need nothing of the field.
template <typename R, int N, int XM, bool AHEAD = false>
__global__ void __launch_bounds__((ColTile<R, N>::NT))
column_kernel(SweepArgs<R> a) {
  using T = ColTile<R, N>;
  using X = typename T::X;
  constexpr int P = T::P, NT = T::NT, RL = T::RL, NSL = N / RL;
  __shared__ cx<R> field[P * T::STR];
  Exchange<cx<R>, P * T::STR, false> lds(field);
  __shared__ cx<R> tw[N];
  extern __shared__ double dyn[];   // histograms, table (2 nb R), thresholds (nb + 1)
  const int tid = threadIdx.x, nb = a.nb, hs = hist_stride(nb);
  const int iy0 = blockIdx.x * P, kz = blockIdx.y, c = blockIdx.z;
  if (AHEAD && kz > N / 2) {
    constexpr int H = N / 2, Q = N / 4;
    const int k = ((kz - H - 1) * static_cast<int>(gridDim.x) + static_cast<int>(blockIdx.x)) * NT + tid;
    if (k >= N * H * Q) return;
    const int p = k % H, q = k / H % Q, ix = k / (H * Q);
    const uint32_t wa = static_cast<uint32_t>((ix * N + 2 * p) * Q + q), sweep = a.ctr[1] + 1u;
    R ga[4], gb[4];
    {
      const Words4 w = philox4x32_10(wa, sweep, kPhaseMessenger, a.chain0 + c, a.key0, a.key1);
      box_muller(w.x0, w.x1, ga[0], ga[1]);
      box_muller(w.x2, w.x3, ga[2], ga[3]);
    }
    {
      const Words4 w = philox4x32_10(wa + Q, sweep, kPhaseMessenger, a.chain0 + c, a.key0, a.key1);
      box_muller(w.x0, w.x1, gb[0], gb[1]);
      box_muller(w.x2, w.x3, gb[2], gb[3]);
    }
    cx<R>* nrm = a.nrm + static_cast<size_t>(c) * (a.m / 2);
#pragma unroll
    for (int j4 = 0; j4 < 4; ++j4) {
      int tile = 0, e = 0;
      nrm[static_cast<uint32_t>(coef_entry<R, N>(ix, p, q + j4 * Q, tile, e))] = cx<R>{ga[j4], gb[j4]};
    }
    return;
  }
  // advance the sweep counter: no column workgroup reads slot 0
  advance_sweep(a);
  cx<R>* spec = a.spec + static_cast<size_t>(c) * a.spec_stride + static_cast<size_t>(kz) * N * N + iy0;
  load_twiddles(tw, a.tw, N, NT);
  const int copies = XM == kXDet ? 0 : column_hist_copies<R, N>(nb), hg = copies / T::NWAVES;
  R* tab = reinterpret_cast<R*>(dyn + copies * hs);
  int32_t* qthr = reinterpret_cast<int32_t*>(tab + 2 * nb);
  for (int i = tid; i < copies * hs; i += NT) dyn[i] = 0.0;
  for (int i = tid; i < 2 * nb; i += NT) tab[i] = a.table[static_cast<size_t>(c) * 2 * nb + i];
  for (int i = tid; i <= nb; i += NT) qthr[i] = i < nb ? a.qthr[i] : INT32_MAX;
  DrawCtx<R> d;
  d.qthr = qthr;
  d.tab = reinterpret_cast<const cx<R>*>(tab);
  d.hist = XM == kXDet ? dyn : dyn + ((tid / 64) * hg + (tid & (hg - 1))) * hs;
  d.hist2 = nullptr;
  d.qscale = static_cast<float>(4.0 * nb * nb / (3.0 * N * N));
  d.nb = nb;
  d.chain = a.chain0 + c;
  d.sweep = a.ctr[1];
  auto idx = [&](int col, int i) { return col * T::STR + i; };
  cx<R> v[X::REGS];
  X::template in<0, false, false>(v, tw, [&](int col, int i) { return spec[static_cast<uint32_t>(i * N + col)]; });
  X::template rest<false, false>(v, tw, lds, idx);
#pragma unroll
  for (int i = 0; i < X::slots(RL); ++i) {
    int col = 0, q = 0;
    if (!X::template at<RL>(i, col, q)) continue;
    cx<R>* x = v + i * RL;
    if constexpr (XM == kXSample) {
      draw_slot<R, N, RL, NSL, false, 1, sizeof(R) == 4>(x, q, iy0 + col, kz, a, d);
    } else {
      cx<R>* aux = a.aux == nullptr ? nullptr : a.aux + (spec - a.spec) + static_cast<size_t>(q) * N + col;
      filter_slot<R, N, RL, NSL, XM>(x, q, iy0 + col, kz, d, aux, static_cast<size_t>(NSL) * N);
    }
    dft<R, RL, true>(x);
  }
  lds.drain();   // the forward transform's reads
  X::template rest<true, true>(v, tw, lds, idx);
  X::template out<X::STAGES - 1, true>(v, [&](int col, int i, cx<R> z) { spec[static_cast<uint32_t>(i * N + col)] = z; });
  if constexpr (XM != kXDet) {
    // fixed-order sums of the copies; rest() has a barrier after the last add
    static_assert(X::STAGES > 1, "a barrier between the draws and the sums");
    const double wgt = (kz == 0 || kz == N / 2) ? 1.0 : 2.0;
    double* part = a.partials + static_cast<size_t>(c) * a.n_wg_x * nb + blockIdx.y * gridDim.x + blockIdx.x;
    for (int b = tid; b < nb; b += NT) {
      double s = 0.0;
      for (int w = 0; w < copies; ++w) s += dyn[w * hs + b];
      part[static_cast<size_t>(b) * a.n_wg_x] = wgt * s;
    }
  }
}

}  // namespace mf
