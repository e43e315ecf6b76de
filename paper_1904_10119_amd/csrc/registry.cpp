// Registry of the compiled pass kernels.
#include <algorithm>
#include <unordered_map>

#include "../../include/dft3d.h"
#include "internal.h"

namespace dft3d {

void register_kernels_small(std::vector<KernelInfo>& v);
void register_kernels_mid(std::vector<KernelInfo>& v);
void register_kernels_1k(std::vector<KernelInfo>& v);
void register_kernels_big(std::vector<KernelInfo>& v);
void register_kernels_mfma_a(std::vector<KernelInfo>& v);
void register_kernels_mfma_b(std::vector<KernelInfo>& v);
void register_kernels_mfma_c(std::vector<KernelInfo>& v);
void register_kernels_mfma_d(std::vector<KernelInfo>& v);
void register_kernels_mfma_e(std::vector<KernelInfo>& v);
void register_kernels_mfma_f(std::vector<KernelInfo>& v);
void register_kernels_mfma_g(std::vector<KernelInfo>& v);
void register_kernels_mfma_h(std::vector<KernelInfo>& v);
void register_kernels_mfma_i(std::vector<KernelInfo>& v);
void register_kernels_plane(std::vector<KernelInfo>& v);
void register_kernels_fused(std::vector<KernelInfo>& v);
void register_kernels_bluestein(std::vector<KernelInfo>& v);
void register_kernels_mixed(std::vector<KernelInfo>& v);
void register_kernels_mixed_fixed(std::vector<KernelInfo>& v);
void register_kernels_rader(std::vector<KernelInfo>& v);
void register_kernels_rader_fixed(std::vector<KernelInfo>& v);
void register_kernels_halves(std::vector<KernelInfo>& v);
void register_kernels_bluestein_two_step_a(std::vector<KernelInfo>& v);
void register_kernels_bluestein_two_step_b(std::vector<KernelInfo>& v);
void register_kernels_bluestein_two_step_c(std::vector<KernelInfo>& v);
void register_kernels_bluestein_two_step_d(std::vector<KernelInfo>& v);
void register_kernels_bluestein_two_step_e(std::vector<KernelInfo>& v);
void register_kernels_rader_two_step(std::vector<KernelInfo>& v);
void register_kernels_two_step_power(std::vector<KernelInfo>& v);
void register_kernels_two_step_a(std::vector<KernelInfo>& v);
void register_kernels_two_step_b(std::vector<KernelInfo>& v);
void register_kernels_two_step_c(std::vector<KernelInfo>& v);
void register_kernels_two_step_d(std::vector<KernelInfo>& v);
void register_kernels_two_step_e(std::vector<KernelInfo>& v);
void register_kernels_two_step_f(std::vector<KernelInfo>& v);
void register_kernels_two_step_g(std::vector<KernelInfo>& v);
void register_kernels_two_step_h(std::vector<KernelInfo>& v);
void register_kernels_two_step_i(std::vector<KernelInfo>& v);
void register_kernels_two_step_j(std::vector<KernelInfo>& v);

const std::vector<KernelInfo>& kernel_registry() {
  static const std::vector<KernelInfo> table = [] {
    std::vector<KernelInfo> v;
    register_kernels_small(v);
    register_kernels_mid(v);
    register_kernels_1k(v);
    register_kernels_big(v);
    register_kernels_mfma_a(v);
    register_kernels_mfma_b(v);
    register_kernels_mfma_c(v);
    register_kernels_mfma_d(v);
    register_kernels_mfma_e(v);
    register_kernels_mfma_f(v);
    register_kernels_mfma_g(v);
    register_kernels_mfma_h(v);
    register_kernels_mfma_i(v);
    register_kernels_plane(v);
    register_kernels_fused(v);
    register_kernels_bluestein(v);
    register_kernels_mixed(v);
    register_kernels_mixed_fixed(v);
    register_kernels_rader(v);
    register_kernels_rader_fixed(v);
    register_kernels_halves(v);
    register_kernels_bluestein_two_step_a(v);
    register_kernels_bluestein_two_step_b(v);
    register_kernels_bluestein_two_step_c(v);
    register_kernels_bluestein_two_step_d(v);
    register_kernels_bluestein_two_step_e(v);
    register_kernels_rader_two_step(v);
    register_kernels_two_step_power(v);
    register_kernels_two_step_a(v);
    register_kernels_two_step_b(v);
    register_kernels_two_step_c(v);
    register_kernels_two_step_d(v);
    register_kernels_two_step_e(v);
    register_kernels_two_step_f(v);
    register_kernels_two_step_g(v);
    register_kernels_two_step_h(v);
    register_kernels_two_step_i(v);
    register_kernels_two_step_j(v);
    return v;
  }();
  return table;
}

namespace {

// The registry by what lookups ask for, every list in registry order.  A plan
// makes some ten lookups; over the whole registry (2400 kernels, most of them
// compiled for one length each) they took 11 to 27 us of a plan's building.
struct KernelIndex {
  std::unordered_map<int64_t, KernelList> of, compiled_for;
  KernelList many;
  KernelIndex() {
    for (const KernelInfo& k : kernel_registry()) {
      (k.fixed_n ? compiled_for[k.fixed_n] : of[k.n]).push_back(&k);
      if (!k.fixed_n && (k.mixed || k.rader || (k.bluestein && k.two_step))) many.push_back(&k);
    }
  }
};

const KernelIndex& kernel_index() {
  static const KernelIndex index;
  return index;
}

const KernelList& list_at(const std::unordered_map<int64_t, KernelList>& m, int64_t n) {
  static const KernelList none;
  const auto it = m.find(n);
  return it == m.end() ? none : it->second;
}

}  // namespace

const KernelList& kernels_of(int64_t n) { return list_at(kernel_index().of, n); }
const KernelList& kernels_compiled_for(int64_t n) {
  return list_at(kernel_index().compiled_for, n);
}
const KernelList& kernels_for_many() { return kernel_index().many; }

const KernelInfo* find_kernel(int n, int tile, int lmode, int smode, int post_twiddle,
                              int persistent, int nontemporal) {
  for (const KernelInfo* k : kernels_of(n))
    if (k->n == n && k->tile == tile && k->lmode == lmode && k->smode == smode &&
        k->post_twiddle == post_twiddle && k->persistent == persistent &&
        k->nontemporal == nontemporal && k->precision == 0 && k->plane_rows == 0 &&
        k->fused_axes == 0 && k->bluestein == 0 && k->mixed == 0 && k->rader == 0 &&
        k->halves == 0 && k->two_step == 0 && k->move_only == 0)
      return k;
  return nullptr;
}

// Measured on MI355X, one-tile pass kernel / two-step kernel per launch, in
// us: length 16 (16 x 32 x 512) 4.2 / 3.3, 32 (32^3) 4.4 / 3.0, 64 (64^3) 4.4
// / 3.7, 128 (128^3) 9.7 / 8.5, 256 (256^3 rows, columns) 56.9, 44.8 / 54.7,
// 44.0, 512 (512^3) 1252 / 1216 (whole transform), 1024 (64 x 1024 x 1024)
// 251 / 246; 1024^3 is level, 10.50 / 10.40 ms timed in turn (whole transform).
// Tiles of 16 pencils, with these exceptions:
//  - 64 at 2^22 points 32 pencils (level with the pass kernel: 64 x 1024 x 64
//    rows 12.0 / 12.0), above them the pass kernel in 64 pencils (1201 x 1201 x
//    64 rotated 279 against 302 us, in layout 249 / 261, 1024 x 1024 x 64 rows 184
//    / 193, 2048 x 1024 x 64 409 / 427; 64 x 512 x 512 is the best case for two
//    steps, 43.0 / 41.9);
//  - 128 from 2^23 points up the 32-pencil pass kernel (64 x 1024 x 128 rows
//    29.3 against 33.0, 256 x 256 x 128 30.0 / 32.9; 512 x 512 x 128 rows
//    95.8 against 101 us with two steps in 32 pencils, 104 in 16);
//  - 256 above 2^25 points 32 pencils (1024 x 512 x 256 437 / 412; below, 16
//    are faster: 128 x 1024 x 256 rows 97.6 against 103.7);
//  - 16, 32 and 64 along strided axes from 2^21 points up the pass kernel,
//    whose 256, 128 or 64 pencils are long row segments (16 x 512 x 512 depth
//    11.8 against 12.7, 32 x 256 x 512 10.9 against 13.0);
//  - 64 from 2^20 points and 256 from 2^24, where rotated rows do not start on
//    lines, the pass kernel's 64 and 32 pencils (251 x 64 x 251 11.7 against 12.7,
//    255 x 256 x 511 109 / 124; below 127 x 64 x 129 8.1 / 7.1, 127 x 256 x 129
//    13.1 / 13.3; 128 and 512 are level or ahead in two steps);
//  - 512 from 2^23 points up along strided axes whose points lie less than 2 KB
//    or 128 KB and more apart, and from 2^23 to 2^24 in the rotation, the pass
//    kernel (512 x 64 x 256 depth 25.0 against 27.0, 512 x 512 x 64 columns 45.3
//    / 48.7, 512 x 256 x 64 rotated 24.9 / 27.3; columns between, rows and the
//    rotation from 2^24 points up are level or 1 to 3 % faster in two steps:
//    whole slabs 16 x 512 x 1024 79.9 / 78.5, 8 x 512 x 2048 84.1 / 82.9, 64 x
//    512 x 256 74.8 / 74.1);
//  - 16 and 32 from 2^25 points up the pass kernel in every order: the cycled
//    pencil passes of such arrays read pencils a plane apart and write row
//    segments of a tile's pencils (16 x 1024 x 2048 102 against 127, 32 x 1024
//    x 1024 111 / 140; half the points 42 against 48 the other way round);
//  - from 256 up, where tiles of 16 are at most 512 (two a CU), 8 pencils
//    (16 x 256 x 256 8.3 / 7.2, 16 x 64 x 1024 12.2 / 9.1, 16 x 512 x 512 rows
//    15.3 / 14.2; tiles of 4 gain no more, and at 1024 tiles 16 are faster:
//    32 x 512 x 512 rows 32.4 against 34.7).
const KernelInfo* find_two_step_power_kernel(int n, int64_t pencils, int lmode, int smode,
                                             int64_t oks) {
  const int64_t points = pencils * n;
  if (rows_off_lines(pencils, lmode, smode, oks) &&
      ((n == 64 && points >= (int64_t(1) << 20)) || (n == 256 && points >= (int64_t(1) << 24))))
    return nullptr;
  int tile = 16;
  if (n == 64 && points > (int64_t(1) << 22)) return nullptr;
  if (n == 64 && points >= (int64_t(1) << 22)) tile = 32;
  if (n == 128 && points >= (int64_t(1) << 23)) return nullptr;
  if (n == 256 && points > (int64_t(1) << 25)) tile = 32;
  if (n == 512 && smode == MODE_COL && points >= (int64_t(1) << 23) &&
      (lmode == MODE_COL ? oks < 256 || oks >= (1 << 14) : points < (int64_t(1) << 24)))
    return nullptr;
  if (n <= 32 && points >= (int64_t(1) << 25)) return nullptr;
  if (n <= 64 && lmode == MODE_COL && points >= (int64_t(1) << 21)) return nullptr;
  if (n >= 256 && pencils <= 16 * 512) tile = 8;
  for (const KernelInfo* k : kernels_of(n))
    if (k->two_step && !k->mixed && !k->bluestein && !k->rader && !k->move_only && k->n == n &&
        k->tile == tile && k->lmode == lmode && k->smode == smode)
      return k;
  return nullptr;
}

const KernelInfo* find_halves_kernel(int n, int lmode, int smode, int persistent,
                                     int nontemporal, int move_only) {
  for (const KernelInfo* k : kernels_of(n))
    if (k->halves && k->n == n && k->lmode == lmode && k->smode == smode &&
        k->persistent == persistent && k->nontemporal == nontemporal &&
        k->move_only == move_only)
      return k;
  return nullptr;
}

const KernelInfo* find_move_only_kernel(const KernelInfo* k, int mode) {
  if (!k || k->precision || k->plane_rows || k->fused_axes || k->bluestein || k->mixed ||
      k->rader || k->move_only)
    return nullptr;
  if (k->halves && mode == 1)
    return find_halves_kernel(k->n, k->lmode, k->smode, k->persistent, k->nontemporal, 1);
  for (const KernelInfo* c : kernels_of(k->n)) {
    if (c->move_only != mode || c->halves || (mode == 1 && c->two_step != k->two_step)) continue;
    if (mode == 2 && c->n == k->n) return c;
    if (mode == 1 && c->n == k->n && c->tile == k->tile && c->lmode == k->lmode &&
        c->smode == k->smode && c->post_twiddle == k->post_twiddle &&
        c->persistent == k->persistent && c->nontemporal == k->nontemporal &&
        c->r0 == k->r0 && c->r1 == k->r1 && c->r2 == k->r2)
      return c;
  }
  return nullptr;
}

bool mixed_kernel_runs(int variant, int nmax, uint64_t code) {
  for (uint64_t c = code; c; c >>= 8) {
    const int r = (int)(c & 255);
    if (r == 11 || r == 13) {
      if (variant < 2) return false;
    } else if (r == 10 || r == 16) {  // composites: variant 1 up to 2048 only
      if (variant != 1 || nmax > 2048) return false;
    } else if (r != 2 && r != 3 && r != 4 && r != 5 && r != 7 && r != 8) {
      return false;
    }
  }
  return true;
}

const KernelInfo* find_mixed_kernel(int64_t n, uint64_t code, int tile, int lmode, int smode) {
  const int variant = mixed_variant(code);
  const KernelInfo* best = nullptr;
  if (tile <= 0)  // a kernel compiled for this length, code and modes, if any
    for (const KernelInfo* k : kernels_compiled_for(n))
      if (k->mixed && !k->two_step && k->fixed_n == n && k->fixed_code == code &&
          k->lmode == lmode && k->smode == smode)
        return k;
  for (const KernelInfo* k : kernels_for_many())
    if (k->mixed == variant && !k->two_step && k->fixed_n == 0 && k->n > n && k->lmode == lmode &&
        k->smode == smode && mixed_kernel_runs(k->mixed, k->n, code)) {
      if (tile > 0 && k->tile == tile) return k;  // the asked-for tile, if any
      if (!best || k->n < best->n) best = k;      // else the first, smallest
    }
  return best;
}

const KernelInfo* find_two_step_kernel(int64_t n, int64_t pencils, int lmode, int smode,
                                       int64_t oks) {
  if (!two_step_split(n)) return nullptr;
  int tile = two_step_tile(n);
  const bool misaligned = rows_off_lines(pencils, lmode, smode, oks);
  if (const int wide = two_step_wide_tile(n, pencils))
    tile = wide;
  else if (misaligned && two_step_misaligned_tile(n, pencils))
    tile = two_step_misaligned_tile(n, pencils);
  else if (tile == 16 && pencils <= 16 * (int64_t)(misaligned ? two_step_idle_tiles_off_lines(n)
                                                             : two_step_idle_tiles(n)))
    tile = 8;
  for (const KernelInfo* k : kernels_compiled_for(n))
    if (k->two_step && k->mixed && k->fixed_n == n && k->tile == tile && k->lmode == lmode &&
        k->smode == smode)
      return k;
  return nullptr;
}

uint64_t mixed_radix_code(int64_t n) {
  if (n < 2) return 0;
  const int64_t n0 = n;
  int count[14] = {0};
  for (int f : {2, 3, 5, 7, 11, 13})
    while (n % f == 0) {
      n /= f;
      ++count[f];
    }
  if (n != 1) return 0;
  // Composite radices (10 = 5 * 2, 16) only where the kernel without the
  // 11 and 13 stages runs them (lengths below 2048): fewer stages, each an
  // LDS round trip.
  const bool comp = count[11] == 0 && count[13] == 0 && n0 < 2048;
  // Odd radices first, then 10s, then powers of two: the first stage writes
  // its outputs at stride R in LDS, which an odd R spreads over every bank
  // (measured with SQ_LDS_BANK_CONFLICT at 1000^3); later stages write runs
  // of ns consecutive points.
  std::vector<int> radices;
  const int tens = comp ? std::min(count[5], count[2]) : 0;
  for (int f : {13, 11, 7, 5, 3})
    for (int i = 0; i < count[f] - (f == 5 ? tens : 0); ++i) radices.push_back(f);
  for (int i = 0; i < tens; ++i) radices.push_back(10);
  // the remaining power of two in as few stages as allowed (radix <= 16
  // with composites, else <= 8), the exponents spread evenly
  const int e = count[2] - tens, emax = comp ? 4 : 3;
  if (e > 0) {
    const int stages = (e + emax - 1) / emax;
    std::vector<int> ex(stages, e / stages);
    for (int i = 0; i < e % stages; ++i) ++ex[i];
    std::sort(ex.begin(), ex.end());
    for (int x : ex) radices.push_back(1 << x);
  }
  if (radices.size() > 8) return 0;
  uint64_t code = 0;
  for (size_t i = 0; i < radices.size(); ++i) code |= (uint64_t)radices[i] << (8 * i);
  return code;
}

int mixed_variant(uint64_t code) {
  for (uint64_t c = code; c; c >>= 8)
    if ((c & 255) == 11 || (c & 255) == 13) return 2;
  return 1;
}

int64_t radix_code_length(uint64_t code) {
  int64_t n = 1;
  for (uint64_t c = code; c; c >>= 8) n *= (int64_t)(c & 255);
  return n;
}

bool radix_code_valid(uint64_t code) {
  if (code == 0) return true;
  int stages = 0;
  int64_t n = 1;
  for (uint64_t c = code; c; c >>= 8) {
    const int r = (int)(c & 255);
    if (r != 2 && r != 3 && r != 4 && r != 5 && r != 7 && r != 8 && r != 10 && r != 11 &&
        r != 13 && r != 16)
      return false;  // a zero byte inside the code ends it early: rejected here too
    n *= r;
    if (++stages > 8 || n > 2048) return false;
  }
  // and a mixed-radix kernel runs the stages at that length
  return find_mixed_kernel(n, code, 0) != nullptr;
}

bool length_supported(int64_t n) { return n >= 1 && n <= 4096; }

namespace {
bool is_prime(int64_t n) {
  if (n < 2) return false;
  for (int64_t f = 2; f * f <= n; ++f)
    if (n % f == 0) return false;
  return true;
}
}  // namespace

const KernelInfo* find_rader_kernel(int64_t n, int tile) {
  const uint64_t code = mixed_radix_code(n - 1);
  if (!code) return nullptr;
  if (tile <= 0)  // a kernel compiled for this prime and code, if any
    for (const KernelInfo* k : kernels_compiled_for(n))
      if (k->rader && k->fixed_n == n && k->fixed_code == code) return k;
  const int variant = mixed_variant(code);
  const KernelInfo* best = nullptr;
  for (const KernelInfo* k : kernels_for_many())
    if (k->rader == variant && !k->two_step && k->fixed_n == 0 && k->n >= n + 1 &&
        mixed_kernel_runs(variant, k->n, code)) {
      if (tile > 0 && k->tile == tile) return k;
      if (!best || k->n < best->n) best = k;
    }
  return best;
}

bool rader_length(int64_t n, bool any_kernel) {
  if (n < 3 || !is_prime(n) || mixed_radix_code(n - 1) == 0) return false;
  const KernelInfo* k = find_rader_kernel(n, 0);
  return k && (any_kernel || k->fixed_n == n);
}

const KernelInfo* find_bluestein_kernel(int m, int tile) {
  const KernelInfo* first = nullptr;
  for (const KernelInfo* k : kernels_of(m))
    if (k->bluestein && !k->two_step && k->n == m) {
      if (k->tile == tile) return k;
      if (!first) first = k;
    }
  return first;
}

const KernelInfo* find_bluestein_two_step_kernel(int64_t n, int lmode, int smode) {
  const KernelInfo* best = nullptr;
  for (const KernelInfo* k : kernels_for_many())
    if (k->bluestein && k->two_step && k->n >= 2 * n && k->lmode == lmode && k->smode == smode &&
        (!best || k->n < best->n))
      best = k;
  return best;
}

const KernelInfo* find_fused_axes_kernel(int a, int contig, int persistent, int kind) {
  const int mode = contig ? MODE_ROW : MODE_COL;
  const KernelInfo* other = nullptr;
  for (const KernelInfo* k : kernels_of(a))
    if (k->fused_axes == kind && k->n == a && k->lmode == mode) {
      if (k->persistent == persistent) return k;
      other = k;
    }
  return other;
}

const KernelInfo* find_plane_kernel(int n1, int n2) {
  for (const KernelInfo* k : kernels_of(n2))
    if (k->plane_rows == n1 && k->n == n2) return k;
  return nullptr;
}

// Measured on MI355X (pencil plans, same box): leaf 32 / leaf 16 time at
// 128^3, 256^3 and 4096 x 256 x 256 0.87 .. 0.97 in every split form, 64^3
// 1.10 .. 1.13 (64 = 32 * 2 against 16 * 4).  At lengths 1024 and 2048,
// with the cycled intermediate orders that split-precision pencil plans
// run, leaves of 16 are faster in every split form: 1024^3 bf16x6 10.57 ms
// (16) against 11.76 (32), bf16x9 11.43 / 12.83, fp16x3 12.19 / 12.46;
// 2048 x 1024 x 512 bf16x6 12.50 / 13.06, bf16x9 13.32 / 13.86, fp16x3
// 12.15 / 12.31.
int default_mfma_leaf(int n, int precision) {
  (void)precision;
  if (n == 128 || n == 256 || n == 4096) return 32;
  return 16;
}

// The persistent MFMA form (one workgroup per CU, next tile prefetched)
// against the one-tile form (two workgroups per CU, four waves per SIMD),
// cycled pencil orders: slower in every form measured (1024^3 fp16x3
// 14.46 against 12.19 ms, bf16x6 equal within 0.5 %; 2048 x 1024 x 512
// fp16x3 12.89 against 12.15), so the one-tile form is the default
// wherever both exist; the persistent form stays an option (nontemporal = 1
// with persistent on).
bool default_mfma_persistent(int n, int precision) {
  (void)n;
  (void)precision;
  return false;
}

// Tile elements of the one-tile MFMA form: 8192 (4096 at length 4096) fill
// the chip only from about 2^22 points on, two workgroups a CU.  Smaller grids
// take less.  Measured on MI355X, bf16x6, us a pass at 2^17, 2^19, 2^20, 2^21 and
// 2^22 points:
//   length 64:   8192 5.9 6.9 9.3 10.1 14.4   1024 4.3 5.6 8.5 9.8 14.9   4096 4.7 5.9 8.4 9.5 14.2
//   length 256:  8192 6.2 7.8 10.0 11.2 15.4  2048 4.4 6.5 9.6 11.3 15.0  4096 5.0 6.8 8.7 11.2 13.9
//   length 512:  8192 8.4 9.0 10.8 15.7 19.1  2048 6.1 6.7 10.5 14.3 22.1  4096 6.2 6.7 8.2 14.0 19.3
//   length 1024: 8192 8.9 9.4 10.2 13.1 20.6  2048 6.9 7.9 11.4 16.2 26.9  4096 6.9 7.5 9.4 14.0 21.4
// and at 2^24 8192 is ahead at every length (256^3 55.2 against 59.3 in 4096).
// Passes that keep the layout stop at 2^20 (slab, whole transforms, 8192 / 4096:
// 256 x 128 x 64 34.2 / 35.3, 16 x 512 x 256 33.2 / 34.9, 32 x 256 x 256 30.9 / 31.5;
// at 2^20 16 x 256 x 256 is 10 % faster in 4096).  The other split precisions
// take the same rule: over 26 grids of 2^12 to 2^22 points, lengths 16 to 1024
// and both orders, bf16x9, fp16x3, bf16x1 and fp16x1 take 0.71 to 1.00 of the time in 8192.
static int mfma_tile_points(int n, int64_t points, bool keeps) {
  const int most = n == 1024 || keeps ? 20 : n == 512 ? 21 : 22;
  if (n > 1024 || points > (int64_t(1) << most)) return 0;
  if (n > 256 || points > (int64_t(1) << 19)) return 4096;
  return n == 256 ? 2048 : 1024;
}

const KernelInfo* find_mfma_kernel(int n, int64_t pencils, int lmode, int smode, int precision,
                                   int persistent, int leaf, int tile) {
  // small grids: the narrow one-tile form of the default leaves, unless the
  // persistent form, a tile or a leaf is asked for
  if (tile <= 0 && !persistent && leaf == 0)
    if (const int te = mfma_tile_points(n, pencils * n, lmode == smode))
      for (const KernelInfo* k : kernels_of(n))
        if (k->mfma_wide < 0 && k->n == n && k->tile == te / n && k->lmode == lmode &&
            k->smode == smode && k->precision == precision)
          return k;
  if (leaf == 0) leaf = default_mfma_leaf(n, precision);
  // the wide one-tile form where compiled (length 2048 rotated on write),
  // unless the persistent form or another tile is asked for
  if (tile > 0 || !persistent)
    for (const KernelInfo* k : kernels_of(n))
      if (k->mfma_wide > 0 && k->n == n && k->lmode == lmode && k->smode == smode &&
          k->precision == precision && k->mfma_leaf == leaf && (tile <= 0 || k->tile == tile))
        return k;
  const KernelInfo* other = nullptr;
  for (const KernelInfo* k : kernels_of(n))
    if (!k->mfma_wide && k->n == n && k->lmode == lmode && k->smode == smode &&
        k->precision == precision && k->mfma_leaf == leaf) {
      if (k->persistent == persistent) return k;
      other = k;
    }
  return other;
}

int device_cu_count() {
  // One entry per device; CU counts do not change while the process runs.
  static int counts[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (counts[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        n <= 0)
      n = 256;
    counts[dev] = n;
  }
  return counts[dev];
}

}  // namespace dft3d
