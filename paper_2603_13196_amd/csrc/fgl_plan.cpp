// Launch planning: host-side shape arithmetic of the kernels in
// fgl_kernels.hip (the LDS a tile stages, the reduction groups and channel
// chunks of a launch, the workgroup ranges of a launch shared by several
// models, the gradient kernel's chunking).  No device code: the library
// compiles it with hipcc, and the sanitizer build of the host code on the
// CPU compiles the same file with g++.
#include "fgl_internal.h"

#include <algorithm>

namespace fgl {

constexpr double kThinRowsOps = 2.0e8;   // one-launch calls: a few us of the vector units
constexpr int kThinRowsMax = 2048;       // and eight rows or fewer for each CU

int cols_per_wave(Kind k) { return k == kFP64 ? 16 : (k == kThin ? 64 : 32); }

int max_lds_bytes() { return 160 * 1024; }

int lds_bytes(Kind k, const DevModel& m, const Tile& t) {
  const int d = t.fc * m.TT * 32 * 8;
  switch (k) {
    case kMixed:
      if (m.proj)
        return t.fc * (kProjDigits * m.KC * m.RT * 1024 + m.RT * 32 * 8) +
               (kTabSize + 2 * kFracSize) * 8;
      return t.fc * 4 * m.KC * m.TT * 1024 + d + (kTabSize + 2 * kFracSize) * 8;
    case kFP32:
      if (m.pplain) return t.fc * (m.NP2 * m.RT * 64 * 4 + m.RT * 32 * 8);
      return t.fc * m.NP2 * m.TT * 64 * 4 + d;
    case kThin: return 512 + t.fc * m.T * m.NT * 4 + d;
    default:
      if (m.pplain) return 512 + t.fc * (m.NQ * m.RT16 * 64 * 8 + m.RT16 * 16 * 8);
      return 512 + t.fc * m.NQ * m.TT16 * 64 * 4 + d;
  }
}

int n_chunks(const DevModel& m, const Tile& t) { return (m.F + t.fc - 1) / t.fc; }

// A round is one workgroup on every slot of the chip: the CUs times the
// workgroups that registers (four SIMDs of `occ` waves) and LDS let share a
// CU.  With uniform chunks the last round of a launch can be nearly empty
// (at N32 F301 B16384, eight-channel chunks make 9.5 rounds of 256
// workgroups).  Whole rounds of large chunks followed by half-size chunks
// cut the busiest CU's channels from ceil(rounds) * fc toward the mean
// (there from 80 to 76, against 75.25).
Chunks chunk_plan(Kind k, const DevModel& m, const Tile& t, int nb) {
  const int nc = n_chunks(m, t);
  const Chunks even{t.fc, t.fc, nc, nc};
  if (k != kMixed || nb < 1) return even;
  const int fs = std::max(t.group, t.fc / 2 / t.group * t.group);
  if (fs >= t.fc) return even;
  const int per_cu = std::max(1, std::min(4 * t.occ / t.waves,
                                          max_lds_bytes() / lds_bytes(k, m, t)));
  const long slots = (long)kCUs * per_cu;
  const long rounds = (long)nb * (m.F / t.fc) / slots;
  if (rounds == 0) return even;
  const int nbig = (int)(rounds * slots / nb);
  const int nsmall = (m.F - nbig * t.fc + fs - 1) / fs;
  auto up = [&](long wg) { return (wg + slots - 1) / slots; };
  const long now = up((long)nb * nc) * t.fc;
  const long split = up((long)nb * nbig) * t.fc + up((long)nb * nsmall) * fs;
  // only where it cuts the busiest CU's share by 2% or more; and the block
  // map needs at least one small chunk per XCD
  if (nbig < 1 || 50 * (now - split) < now || (long)nb * nsmall < 8) return even;
  return Chunks{t.fc, fs, nbig, nbig + nsmall};
}

int n_groups(const DevModel& m, const Tile& t) {
  return (m.F + t.group - 1) / t.group;
}

size_t thin_rows_lds(const DevModel& m, int rows) {
  const size_t groups = (m.F + 3) / 4;
  return ((size_t)rows * (m.P + m.NT * (m.NA > 0 ? 2 : 1) + groups + 16) + 64) * 8 + rows * 4;
}

// Times (us) of a call from device memory by the slots its regions take: a turn of
// the one-launch kernel without its bins and with each step of thin_rows_bins, and
// the three launches without their bins and with each.
struct ThinCost {
  double turn, step, launches, bin;
};
static ThinCost thin_cost(int NT) {
  switch (NT) {
    case 4: return {1.25, 2.6, 10.3, 0.114};
    case 8: return {1.9, 1.3, 10.3, 0.30};
    case 12: return {2.3, 1.0, 10.5, 0.39};
    case 16: return {2.9, 1.2, 12.2, 0.55};
    case 24: return {4.1, 1.55, 13.3, 0.85};
    default: return {5.7, 1.9, 13.2, 0.70};
  }
}

// A small batch of a thin model is bound by its three launches, about 12 us and
// the latency of the four channels that a thread takes in turn.  One kernel can do
// the whole of it in about 5 us and that latency for each turn its 256 / rows
// threads per row need to cover the channel groups; it reads K per lane from the
// caches instead of staging it for 256 rows, so large batches stay with the staged
// kernel.  A channel's latency goes as c = 12 NT + T (NT + 30), about 3.5 ns a unit
// and four channels a turn: (turns - 1) c <= 450 is the widest range.  Whole calls,
// three launches and one (us):
//   N4 F151 T1 B1000 14.9, 7.8; B2000 15.4, 10.7     N32 F301 T1 B1000 20.0, 18.2
//   N24 F200 T6 B300 21.0, 12.8     N16 F151 T20 B900 26.1, 18.5
// From host memory the three launches come with two copies, 15-20 us more, and one
// launch is 1.1 to 1.6 times as fast over all of that range.  From device memory it
// has to be faster by ThinCost, fitted to timed calls on a grid of shapes (standard
// deviations of 0.4 to 1.0 us for one launch and 0.2 to 1.6 for three).  Of 3236
// calls of random shapes that it takes, 24 are slower by more than 2 %, 10 % at worst.
//   left out: N3 F395 T2 B1292 15.3, 18.9     N2 F200 T45 B200 17.1, 22.1
//   N4 F301 T9 B200 12.8, 15.9     N30 F301 T1 B1 15.2, 17.9
// A channel of more than c = 1650 (many bins), or 1000 with eight rows, is slower
// from the caches even in one turn, and past eight rows for each of the 256 CUs the staged kernel's rows
// fill the chip too.
//   past the line: N10 F301 T1 B3000 18.5, 19.5     N16 F151 T20 B1500 26.0, 32.5
//   N4 F301 T8 B3000 17.0, 23.4     N8 F301 T40 B500 26.1, 33.5
//   N4 F151 T64 B300 19.4, 25.4     N4 F151 T1 B6000 15.0, 19.0; B16384 23.6, 27.7
//   N4 F120 T30 B2000 15.4, 16.0    N16 F120 T10 B2000 19.6, 12.7 (c 652, taken)
//   N10 F151 T1 B6000 18.6, 18.4    N4 F100 T1 B6000 15.4, 14.2 (left out for one line)
//
// A tile that the caller chose has to run: such calls stay with the three launches.
int thin_rows_of(Kind k, const DevModel& m, const Tile& t, int B, bool host) {
  if (k != kThin || t.group != 4 || t.chosen) return 0;
  if ((double)B * m.F * (m.NT * m.T + 12 * m.NT + 2 * m.T) > kThinRowsOps) return 0;
  if (B > kThinRowsMax) return 0;
  const int rows = B <= 1024 ? 4 : 8;
  const int64_t turns = ((m.F + 3) / 4 * rows + 255) / 256;
  const int64_t c = 12 * m.NT + m.T * (m.NT + 30);
  if ((turns - 1) * c > 450 || c > (rows == 4 ? 1650 : 1000)) return 0;
  if (!host) {
    const ThinCost w = thin_cost(m.NT);
    const double bins = (m.T + thin_rows_bins(m.NT) - 1) / thin_rows_bins(m.NT);
    const double ops = (double)B * m.F * (m.NT * m.T + 12 * m.NT + 2 * m.T);
    const double one = 3.9 + turns * (w.turn + w.step * bins);
    const double three = std::max(12.4, w.launches + w.bin * m.T + 3e-5 * m.F * std::min(B, 200) +
                                            2.8e-8 * ops);
    if (one > three) return 0;
  }
  return thin_rows_lds(m, rows) > 48 * 1024 ? 0 : rows;
}

int thin_rows_of(Kind k, const DevModel& m, const Tile& t, int B, bool host, const double* theta,
                 const double* out) {
  // results over the rows they come from: every row is read before any is written
  // only by the three launches
  const char *t0 = reinterpret_cast<const char*>(theta), *o0 = reinterpret_cast<const char*>(out);
  if (o0 < t0 + (size_t)B * m.P * 8 && t0 < o0 + (size_t)B * 8) return 0;
  return thin_rows_of(k, m, t, B, host);
}

uint64_t variant_of(Kind k, const DevModel& m, const Tile& t) {
  if (m.NA != 0) return 0;
  if (k == kMixed) {
    if (t.waves != 8 || m.KC > 2 || (t.occ == 3 && !(m.proj && m.KC == 1))) return 0;
    return 1ull | (uint64_t)m.KC << 8 | (uint64_t)m.proj << 12 | (uint64_t)t.occ << 16;
  }
  if (k == kThin) return 2ull | (uint64_t)m.NT << 8 | (uint64_t)t.waves << 16;
  return 0;
}

void plan_groups(Kind k, const Tile& tile, GroupDesc* h, int n, int grid[3], int* lds) {
  const int cols = cols_per_wave(k) * tile.waves;
  int main = 0, prep = 0, fin = 0, l = 0;
  for (int j = 0; j < n; ++j) {
    GroupDesc& g = h[j];
    const Tile tj{tile.waves, g.fc, g.G, tile.occ};
    g.nb = g.w.Bpad / cols;
    g.nc = n_chunks(g.m, tj);
    main = (main + 7) & ~7;
    g.start[0] = main;
    main += g.nb * g.nc;
    g.start[1] = prep;
    prep += (g.w.Bpad + kPrepRows - 1) / kPrepRows;
    g.start[2] = fin;
    fin += (g.w.B * 16 + 255) / 256;
    l = std::max(l, lds_bytes(k, g.m, tj));
  }
  grid[0] = main;
  grid[1] = prep;
  grid[2] = fin;
  *lds = l;
}

// 4-wave workgroups (64 rows); chunks of kGradChunk channels, fixed per
// model so that a row's sums do not depend on the batch it came in; as many
// channels staged at once as fit in 40 KB (at least one; measured faster than
// 24 KB or 64 KB at the headline shape, for the workgroups it lets share a CU).
constexpr int kGradChunk = 16;

GradShape grad_shape(const DevModel& m, int Bpad) {
  GradShape g;
  g.nb = Bpad / 64;
  const int per_ch = m.proj ? m.NQ * grad_kstride(m.RT16) * 8 + m.RT16 * 16 * 8
                           : m.NQ * grad_kstride(m.TT16) * 4 + m.TT * 32 * 8;
  g.per = std::min(m.F, kGradChunk);
  g.chunks = (m.F + g.per - 1) / g.per;
  // stages of <= 40 KB with the power table (four workgroups per CU)
  g.fs = std::max(1, std::min(g.per, (40 * 1024 - 512) / per_ch));
  g.lds = 512 + g.fs * per_ch;
  return g;
}

}  // namespace fgl
