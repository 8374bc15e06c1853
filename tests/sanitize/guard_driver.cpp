// Host bounds of the per-wavefront kernels' register stage: a tile whose input a thread
// cannot hold must not be set.  Includes the planner itself for its internal functions.
#include "../../paper_2211_07777_amd/csrc/fm_plan.cpp"

static int set(int M, bool half, int in_n, int E, size_t elem) {
  fm::PassDesc d{};
  d.M = M;
  d.gather = fm::G_R2R;
  d.scatter = fm::S_R2R;
  d.r2r.half = half ? fm::R2R_II : fm::R2R_EXTEND;
  d.form_mode = half ? 7 : 0;
  d.in_n = d.out_n = in_n;
  d.nb = 64;
  d.nc = d.ncomp = 1;
  return set_wave(&d, elem, 4, 1, E);
}

int main() {
  int bad = 0;
  for (const size_t elem : {4, 8})
    for (const int E : {4, 8, 16})
      for (const int M : {32, 64, 128, 256, 512, 1024}) {
        if (!fm::wave_length(M, E)) continue;
        // the kernel stages U = E + 1 values (extension) or 2 E + 1 (half form) of each of the
        // 256 threads; a tile has 8 lines per FFT line of a wavefront
        const int B = 8 * fm::wave_lines(M, E);
        for (const bool half : {false, true}) {
          const int fits = 256 * (half ? 2 * E + 1 : E + 1) / B;
          for (int n = 1; n <= 2 * M; ++n)
            if (set(M, half, n, E, elem) && n > fits) {
              std::fprintf(stderr, "M %d E %d half %d: %d inputs a line accepted, %d fit\n", M, E, half, n, fits);
              ++bad;
              break;
            }
          // what real-to-real lines need is accepted
          const int need = half ? M : M / 2 + 1;
          if (M <= 512 && E != 16 && !set(M, half, need, E, elem)) {
            std::fprintf(stderr, "M %d E %d half %d: %d inputs refused\n", M, E, half, need);
            ++bad;
          }
        }
      }
  std::printf("%d wrong\n", bad);
  return bad != 0;
}
