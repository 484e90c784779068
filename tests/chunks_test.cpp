// Host-only test of the chunk sizes (chunks.h): the bytes that a chunk's
// intermediates hold, the frames that overlapping chunks share, and the smaller
// chunks taken where memory is short.  Built with g++ by tests/test_chunks.py.
#include <cstdio>
#include <cstdlib>

#include "chunks.h"

static int failures = 0;
#define CHECK(c)                                                                                        \
  do {                                                                                                  \
    if (!(c)) {                                                                                         \
      std::fprintf(stderr, "%s:%d CHECK failed: %s (pix %ld w %d s %d n %d)\n", __FILE__, __LINE__, #c, pix, w, s, \
                   nwin);                                                                               \
      ++failures;                                                                                       \
    }                                                                                                   \
  } while (0)

int main() {
  const int sides[] = {64, 128, 256, 320, 384, 512, 800, 1024, 1280};
  for (int ny : sides)
    for (int nx : sides)
      for (int cplx : {4, 8})
        for (bool as : {false, true})
          for (int w : {8, 16, 32, 64, 128, 512})
            for (int s : {1, 3, w / 4, w / 2, w - 1, w, w + 5})
              for (int nwin : {1, 2, 3, 17, 100, 100000}) {
                const long pix = (long)ny * nx;
                const hvc::Chunk c = hvc::stft_chunk(pix, cplx, as, 0, w, s, nwin);
                CHECK(c.windows >= 1 && c.windows <= nwin && c.least >= 1 && c.least <= c.windows);
                const long frames = (long)(c.windows - 1) * s + w, small = (long)(c.least - 1) * s + w;
                // three complex values per pixel at most
                CHECK(c.windows == c.least || frames * pix * cplx * 3 <= 2L << 30);
                CHECK(c.least == 1 || small <= hvc::auto_frames(pix, cplx));
                // without overlap the whole windows nearest to 96 MiB (angular spectrum), or that fit it,
                // where it is 32 to 64 frames
                const long fit = (96L << 20) / (pix * cplx * 3 / 2);
                if (s >= w && fit >= 32 && fit < 64 && nwin == 100000) {
                  CHECK(c.windows == 1 || small - s < fit);
                  CHECK(as || c.windows == 1 || small <= fit);
                  if (as && w <= fit) CHECK(std::labs(fit - small) * 2 <= s || small + s > 64);
                }
                if (s >= w) CHECK(c.windows == c.least);
                // at most a sixteenth of a chunk's new frames shared, or all the memory
                const long more = frames + s;
                if (s < w && c.windows < nwin && (long)c.windows * s * 2 < 16L * (w - s))
                  CHECK(more * 2 * pix * cplx * 3 / 2 > 1L << 30 || c.windows == 1);
                // the caller's frames are obeyed
                for (int set : {1, w, 3 * w + 1}) {
                  const hvc::Chunk f = hvc::stft_chunk(pix, cplx, as, set, w, s, nwin);
                  CHECK(f.windows == f.least && (f.windows == 1 || (long)(f.windows - 1) * s + w <= set));
                }
                // host frames: the larger chunks only where the smaller share over a quarter
                const hvc::Chunk h = hvc::stft_chunk(pix, cplx, as, 0, w, s, nwin, true);
                const long shared = s < w ? w - s : 0;
                CHECK(h.windows <= nwin && h.least <= h.windows);
                CHECK(h.windows == c.windows || (h.windows == h.least && 4 * shared <= (long)h.windows * s));
                CHECK(h.windows >= c.windows || h.least == h.windows);
                // memory for chunks of `room` windows
                for (int room : {0, c.least, c.windows - 1, c.windows}) {
                  hvc::Chunk d = c;
                  int calls = 0;
                  const int r = hvc::with_room(d, -3, [&](int g) { return ++calls, g <= room ? 0 : -3; });
                  CHECK((r == 0) == (room >= c.least));
                  CHECK(d.windows == (room >= c.windows ? c.windows : c.least));
                  CHECK(calls == (room >= c.windows || c.least == c.windows ? 1 : 2));
                  hvc::Chunk e = c;  // another failure is not tried again
                  calls = 0;
                  CHECK(hvc::with_room(e, -3, [&](int) { return ++calls, -5; }) == -5 && calls == 1);
                }
              }
  if (failures) return 1;
  std::puts("all checks passed");
  return 0;
}
