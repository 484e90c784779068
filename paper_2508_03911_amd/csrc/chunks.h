// Sizes of the chunks in which a call's frames are processed (host arithmetic,
// no HIP).
#pragma once
#include <algorithm>

namespace hvc {

// Frames of a chunk, automatic: about 96 MiB of intermediate spectra (half
// spectrum + full spectrum = 1.5 complex values per pixel), at least 64 frames:
// 128 frames (FP32) and 256 (fp16) at 256 x 256, the fastest measured with two
// streams in flight.  cplx: bytes of a complex value (8 or 4).
inline int auto_frames(long pix, int cplx) {
  const long f = (96L << 20) / (pix * cplx * 3 / 2);
  return (int)std::max(64L, std::min(2048L, f));
}

// Windows of a chunk of the STFT paths.
struct Chunk {
  int windows;  // taken
  int least;    // taken where the device has not the room for that many
};

// The W - stride frames that a chunk shares with the next are propagated in both,
// so where windows overlap a chunk holds at least 16 times as many new frames, as
// far as 1 GiB of 1.5 complex values per pixel goes.  The passes of the angular
// spectrum hold 1.5 to 3 values per pixel (a half or a whole spectrum, the columns, the
// field), those of Fresnel 2, so that is 1 to 2 GiB per stream (times of the moments
// call, us, with chunks of the size below and with these: 1024x512 W 32 stride 16
// 1097 -> 884, 384^2 W 64 stride 16 6266 -> 2213, 256^2 W 32 stride 8 1039 -> 962;
// fp16 916 -> 743, 2505 -> 1768, 839 -> 787).  Without overlap the size of
// auto_frames, but no more than its 96 MiB where that is 32 frames or more (512^2
// FP32, 64 -> 32 frames: 1711 -> 1512; smaller launches lose at larger frames), in
// whole windows: for the angular spectrum the nearest number, for Fresnel no more
// than fit (about 2^27 pixels of frames, us, with one window of 32 frames and with two:
// angular spectrum, rows x columns, 320x512 794 and 679, 384^2 1235 and 1191, 1280x128
// 1043 and 996, 128x1280 1355 and 1384, 1280x256 mixed 871 and 824, where 51 to 57
// frames fit; 384x512 785 and 756, 256x800 1254 and 1283, where 40 to 43 fit; Fresnel
// 320x512 875 and 920, 384^2 1041 and 1016, 1280x128 875 and 988).
// set_frames: the caller's frames per chunk (0: automatic).
//
// uploaded: frames from host memory, whose chunks are copied in and out beside the
// kernels of others.  Their chunks keep the size without overlap where that shares a
// quarter of its new frames or less: the copies take far longer than the kernels,
// and those of larger chunks get in each other's way (us, median, with the size
// without overlap and with the larger: 4096 frames of 256^2 W 32 stride 16 7,995 to
// 8,269 and 8,375 to 10,200, 2048 of stride 8 6,167 to 6,227 and 6,930, but 512 of
// stride 16 1,360 and 1,288; 211 of 1024x512 stride 16, a third shared, 7,086 and
// 6,430, 1024 of 384^2 W 64 stride 16, 48 frames for 16 new ones, 13,500 and 6,830).
inline Chunk stft_chunk(long pix, int cplx, bool as, int set_frames, int w, int stride, int nwin,
                        bool uploaded = false) {
  const long per = pix * cplx * 3 / 2;
  long f = set_frames > 0 ? set_frames : auto_frames(pix, cplx);
  if (set_frames <= 0 && (96L << 20) / per >= 32) f = std::min(f, (96L << 20) / per);
  auto windows = [&](long frames) { return frames >= w ? (frames - w) / stride + 1 : 1L; };
  long least = windows(f);
  // one window more where that is nearer to f, and no more than the 64 frames of auto_frames
  const long more = least * stride + w;
  if (as && set_frames <= 0 && stride >= w && f < 64 && more <= 64 && 2 * (more - f) < stride) ++least;
  least = std::min<long>(least, nwin);
  long g = least;
  if (set_frames <= 0 && stride < w && !(uploaded && 4L * (w - stride) <= least * stride)) {
    g = std::max(g, std::min(16L * (w - stride) / stride + 1, windows((1L << 30) / per)));
    const long chunks = (nwin + g - 1) / g;  // of even size
    g = (nwin + chunks - 1) / chunks;
  }
  return {(int)g, (int)std::min(least, g)};
}

// reserve(g) makes room for chunks of g windows, and gives back what it made on
// failure; where it fails for want of memory (status `no_room`), chunks of
// c.least windows.  The windows to take go to c.windows.
template <class S, class F>
S with_room(Chunk& c, S no_room, F&& reserve) {
  S s = reserve(c.windows);
  if (s == no_room && c.least < c.windows) {
    c.windows = c.least;
    s = reserve(c.windows);
  }
  return s;
}

}  // namespace hvc
