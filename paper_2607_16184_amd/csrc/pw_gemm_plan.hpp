// The plan of a paged GEMM call: which kernels serve its expert ranges, how the
// down projection is split, the workspace that takes, and whether work is
// forked to the layer's own stream. Pure functions of the layer's shape, its
// page counts and the batch: no HIP, so that the rules run on the CPU as well.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

#include "pw.h"

namespace pw {

// Capacity of the static device scratch of the allocation-free GEMM entry point.
constexpr size_t kStaticScratchBytes = size_t(64) << 20;

// Device workspace layout of pw_moe_paged_gemm.
enum class GemmPath { kDecode, kStream, kTiled };

// One expert range of a call, run by its own GEMM launches: the routed
// experts [0, E - n_shared), and the shared experts (the last n_shared, each
// used by every token). Its kernel path, the decode kernels' slot tiles per
// pass and the down projection's K splits follow the range's own slots.
struct RangePlan {
  int e0, ne;          // experts [e0, e0 + ne)
  size_t S;            // slots routed to them
  GemmPath path;
  int nsplit, kb_per_split, mtb;
  int rt;              // row tiles per wave of the decode kernels (row_tiles)
};

struct WsLayout {
  size_t h_off, h_bytes, op_off, op_bytes, total;
  RangePlan r[2];      // routed, shared (ne = 0 without shared experts)
};

constexpr size_t kCUs = 256;

// The tiled kernel's slot tiles: 256 slots, or 128 while an expert's expected
// slots fit one of those with some room for the spread of the routing:
// half-filled tiles would multiply and stage padding, while two 128-slot tiles
// read the weights twice. Measured (256 / 128 slots, us a step): 8 experts of
// 4096 x 14336 at 75 slots per expert 560 / 490, 105: 567 / 500, 140: 628 / 746,
// 194: 672 / 788; 64 experts of 2048 x 1408 at 75: 291 / 247, 112: 309 / 275,
// 187: 326 / 399.
constexpr int kTileNarrow = 120;

// Below this many slots per expert an expert's slots are about one tile.
constexpr int kOneTileBelow = 128;

// Whether a routed range of 49 to 127 slots per expert runs the tiled kernel, by
// its gate/up tiles (`blocks`: one per expert and 128 rows of F). Figures:
// streaming / tiled, us a step, 25 % of the pages at 16 and at 8 bits.
//   A tile takes its time however few there are, and the streaming kernel's
//   smaller ones, two workgroups per CU, spread the work; half the CUs' worth of
//   large tiles is about one round of it: 128 tiles, 4 experts of 4096 x 4096 at 75
//   slots 116 / 127, 8 of 2048 x 2048 80 / 80; 144, 4 of 4096 x 4608 135 / 133, 8 of 2048
//   x 2304 96 / 82, 16 of 1024 x 1152 68 / 58; 224, 4 of 4096 x 7168 208 / 167, 8 of
//   4096 x 3584 213 / 160, 32 of 1024 x 896 88 / 63.
//   From 16 experts on, half the CUs is enough at 65 to 120 slots, where an expert
//   takes two 64-slot tiles but one of 128 (128 tiles at 75: 16 of 1024 x 1024 60 /
//   55, 32 of 1024 x 512 64 / 57; at 52 and 16 experts 53 / 56).
//   With 8 to 15 experts of up to 56 slots, one 64-slot tile each, the streaming
//   kernel keeps its round (8 of 4096 x 2304 at 52 101 / 114, x 3072 120 / 128; 4 of
//   4096 x 6144 166 / 140; 8 of 4096 x 2304 at 62 124 / 116).
//   At 121 to 127, with half-filled 256-slot tiles, 8 experts take three quarters
//   of the CUs (144 tiles, 8 of 2048 x 2304 100 / 106; 192, x 3072 127 / 116) and
//   fewer a tile for every CU (4 of 1024 x 7168 120 / 129).
inline bool few_experts_tiled(int ne, size_t expect, size_t blocks) {
  if (blocks >= kCUs) return true;
  const bool more = 2 * blocks > kCUs;
  if (expect > static_cast<size_t>(kTileNarrow)) return ne >= 16 ? more : ne >= 8 && 4 * blocks >= 3 * kCUs;
  if (ne >= 16 && 2 * blocks == kCUs) return expect > 64;
  return more && (expect > 56 || ne < 8 || ne >= 16);
}

// Which GEMM kernels serve a range, from its expected slots per expert
// S / ne: up to 48, the decode kernels (weights streamed in registers, exact
// code-domain arithmetic, up to four 16-slot tiles per pass); above, the
// LDS-tiled kernel (256 weight rows x 128 or 256 slots) or the streaming one
// (64-slot tiles). The streaming kernel serves
//   bit-plane layers, and shapes whose down projection is not a multiple of
//   256 rows;
//   ranges below 128 slots per expert whose gate/up has tiles for about half of
//   the CUs or fewer (few_experts_tiled);
//   shared experts whose tiles do not fill the chip (a few experts with a few
//   hundred slots each in a decode-sized batch).
// The last two kernels need 32/64-row staging inside one page, 128-row down
// blocks and 32-bit activation row offsets (and the tiled kernel 256-row down
// blocks).
inline GemmPath pick_path(const pw_layer_desc& d, size_t S, size_t S_all, int ne, bool apl, bool shared) {
  const size_t expect = (S + ne - 1) / ne;
  const bool fits = S_all * d.F * 2 < (size_t(1) << 32) && S_all * d.H * 2 < (size_t(1) << 32);
  const bool tiles = fits && d.G >= 64 && d.R % 64 == 0 && d.F % 128 == 0;
  // nested bit-plane pages are read by the streaming kernel only
  if (apl) return GemmPath::kStream;
  if (expect > 48 && tiles && d.H % 256 == 0) {
    const size_t blocks = static_cast<size_t>(ne) * (d.F / 128);
    if (shared) return blocks * ((expect + 255) / 256) < kCUs ? GemmPath::kStream : GemmPath::kTiled;
    return expect >= kOneTileBelow || few_experts_tiled(ne, expect, blocks) ? GemmPath::kTiled : GemmPath::kStream;
  }
  if (expect > 48 && tiles && d.H % 128 == 0) return GemmPath::kStream;
  return GemmPath::kDecode;
}

inline RangePlan plan_range(const pw_layer_desc& d, int e0, int ne, size_t S, size_t S_all, bool apl) {
  RangePlan r{};
  r.e0 = e0;
  r.ne = ne;
  r.S = S;
  if (ne <= 0) {
    r.nsplit = 1;
    r.kb_per_split = d.F / 128;
    r.mtb = 1;
    return r;
  }
  const int nkbF = d.F / 128;
  const int expect = static_cast<int>((S + ne - 1) / ne);
  r.path = pick_path(d, S, S_all, ne, apl, e0 > 0);
  // The decode kernels split the down projection's K = F when too few
  // (expert, 64-row block) units exist to fill the chip; deterministic in
  // (desc, T, K). At four slot tiles a workgroup covers 256 rows, so fewer
  // workgroups result, and that is kept: with that many slots per expert the
  // fp32 partials of a split cost more than the fuller chip gains.
  int nsplit = 1;
  if (r.path == GemmPath::kDecode && S <= 4096) {
    const size_t active = std::min<size_t>(ne, S);
    const size_t units = active * (d.H / 64);
    nsplit = static_cast<int>(std::max<size_t>(1, std::min<size_t>(8, 2048 / std::max<size_t>(units, 1))));
  }
  // likewise the streaming kernel with 32-slot tiles (bit-plane layers at
  // decode sizes): 128-row down workgroups, two per CU
  if (r.path == GemmPath::kStream && apl && expect <= 24 && S <= 4096) {
    const size_t active = std::min<size_t>(ne, S);
    const size_t units = active * (d.H / 128);
    nsplit = static_cast<int>(std::max<size_t>(1, std::min<size_t>(8, 1024 / std::max<size_t>(units, 1))));
  }
  // and the tiled kernel in two, by the tiles that its down projection has
  // (one workgroup per CU). From 128 slots per expert: where they fill fewer
  // than three rounds of the chip, so that the last, partly filled round weighs
  // less. One split, or more than two, is at times better (8 experts of 4096 x
  // 14336, one / two / three / four splits, us a step: 777 tokens 795 / 794 /
  // 746 / 772, 1200 tokens 1020 / 1038 / 1049 / 1063). Below, about one tile per
  // expert and 256 rows: where the halves still fit one round (one / two: 80
  // slots each, 8 experts of 2048 x 4096 123 / 92, of 4096 x 7168 284 / 252, of
  // 4096 x 14336 542 / 480, 32 of 1024 x 1024 64 / 62, 16 of 1024 x 2048 77 / 63; 126
  // slots, 8 of 4096 x 14336 722 / 584, 32 of 1024 x 1024 82 / 75); with
  // more tiles the partials cost more than the halves save (80 slots, 32 of
  // 2048 x 512 75 / 86, 64 of 1024 x 512 63 / 74, of 2048 x 1408 222 / 243; 126
  // slots 96 / 109, 77 / 91, 273 / 300).
  if (r.path == GemmPath::kTiled) {
    const size_t rows = d.H / 256, one = static_cast<size_t>(ne) * rows;
    nsplit = expect < kOneTileBelow ? (2 * one <= kCUs ? 2 : 1) : (S / 256 * rows + one < 3 * kCUs ? 2 : 1);
  }
  nsplit = std::min(nsplit, nkbF);
  // a split holds whole quantization groups (G = 256, 512 span 2, 4 blocks)
  const int bpg = d.G > 128 ? d.G / 128 : 1;
  r.kb_per_split = ((nkbF + nsplit - 1) / nsplit + bpg - 1) / bpg * bpg;
  r.nsplit = (nkbF + r.kb_per_split - 1) / r.kb_per_split;
  // slot tiles per pass of the decode kernels: 1, 2 or 4 (with 4, a wave
  // streams two 16-row weight tiles)
  r.mtb = expect <= 12 ? 1 : expect <= 20 ? 2 : 4;
  r.rt = 1;
  return r;
}

// 16-row weight tiles per wave of the decode kernels at one or two slot tiles
// per pass (the bits are the same either way), for a whole expert range. Two
// halve the LDS operand reads and the activation staging per weight byte, which
// is what waves on 8- and 4-bit pages spend their issue slots on; waves on
// 16-bit pages wait for memory, and there half as many, longer workgroups
// balance worse, the more so the longer their rows. So two where the
// workgroups still cover the chip and
//   at two slot tiles, at most an eighth of the pages are 16-bit (one / two, us
//   a step: 8 experts of 4096 x 14336, 64 tokens, no 16-bit page 231 / 202, 12 %
//   253 / 241, 25 % 284 / 281, 50 % 347 / 357; of 4096 x 4096, 12 % 96 / 93);
//   at one, the share of 16-bit pages times H is at most 128 up to H = 2048, and 96
//   above (9 slots per expert, 25 % of the pages 8-bit: 8 experts of 4096 x 14336,
//   none 207 / 184, 2 % 203 / 200, 3 % 208 / 204, 6 % 213 / 217, 12 % 230 / 238, of
//   4096 x 4096, 2 % 76 / 72, and with 4 slots 3 % 72 / 75; 16 of 4096 x 2048, none
//   79 / 73, 3 % 78 / 81, 12 % 89 / 93; 8 of 2048 x 4096, none 49 / 45, 6 % 51 / 49,
//   12 % 54.5 / 55.1; 64 of 1024 x 1408, none 72 / 62, 6 % 76 / 68, 12 % 80 / 74), and
//   every expert expects two slots or more (4 tokens: 8 of 4096 x 4096 53 / 55, one
//   token of 4096 x 14336 62 / 66).
inline int row_tiles(const pw_layer_desc& d, size_t n_16, size_t n_pages, const RangePlan& r) {
  const size_t ne = static_cast<size_t>(r.ne);
  if (ne * (d.F / 64) < kCUs) return 1;
  if (r.mtb == 2) return n_16 * 8 <= n_pages ? 2 : 1;
  return n_16 * d.H <= (d.H <= 2048 ? 128 : 96) * n_pages && r.S >= 2 * ne ? 2 : 1;
}

// The workspace of a call that has `ws_bytes` of it. A tiled range below
// kOneTileBelow needs one copy of the down partials, as it did when the
// streaming kernel, which does not split, served it: where two do not fit, it
// runs unsplit. The call is refused where `total` is still above ws_bytes.
// Without a limit, `total` is what the plan can use (pw_workspace_bytes).
inline WsLayout ws_layout(const pw_layer_desc& d, int T, int K, bool apl, int n_shared, size_t ws_bytes = SIZE_MAX) {
  WsLayout w{};
  const size_t S = static_cast<size_t>(T) * K;
  const size_t S_sh = static_cast<size_t>(T) * n_shared;
  w.r[0] = plan_range(d, 0, d.E - n_shared, S - S_sh, S, apl);
  w.r[1] = plan_range(d, d.E - n_shared, n_shared, S_sh, S, apl);
  auto al = [](size_t b) { return (b + 255) / 256 * 256; };
  auto place = [&]() {
    w.h_off = 0;
    w.h_bytes = al(S * d.F * 2);
    w.op_off = w.h_bytes;
    w.op_bytes = al(static_cast<size_t>(std::max(w.r[0].nsplit, w.r[1].nsplit)) * S * d.H * 4);
    w.total = w.h_bytes + w.op_bytes;
  };
  place();
  if (w.total > ws_bytes) {
    for (RangePlan& r : w.r) {
      if (r.ne <= 0 || r.path != GemmPath::kTiled || (r.S + r.ne - 1) / r.ne >= kOneTileBelow) continue;
      r.nsplit = 1;
      r.kb_per_split = d.F / 128;
    }
    place();
  }
  return w;
}

// Whether a call forks work to the layer's own stream. A fork and join cost a
// few microseconds in a graph; call by call the launches, event records and
// cross-stream waits take the host 60 to 70 us a step, which hides only behind
// enough work. In layers of kForkPages or more every call may fork; below, the
// shared experts fork where that pays, by what the step reads.
//
// Shared experts, whose few workgroups run beside the routed ones (one stream /
// forked, us a step; page bytes and tokens):
//   in a graph, from about 20 MiB of pages of experts in use (60 + 4 experts: 48
//     MiB, 1 token 36 / 47, 4 41 / 47, 16 47 / 46, 64 63 / 56, 512 91 / 74; 96
//     MiB, 1 40 / 47, 4 48 / 47, 128 74 / 67; 192 MiB, 1 47 / 48, 4 61 / 54; 16 + 1
//     experts, 102 MiB, 1 54 / 47);
//   call by call, from about 6400 MiB times tokens (60 + 4: 48 MiB, 256 tokens 71 /
//     72, 512 86 / 80; 96 MiB, 128 71 / 73, 256 81 / 82, 1024 107 / 100; 192 MiB, 16
//     64 / 71, 64 88 / 89, 256 108 / 95; 32 + 2, 51 MiB, 128 70 / 71, 256 80 / 73; 16 +
//     1, 102 MiB, 16 61 / 69, 64 91 / 85; 64 + 1, 146 MiB, 16 57 / 71, 64 81 / 79);
//   from kForkPages on always (288 MiB, 64 tokens 113 / 106, 512 166 / 152; 528 MiB,
//     128 170 / 159; at a few tokens call by call it costs: 288 MiB, 1 token 54 / 71,
//     16 82 / 85).
// The second routed chain forks only under stream capture, in layers of
// kForkPages or more and where every expert expects a slot. In a graph it gains
// in large layers of few experts (one chain / two: 8 experts of 4096 x 14336, 16
// tokens 342 / 336, 64 tokens 362 / 355; no 16-bit page, 4 tokens 134 / 129), is
// even around 500 MiB (of 4096 x 4096, 557 MiB, 4 tokens 84 / 86, 16 118 / 116, 64
// 130 / 127, 100 135 / 136; 64 experts of 2048 x 1408, 766 MiB, 16 tokens 122 / 123,
// 64 158 / 159) and costs a little around 300 (of 2048 x 4096, 278 MiB, 16 tokens
// 69 / 72, 64 80 / 79); call by call it loses (8 experts of 4096 x 14336, 64 tokens
// 358 / 362; of 2048 x 4096 75 / 85).
constexpr uint64_t kForkPages = uint64_t(256) << 20;
constexpr uint64_t kForkGraphBytes = uint64_t(20) << 20;
constexpr uint64_t kForkByteTokens = uint64_t(6400) << 20;

// The shared experts' launches beside the routed ones.
inline bool fork_shared(const WsLayout& w, const pw_layer_desc& d, int T, uint64_t pages, bool captured) {
  if (w.r[0].ne <= 0 || w.r[1].ne <= 0) return false;
  if (pages >= kForkPages) return true;
  const uint64_t used = std::min<uint64_t>(d.E, w.r[0].S + static_cast<uint64_t>(w.r[1].ne));   // experts in use
  return captured ? pages / d.E * used >= kForkGraphBytes : pages * static_cast<uint64_t>(T) >= kForkByteTokens;
}

// The routed range as two chains, under capture.
inline bool fork_chains(const WsLayout& w, uint64_t pages) {
  const RangePlan& r = w.r[0];
  return pages >= kForkPages && w.r[1].ne <= 0 && r.path == GemmPath::kDecode && r.ne >= 2 &&
         r.S >= static_cast<size_t>(r.ne);
}

}  // namespace pw
