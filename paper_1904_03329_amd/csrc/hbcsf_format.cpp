// Host-side format builder: COO -> per-mode HB-CSF (Sections III-B, IV, V).
//
// For the root mode n the nonzeros are sorted by (root, middle level(s), leaf) index, which
// gives the compressed-sparse-fiber tree (Section III-B).  The levels below the root follow one list of modes
// whatever the root is, so the nonzeros are sorted by that list once and every mode's order is one stable sort
// of the result by the mode's own index.  Each slice is then put into one of
// three groups (Section V and Section VI-D: one nonzero -> COO; every fiber a single nonzero
// -> CSL; otherwise CSF).  Inside the CSL and CSF groups the group's nonzero stream is cut
// into runs of T_f nonzeros: a fiber is cut wherever it crosses a run boundary (fbr-split,
// Sections IV-B and VI-B, so no segment exceeds T_f nonzeros), and a slice that crosses a run
// boundary is handled by several lane groups whose partial rows are merged with atomic adds
// (slc-split, Section IV-A: slices stay whole in the arrays, more workers are assigned).
// The run tables say which slice / segment holds the first nonzero of each run.

#include "hbcsf_internal.h"

#include <algorithm>
#include <chrono>
#include <cstring>
#include <memory>
#include <utility>

#include <omp.h>

namespace hbcsf {
namespace {

// Chunks to cut n items into for the threads: not so small that a parallel region costs more than it saves.
int chunks_for(size_t n) {
  const size_t most = n / 8192 + 1;
  const int nt = omp_get_max_threads();
  return (size_t)nt < most ? nt : (int)most;
}

// Stable parallel LSD radix sort of (key, payload) pairs on key bits fromBit .. fromBit + totalBits - 1.
// On return k / v point at the sorted data (either the first or the second buffer pair).
template <typename Key>
void radix_sort_pairs(Key*& k, uint32_t*& v, Key*& k2, uint32_t*& v2, size_t n, int fromBit, int totalBits) {
  if (n < 2 || totalBits <= 0) return;
  const int passes = (totalBits + 11) / 12;
  const int digit = (totalBits + passes - 1) / passes;
  const size_t buckets = (size_t)1 << digit;
  const int nt = chunks_for(n);
  // (a chunk's counts begin two lines past a whole power of two: the pass over one bucket of all chunks would otherwise
  // go through a single cache set, and each of its loads wait for the store before it, whose address ends in the same bits)
  const size_t row = buckets + 16;
  std::vector<size_t> hist((size_t)nt * row);
  for (int pass = 0; pass < passes; ++pass) {
    const int shift = fromBit + pass * digit;
    std::fill(hist.begin(), hist.end(), 0);
    const Key* src = k;
    const uint32_t* srcv = v;
    Key* dst = k2;
    uint32_t* dstv = v2;
    // The data is cut into nt chunks and the loops run over chunk numbers, so the result does not depend on how
    // many threads the runtime really grants.
#pragma omp parallel num_threads(nt)
    {
#pragma omp for schedule(static, 1)
      for (int c = 0; c < nt; ++c) {
        const size_t lo = n * (size_t)c / nt, hi = n * (size_t)(c + 1) / nt;
        size_t* h = &hist[(size_t)c * row];
        for (size_t i = lo; i < hi; ++i) ++h[(size_t)(src[i] >> shift) & (buckets - 1)];
      }
#pragma omp single
      {
        size_t run = 0;
        for (size_t d = 0; d < buckets; ++d)
          for (int tt = 0; tt < nt; ++tt) {
            const size_t c = hist[(size_t)tt * row + d];
            hist[(size_t)tt * row + d] = run;
            run += c;
          }
      }
#pragma omp for schedule(static, 1)
      for (int c = 0; c < nt; ++c) {
        const size_t lo = n * (size_t)c / nt, hi = n * (size_t)(c + 1) / nt;
        size_t* h = &hist[(size_t)c * row];
        for (size_t i = lo; i < hi; ++i) {
          const size_t at = h[(size_t)(src[i] >> shift) & (buckets - 1)]++;
          dst[at] = src[i];
          dstv[at] = srcv[i];
        }
      }
    }
    std::swap(k, k2);
    std::swap(v, v2);
  }
}

// Where the bits of each tree level lie in a packed (root, ..., leaf) key.
struct KeyLayout {
  int lv[HBCSF_MAX_ORDER];     // mode of each level
  int shift[HBCSF_MAX_ORDER];  // by level
  uint64_t mask[HBCSF_MAX_ORDER];
  int total;
};

KeyLayout key_layout(int N, const uint64_t* dims, const int* lv) {
  KeyLayout k{};
  for (int l = N - 1; l >= 0; --l) {
    const int b = bits_for(dims[lv[l]]);
    k.lv[l] = lv[l];
    k.shift[l] = k.total;
    k.mask[l] = (1ull << b) - 1;
    k.total += b;
  }
  return k;
}

// The nonzeros in the common order, and two buffer pairs in which one mode after the other is sorted: 12 bytes (20 with
// wide keys) a nonzero and pair.  The mode that is sorted already comes first; the last one sorts in the common order's own
// buffers, so that of a large tensor the last mode but one and the last can give back what their sort did not end in before
// their arrays are made, and none gives back pages that a later mode asks for again.  Peak of a build, 20 M nonzeros of order
// 3 / 10 M of order 4: 51 / 73 bytes a nonzero (75 / 97 with all pairs kept to the end, in the same time).
template <typename Key>
struct Sorted {
  std::unique_ptr<Key[]> key[3];
  std::unique_ptr<uint32_t[]> val[3];
  Key* K = nullptr;  // the common order: one of the three buffers
  uint32_t* V = nullptr;
  KeyLayout at;
  int spare[2];      // the other two buffers

  bool alloc(int i, size_t M) {
    if (!key[i]) key[i].reset(new (std::nothrow) Key[M + 1]);
    if (!val[i]) val[i].reset(new (std::nothrow) uint32_t[M + 1]);
    return key[i] && val[i];
  }
  void release(int i) {
    key[i].reset();
    val[i].reset();
  }
};

template <typename Key>
int sort_common(int N, const uint64_t* dims, size_t M, const uint32_t* const* inds, const float* vals,
                const KeyLayout& at, Sorted<Key>* so, std::string* err) {
  so->at = at;
  if (!so->alloc(0, M) || !so->alloc(1, M)) {
    *err = "out of host memory while sorting";
    return HBCSF_ENOMEM;
  }
  Key* K = so->key[0].get();
  Key* K2 = so->key[1].get();
  uint32_t* V = so->val[0].get();
  uint32_t* V2 = so->val[1].get();
  const int nt = chunks_for(M);
  int bad = 0;
  int unsorted = 0;
#pragma omp parallel for schedule(static) reduction(| : bad) num_threads(nt)
  for (int64_t z = 0; z < (int64_t)M; ++z) {
    Key key = 0;
    for (int l = 0; l < N; ++l) {
      const uint32_t i = inds[at.lv[l]][z];
      if ((uint64_t)i >= dims[at.lv[l]]) bad |= 1;
      key |= (Key)i << at.shift[l];
    }
    K[z] = key;
    uint32_t vb;
    std::memcpy(&vb, &vals[z], 4);
    V[z] = vb;
  }
  if (bad) {
    *err = "an index is not below its dimension";
    return HBCSF_ERANGE;
  }
#pragma omp parallel for schedule(static) reduction(| : unsorted) num_threads(nt)
  for (int64_t z = 1; z < (int64_t)M; ++z)
    if (K[z] < K[z - 1]) unsorted |= 1;
  if (unsorted) radix_sort_pairs<Key>(K, V, K2, V2, M, 0, at.total);
  so->K = K;
  so->V = V;
  const int common = K == so->key[0].get() ? 0 : 1;
  so->spare[0] = 1 - common;
  so->spare[1] = 2;
  return HBCSF_OK;
}

// One mode's representation from the common order, which the last mode may overwrite.  left: modes still to come.
template <typename Key>
int build_mode_t(int order, const uint64_t* dims, uint64_t nnz, Sorted<Key>& so, const hbcsf_opts& opts, int mode,
                 int left, ModeFormat* out, std::string* err) {
  const bool last = left == 0;
  const auto t_begin = std::chrono::steady_clock::now();
  const int N = order;
  const uint32_t L = opts.fiber_threshold ? opts.fiber_threshold : 64;
  const uint32_t gmask = opts.group_mask == 0 ? 3u : (opts.group_mask & 3u);
  const int bb = mid_block_bits(order, dims, opts, mode);   // level-1 blocking: block number above the root in the key
  const bool cooOn = (gmask & 1u) && bb == 0, cslOn = gmask & 2u;

  // Tree levels: root = the target mode; the other modes ordered by the policy.
  int lv[HBCSF_MAX_ORDER];
  level_order(N, dims, mode, opts.mode_order_policy, lv);
  const KeyLayout kl = key_layout(N, dims, lv);
  const int* shift = kl.shift;
  const uint64_t* mask = kl.mask;

  out->order = N;
  out->mode = mode;
  out->L = L;
  out->cooRowFlags = opts.coo_row_flags == 1;
  out->blockBits = bb;
  out->rows = dims[mode];
  for (int l = 0; l < N; ++l) out->levelMode[l] = lv[l];

  // ---- this mode's order: a stable sort of the common one by (block,) root; the value rides along as payload ----
  const size_t M = (size_t)nnz;
  const int nt = chunks_for(M);
  Key* K = so.K;
  uint32_t* V = so.V;
  const bool sorted = mode == so.at.lv[0] && bb == 0;  // the common order is this mode's own
  if (!sorted) {
    if (!so.key[so.spare[0]]) std::swap(so.spare[0], so.spare[1]);
    const int other = last ? 3 - so.spare[0] - so.spare[1] : so.spare[1];
    if (!so.alloc(so.spare[0], M) || !so.alloc(other, M)) {
      *err = "out of host memory while sorting";
      return HBCSF_ENOMEM;
    }
    K = so.key[so.spare[0]].get();
    V = so.val[so.spare[0]].get();
    Key* K2 = so.key[other].get();
    uint32_t* V2 = so.val[other].get();
    int from[HBCSF_MAX_ORDER];
    for (int l = 0; l < N; ++l)
      for (int c = 0; c < N; ++c)
        if (so.at.lv[c] == lv[l]) from[l] = so.at.shift[c];
    const int drop = bb ? bits_for(dims[lv[1]]) - bb : 0;
#pragma omp parallel for schedule(static) num_threads(nt)
    for (int64_t z = 0; z < (int64_t)M; ++z) {
      const Key c = so.K[z];
      Key key = 0;
      for (int l = 0; l < N; ++l) {
        const uint64_t i = (uint64_t)(c >> from[l]) & mask[l];
        key |= (Key)i << shift[l];
        if (l == 1 && bb) key |= (Key)(i >> drop) << kl.total;
      }
      K[z] = key;
      V[z] = so.V[z];
    }
    radix_sort_pairs<Key>(K, V, K2, V2, M, shift[0], kl.total - shift[0] + bb);
  }
  // Buffers are given back only where the allocator maps each by itself, from 32 MB on: smaller ones stay with the process
  // either way, and freed before the arrays are made they leave the top of its heap, which is then cut and faulted in again.
  if ((last || (left == 1 && !sorted)) && M * sizeof(Key) >= ((size_t)32 << 20))
    for (int i = 0; i < 3; ++i)
      if (so.key[i].get() != K && (last || so.key[i].get() != so.K)) so.release(i);

  auto idx = [&](int l, size_t p) -> uint32_t { return (uint32_t)((uint64_t)(K[p] >> shift[l]) & mask[l]); };
  auto fresh = [&](int l, size_t p) -> bool { return p == 0 || (K[p] >> shift[l]) != (K[p - 1] >> shift[l]); };

  // ---- slices ----
  const int NF = N - 2;  // fiber levels 1..NF
  std::vector<uint64_t> tcount[HBCSF_MAX_ORDER - 1];  // by level: slices, then fibers, before each chunk
  for (int l = 0; l <= NF; ++l) tcount[l].assign(nt + 1, 0);
#pragma omp parallel for schedule(static, 1) num_threads(nt)
  for (int t = 0; t < nt; ++t) {  // chunk numbers, not thread numbers: any team size gives the same result
    const size_t lo = M * (size_t)t / nt, hi = M * (size_t)(t + 1) / nt;
    uint64_t c[HBCSF_MAX_ORDER - 1] = {};
    for (size_t p = lo; p < hi; ++p) {
      const Key x = p == 0 ? ~(Key)0 : K[p] ^ K[p - 1];  // fresh() of all levels from one difference
      for (int l = 0; l <= NF; ++l) c[l] += (x >> shift[l]) != 0;
    }
    for (int l = 0; l <= NF; ++l) tcount[l][t + 1] = c[l];
  }
  for (int l = 0; l <= NF; ++l)
    for (int t = 0; t < nt; ++t) tcount[l][t + 1] += tcount[l][t];
  const uint64_t S = tcount[0][nt];
  std::vector<uint32_t> sStart(S + 1);
  std::vector<uint32_t> fStart[HBCSF_MAX_FIBER_LEVELS];  // fibers of each level before every slice
  for (int f = 0; f < NF; ++f) fStart[f].resize(S + 1);
#pragma omp parallel for schedule(static, 1) num_threads(nt)
  for (int t = 0; t < nt; ++t) {
    const size_t lo = M * (size_t)t / nt, hi = M * (size_t)(t + 1) / nt;
    uint64_t c[HBCSF_MAX_ORDER - 1] = {};
    for (int l = 0; l <= NF; ++l) c[l] = tcount[l][t];
    for (size_t p = lo; p < hi; ++p) {
      const Key x = p == 0 ? ~(Key)0 : K[p] ^ K[p - 1];
      if ((x >> shift[0]) != 0) {
        for (int f = 0; f < NF; ++f) fStart[f][c[0]] = (uint32_t)c[1 + f];
        sStart[c[0]] = (uint32_t)p;
      }
      for (int l = 0; l <= NF; ++l) c[l] += (x >> shift[l]) != 0;
    }
  }
  sStart[S] = (uint32_t)M;
  for (int f = 0; f < NF; ++f) fStart[f][S] = (uint32_t)tcount[1 + f][nt];

  // ---- classify slices (Section V; Section VI-D) ----
  // Per slice (the paper's rule): one nonzero -> COO; every deepest-level fiber a singleton -> CSL; else CSF.
  // With hybrid_granularity = 1 the choice is made per fiber inside heavy slices: a slice of at least 2 L
  // nonzeros (it spans several runs, so its row is merged with atomic adds anyway) of which at least an eighth
  // sit in singleton deepest-level fibers is split: those nonzeros form a CSL-group slice of the same root index,
  // the others a CSF-group slice; both pieces are marked shared.
  const bool perFiber = opts.hybrid_granularity == 1 && cslOn;
  // a nonzero whose deepest-level fiber holds only itself
  auto single = [&](size_t p, size_t e) -> bool { return fresh(NF, p) && (p + 1 == e || fresh(NF, p + 1)); };
  constexpr uint8_t kSplit = 3;  // CSL piece + CSF piece
  std::vector<uint8_t> grp(S);
  std::vector<uint32_t> nSingle(perFiber ? S : 0);
  constexpr int kFL = HBCSF_MAX_FIBER_LEVELS;
  uint64_t fibNat[kFL] = {0, 0, 0};
  uint64_t fibNatCsf[kFL] = {0, 0, 0};
  {
    uint64_t f0 = 0, f1 = 0, f2 = 0, c0 = 0, c1 = 0, c2 = 0;
#pragma omp parallel for schedule(dynamic, 64) reduction(+ : f0, f1, f2, c0, c1, c2) num_threads(nt)
    for (int64_t s = 0; s < (int64_t)S; ++s) {
      const size_t b = sStart[s], e = sStart[s + 1];
      uint64_t nf[kFL] = {0, 0, 0};
      for (int f = 0; f < NF; ++f) nf[f] = fStart[f][s + 1] - fStart[f][s];
      const uint64_t n = e - b, deep = nf[NF - 1];
      uint8_t g;
      if (n == 1 && cooOn) g = kCoo;
      else if (deep == n && cslOn) g = kCsl;
      else g = kCsf;
      uint64_t kept[kFL] = {nf[0], nf[1], nf[2]};  // fibers that stay in the CSF group
      if (perFiber && g == kCsf && n >= 2ull * L) {
        uint64_t ns = 0;
        for (size_t p = b; p < e; ++p) ns += single(p, e);
        if (ns * 8 >= n) {
          g = kSplit;
          nSingle[s] = (uint32_t)ns;
          // fibers of the CSF piece: a fiber level counts once per run of kept nonzeros that share it
          kept[0] = kept[1] = kept[2] = 0;
          bool pend[kFL] = {false, false, false};
          for (size_t p = b; p < e; ++p) {
            for (int f = 0; f < NF; ++f) pend[f] = pend[f] || fresh(f + 1, p);
            if (single(p, e)) continue;
            for (int f = 0; f < NF; ++f) {
              kept[f] += pend[f];
              pend[f] = false;
            }
          }
        }
      }
      grp[s] = g;
      f0 += nf[0];
      f1 += nf[1];
      f2 += nf[2];
      if (g == kCsf || g == kSplit) { c0 += kept[0]; c1 += kept[1]; c2 += kept[2]; }
    }
    fibNat[0] = f0; fibNat[1] = f1; fibNat[2] = f2;
    fibNatCsf[0] = c0; fibNatCsf[1] = c1; fibNatCsf[2] = c2;
  }

  // ---- position of each slice (piece) inside its group ----
  // ord / off: the slice's entry and first nonzero in its group; a split slice's CSL piece is in ordL / offL
  std::vector<uint32_t> ord(S), off(S), ordL(perFiber ? S : 0), offL(perFiber ? S : 0);
  uint64_t gS[3] = {0, 0, 0}, gM[3] = {0, 0, 0};
  for (uint64_t s = 0; s < S; ++s) {
    const uint64_t n = sStart[s + 1] - sStart[s];
    if (grp[s] == kSplit) {
      ordL[s] = (uint32_t)gS[kCsl];
      offL[s] = (uint32_t)gM[kCsl];
      gS[kCsl] += 1;
      gM[kCsl] += nSingle[s];
      ord[s] = (uint32_t)gS[kCsf];
      off[s] = (uint32_t)gM[kCsf];
      gS[kCsf] += 1;
      gM[kCsf] += n - nSingle[s];
      continue;
    }
    const int g = grp[s];
    ord[s] = (uint32_t)gS[g];
    off[s] = (uint32_t)gM[g];
    gS[g] += 1;
    gM[g] += n;
  }

  // ---- pieces: at most kPiece nonzeros of one slice each ----
  // (a slice of a power-law tensor holds up to a fifth of all nonzeros; as one item it was the whole loop's time.)
  // A split slice is one piece: what it has kept so far decides the places.  A thread takes the pieces that begin in one
  // of `parts` equal ranges of the nonzeros.
  constexpr size_t kPiece = 4096;
  std::vector<uint64_t> pieceAt(S + 1);  // first piece of every slice
  pieceAt[0] = 0;
  for (uint64_t s = 0; s < S; ++s) {
    const size_t n = sStart[s + 1] - sStart[s];
    pieceAt[s + 1] = pieceAt[s] + (grp[s] == kSplit ? 1 : (n + kPiece - 1) / kPiece);
  }
  const uint64_t P = pieceAt[S];
  struct Piece {
    uint32_t s, b, e;
  };
  std::vector<Piece> piece(P);
#pragma omp parallel for schedule(static) num_threads(nt)
  for (int64_t s = 0; s < (int64_t)S; ++s) {
    const size_t e = sStart[s + 1];
    size_t b = sStart[s];
    for (uint64_t q = pieceAt[s]; q < pieceAt[s + 1]; ++q) {
      const size_t pe = q + 1 == pieceAt[s + 1] ? e : b + kPiece;
      piece[q] = Piece{(uint32_t)s, (uint32_t)b, (uint32_t)pe};
      b = pe;
    }
  }

  const int parts = nt > 1 ? nt * 8 : 1;
  auto piece_at = [&](int part) -> int64_t {  // first piece that begins at or behind the part's first nonzero
    const size_t z = part == parts ? M : M * (size_t)part / parts;
    return std::lower_bound(piece.begin(), piece.end(), z, [](const Piece& x, size_t at) { return x.b < at; }) - piece.begin();
  };

  // ---- count fiber segments of the CSF group (fbr-split on the run grid) ----
  // A segment starts at a kept nonzero that lies on the run grid or is the first kept one of its fiber.
  std::vector<uint32_t> segOff[kFL];  // by piece
  uint64_t nSeg[kFL] = {0, 0, 0};
  for (int f = 0; f < NF; ++f) segOff[f].assign(P + 1, 0);
#pragma omp parallel for schedule(dynamic, 1) num_threads(nt)
  for (int part = 0; part < parts; ++part)
    for (int64_t q = piece_at(part), qEnd = piece_at(part + 1); q < qEnd; ++q) {
      const uint32_t s = piece[q].s;
      if (grp[s] != kCsf && grp[s] != kSplit) continue;
      const size_t b = piece[q].b, e = piece[q].e;
      const bool split = grp[s] == kSplit;
      uint32_t c[kFL] = {0, 0, 0};
      uint32_t pos = off[s] + (uint32_t)(b - sStart[s]);
      bool pend[kFL] = {false, false, false};
      for (size_t p = b; p < e; ++p) {
        for (int f = 0; f < NF; ++f) pend[f] = pend[f] || fresh(f + 1, p);
        if (split && single(p, e)) continue;
        const bool cut = (pos % L) == 0;
        for (int f = 0; f < NF; ++f) {
          c[f] += cut || pend[f];
          pend[f] = false;
        }
        ++pos;
      }
      for (int f = 0; f < NF; ++f) segOff[f][q + 1] = c[f];
    }
  for (int f = 0; f < NF; ++f) {
    uint64_t run = 0;
    for (uint64_t q = 0; q < P; ++q) {
      const uint32_t c = segOff[f][q + 1];
      segOff[f][q] = (uint32_t)run;
      run += c;
    }
    segOff[f][P] = (uint32_t)run;
    nSeg[f] = run;
  }

  // ---- lay the arrays out in one blob ----
  layout_mode(out, N, gS, gM, nSeg);
  const uint64_t ownedWords = (out->rows + 31) / 32;
  void* mem = nullptr;
  if (posix_memalign(&mem, kAlign, (size_t)out->blobBytes) != 0 || !mem) {
    *err = "out of host memory for the format arrays";
    return HBCSF_ENOMEM;
  }
  out->blob = (uint8_t*)mem;
  auto U32 = [&](const ArrayRef& r) { return (uint32_t*)(out->blob + r.off); };
  uint32_t* owned = U32(out->ownedBits);
  std::memset(owned, 0, ownedWords * 4);
  uint32_t* cooBits = U32(out->cooBits);
  std::memset(cooBits, 0, ownedWords * 4);

  GroupFormat& Go = out->g[kCoo];
  GroupFormat& Gl = out->g[kCsl];
  GroupFormat& Gc = out->g[kCsf];
  uint32_t* cooInd[HBCSF_MAX_ORDER];
  uint32_t* cslInd[HBCSF_MAX_ORDER];
  uint32_t* csfInd[HBCSF_MAX_ORDER];
  uint32_t* csfPtr[HBCSF_MAX_ORDER];
  uint32_t* csfRun[HBCSF_MAX_ORDER];
  for (int l = 0; l < N; ++l) {
    cooInd[l] = U32(Go.ind[l]);
    cslInd[l] = U32(Gl.ind[l]);
    csfInd[l] = U32(Gc.ind[l]);
    csfPtr[l] = l < N - 1 ? U32(Gc.ptr[l]) : nullptr;
    csfRun[l] = l < N - 1 ? U32(Gc.runFirst[l]) : nullptr;
  }
  uint32_t* cooVal = U32(Go.val);
  uint32_t* cslVal = U32(Gl.val);
  uint32_t* csfVal = U32(Gc.val);
  uint32_t* cslPtr = U32(Gl.ptr[0]);
  uint32_t* cslRun = U32(Gl.runFirst[0]);

  uint64_t sharedSlices = 0;
#pragma omp parallel for schedule(dynamic, 1) reduction(+ : sharedSlices) num_threads(nt)
  for (int part = 0; part < parts; ++part)
    for (int64_t q = piece_at(part), qEnd = piece_at(part + 1); q < qEnd; ++q) {
      const uint32_t s = piece[q].s;
      const size_t b = piece[q].b, e = piece[q].e;
      const size_t sb = sStart[s], se = sStart[s + 1];
      const bool first = b == sb;  // the slice's own entries go with its first piece
      const uint32_t root = idx(0, b);
      const int g = grp[s];
      bool own = true;
      if (g == kCoo) {
        const uint32_t a = off[s];
        for (int l = out->cooRowFlags ? 1 : 0; l < N; ++l) cooInd[l][a] = idx(l, b);
        cooVal[a] = V[b];
        __atomic_fetch_or(&cooBits[root >> 5], 1u << (root & 31), __ATOMIC_RELAXED);
      } else {
        const bool split = g == kSplit;
        // the CSL piece (a whole CSL slice, or the singleton-fiber nonzeros of a split slice)
        if (g == kCsl || split) {
          const uint32_t a = split ? offL[s] : off[s], o = split ? ordL[s] : ord[s];
          const uint32_t n = split ? nSingle[s] : (uint32_t)(se - sb);
          own = !split && bb == 0 && (a / L) == ((a + n - 1) / L);
          if (first) {
            for (uint32_t r = (a + L - 1) / L; r <= (a + n - 1) / L; ++r) cslRun[r] = o;
            cslInd[0][o] = root | (own ? kOwnedBit : 0u);
            cslPtr[o] = a;
          }
          uint32_t pos = a + (uint32_t)(b - sb);
          for (size_t p = b; p < e; ++p) {
            if (split && !single(p, e)) continue;
            for (int l = 1; l < N; ++l) cslInd[l][pos] = idx(l, p);
            cslVal[pos] = V[p];
            ++pos;
          }
        }
        // the CSF piece
        if (g == kCsf || split) {
          const uint32_t a = off[s], o = ord[s];
          const uint32_t n = split ? (uint32_t)(se - sb) - nSingle[s] : (uint32_t)(se - sb);
          own = !split && bb == 0 && (a / L) == ((a + n - 1) / L);
          if (first) {
            for (uint32_t r = (a + L - 1) / L; r <= (a + n - 1) / L; ++r) csfRun[0][r] = o;
            csfInd[0][o] = root | (own ? kOwnedBit : 0u);
            csfPtr[0][o] = a;
          }
          uint32_t f[kFL] = {0, 0, 0};
          for (int k = 0; k < NF; ++k) f[k] = segOff[k][q];
          uint32_t pos = a + (uint32_t)(b - sb);
          bool pend[kFL] = {false, false, false};
          for (size_t p = b; p < e; ++p) {
            for (int k = 0; k < NF; ++k) pend[k] = pend[k] || fresh(k + 1, p);
            if (split && single(p, e)) continue;
            const bool cut = (pos % L) == 0;
            for (int l = 1; l <= NF; ++l) {
              if (cut || pend[l - 1]) {
                csfInd[l][f[l - 1]] = idx(l, p);
                csfPtr[l][f[l - 1]] = pos;
                if (cut) csfRun[l][pos / L] = f[l - 1];
                ++f[l - 1];
              }
            }
            pend[0] = pend[1] = pend[2] = false;
            csfInd[N - 1][pos] = idx(N - 1, p);
            csfVal[pos] = V[p];
            ++pos;
          }
        }
        if (!own && first) ++sharedSlices;
      }
      if (own && first) __atomic_fetch_or(&owned[root >> 5], 1u << (root & 31), __ATOMIC_RELAXED);
    }
  {
    // COO-group nonzeros are stored in row order, so a running count over the bitmap locates them
    uint32_t* cooPtr = U32(out->cooPtr);
    uint32_t run = 0;
    for (uint64_t w = 0; w < ownedWords; ++w) {
      cooPtr[w] = run;
      run += (uint32_t)__builtin_popcount(cooBits[w]);
    }
    cooPtr[ownedWords] = run;
  }
  // sentinels and pads
  cslInd[0][Gl.n[0]] = 0;
  cslPtr[Gl.n[0]] = (uint32_t)Gl.nnz;
  cslRun[Gl.runs] = (uint32_t)Gl.n[0];
  for (int l = 0; l < N - 1; ++l) {
    csfInd[l][Gc.n[l]] = 0;
    csfPtr[l][Gc.n[l]] = (uint32_t)Gc.nnz;
    csfRun[l][Gc.runs] = (uint32_t)Gc.n[l];
  }

  // ---- statistics ----
  fill_count_stats(out, N, M, S, fibNat, fibNatCsf, nSeg, gS, gM, sharedSlices);
  hbcsf_stats& st = out->stats;
  {
    uint64_t cnt = 0;
#pragma omp parallel for schedule(static) reduction(+ : cnt) num_threads(nt)
    for (int64_t w = 0; w < (int64_t)ownedWords; ++w) cnt += (uint64_t)__builtin_popcount(owned[w]);
    st.owned_rows = cnt;
  }
  {
    // distinct factor rows each group gathers, per tree level
    std::vector<uint8_t> seen;
    for (int g = 0; g < 3; ++g) {
      const GroupFormat& G = out->g[g];
      for (int l = 1; l < N; ++l) {
        const uint32_t* a = U32(G.ind[l]);
        const uint64_t cnt = (g == kCsf && l < N - 1) ? G.n[l] : G.nnz;
        uint64_t d = 0;
        if (cnt == 0) {
          d = 0;
        } else if (cnt * 16 < dims[lv[l]]) {  // few indices in a long mode: sort and count
          std::vector<uint32_t> tmp(a, a + cnt);
          std::sort(tmp.begin(), tmp.end());
          d = (uint64_t)(std::unique(tmp.begin(), tmp.end()) - tmp.begin());
        } else {
          seen.assign(dims[lv[l]], 0);
          uint8_t* sp = seen.data();
          // Looked at before it is written: a row that many nonzeros share would otherwise take its cache line from
          // one thread to the next with every one of them.  Looked at 64 at a time, without a branch, and then the new
          // ones written: a branch to the store is often predicted wrongly, and the store begun then takes the line all the
          // same, which depended on where the linker had put the loop (1 M nonzeros, all modes on 16 threads: 10.1 to
          // 14.1 ms with the loop at 16, 0, 32 or 48 bytes past a multiple of 64, now 8.8 to 9.6 at all of them).
#pragma omp parallel for schedule(static) num_threads(nt)
          for (int64_t t0 = 0; t0 < (int64_t)cnt; t0 += 64) {
            const int64_t t1 = std::min<int64_t>(t0 + 64, (int64_t)cnt);
            uint32_t fresh[64];
            int n = 0;
            for (int64_t t = t0; t < t1; ++t) {
              fresh[n] = a[t];
              n += __atomic_load_n(&sp[a[t]], __ATOMIC_RELAXED) == 0;
            }
            for (int k = 0; k < n; ++k) __atomic_store_n(&sp[fresh[k]], (uint8_t)1, __ATOMIC_RELAXED);
          }
#pragma omp parallel for schedule(static) reduction(+ : d) num_threads(nt)
          for (int64_t t = 0; t < (int64_t)seen.size(); ++t) d += sp[t];
        }
        st.distinct_rows[g][l] = d;
      }
    }
  }
  st.build_seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t_begin).count();
  return HBCSF_OK;
}

}  // namespace

namespace {

template <typename Key>
int build_modes_t(int order, const uint64_t* dims, uint64_t nnz, const uint32_t* const* inds, const float* vals,
                  const hbcsf_opts& opts, int modes, ModeFormat* const* out, std::string* err) {
  int lv[HBCSF_MAX_ORDER];
  const auto t_begin = std::chrono::steady_clock::now();
  common_order(order, dims, opts.mode_order_policy, modes == 1, lv);
  Sorted<Key> so;
  int rc = sort_common<Key>(order, dims, (size_t)nnz, inds, vals, key_layout(order, dims, lv), &so, err);
  // the sort every mode's order is taken from is part of each mode's time
  const double share = std::chrono::duration<double>(std::chrono::steady_clock::now() - t_begin).count() / modes;
  for (int k = 0; rc == HBCSF_OK && k < modes; ++k) {
    const int m = modes == 1 || k > lv[0] ? k : k == 0 ? lv[0] : k - 1;  // the common order's own mode, then the others
    rc = build_mode_t<Key>(order, dims, nnz, so, opts, m, modes - 1 - k, out[m], err);
    out[m]->stats.build_seconds += share;
  }
  return rc;
}

}  // namespace

double sum_of_squares(const float* v, uint64_t n) {
  constexpr uint64_t kBlock = 16384;
  const int64_t blocks = (int64_t)((n + kBlock - 1) / kBlock);
  std::vector<double> part((size_t)blocks);
#pragma omp parallel for schedule(static) num_threads(chunks_for(n))
  for (int64_t b = 0; b < blocks; ++b) {
    const uint64_t lo = (uint64_t)b * kBlock, hi = lo + kBlock < n ? lo + kBlock : n;
    double s[8] = {};  // one running sum alone would wait for its own last addition at every value
    uint64_t z = lo;
    for (; z + 8 <= hi; z += 8)
      for (int k = 0; k < 8; ++k) s[k] += (double)v[z + k] * (double)v[z + k];
    for (; z < hi; ++z) s[0] += (double)v[z] * (double)v[z];
    part[(size_t)b] = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
  }
  double sum = 0.0;
  for (int64_t b = 0; b < blocks; ++b) sum += part[(size_t)b];
  return sum;
}

int build_modes(int order, const uint64_t* dims, uint64_t nnz, const uint32_t* const* inds,
                const float* vals, const hbcsf_opts& opts, int modes, ModeFormat* const* out,
                std::string* err) {
  int total = 0, blocks = 0;
  for (int m = 0; m < order; ++m) total += bits_for(dims[m]);
  for (int m = 0; m < modes; ++m) {
    const int b = mid_block_bits(order, dims, opts, m);
    blocks = b > blocks ? b : blocks;
  }
  if (nnz > 0 && total + blocks > 128) {
    *err = "the packed coordinates, with a blocked mode's block number, exceed 128 bits";
    return HBCSF_ERANGE;
  }
  try {
    if (total + blocks <= 64)
      return build_modes_t<uint64_t>(order, dims, nnz, inds, vals, opts, modes, out, err);
    return build_modes_t<unsigned __int128>(order, dims, nnz, inds, vals, opts, modes, out, err);
  } catch (const std::bad_alloc&) {
    *err = "out of host memory while building the format";
    return HBCSF_ENOMEM;
  } catch (...) {
    *err = "unexpected failure while building the format";
    return HBCSF_EINVAL;
  }
}

}  // namespace hbcsf
