// HIP kernels of libtdk for gfx950 (MI355X): collective RoPE re-rotation, per-page compare,
// ballot/prefix compaction, payload gather and fused diff restore.
//
// Data movement plan shared by the three page kernels (rerotate, flag, decode):
//   - a workgroup of 4 wavefronts (8 where wide_reads or wide_writes says so) owns one master page (T rows of H*D bf16, K and V) and a group
//     of up to 32 agents of that page's session;
//   - the master page is read from HBM once, 16 bytes per lane, and stays in registers while the
//     workgroup walks its agents (Sec. 4.2: the cost of a shared block is paid once per group);
//   - the item's record is one scalar read; the per-agent cos/sin tables and where the page's rows lie in each
//     agent's pool are then asked for beside the master page and staged in LDS once per workgroup;
//   - a wavefront always handles whole rows: lane l holds 8 consecutive elements of the low half
//     and the 8 matching elements of the high half of head l/8, so both members of every rotation
//     pair sit in the same lane and each load/store instruction covers whole 128-byte segments;
//   - a row of 1, 2 or 4 KV heads fills only part of a wavefront that way, so several rows of the page share each
//     instruction then (PACK: as many as fill it, see Lane).
#include "tdk_internal.h"
#include "tdk_plan.h"

#include <algorithm>
#include <map>
#include <mutex>
#include <type_traits>

namespace tdk {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------------------------------------
// bf16 <-> fp32
// ---------------------------------------------------------------------------------------------

__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// two fp32 -> packed bf16 (a in the low half), round-to-nearest-even
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  f32x2 v = {a, b};
  bf16x2 r = __builtin_convertvector(v, bf16x2);
  return __builtin_bit_cast(uint32_t, r);
}

// y_a = fma(x_a, c, -(x_b * s)), y_b = fma(x_b, c, x_a * s): one rounded product, one fma.
__device__ __forceinline__ void rot(float xa, float xb, float c, float s, float& ya, float& yb) {
  float t = __fmul_rn(xb, s);
  float u = __fmul_rn(xa, s);
  ya = __builtin_fmaf(xa, c, -t);
  yb = __builtin_fmaf(xb, c, u);
}

// Rotates the 16 elements a lane holds.  Half style: lo[e] pairs with hi[e], table entry e.
// Interleaved style: each 32-bit word is one pair; lo uses entries 0..3, hi entries 4..7.
template <bool IL>
__device__ __forceinline__ void rotate16(const u32x4 lo, const u32x4 hi, const float (&c)[8],
                                         const float (&s)[8], u32x4& olo, u32x4& ohi) {
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    if (!IL) {
      float yl0, yh0, yl1, yh1;
      rot(bf_lo(lo[w]), bf_lo(hi[w]), c[2 * w], s[2 * w], yl0, yh0);
      rot(bf_hi(lo[w]), bf_hi(hi[w]), c[2 * w + 1], s[2 * w + 1], yl1, yh1);
      olo[w] = pack_bf16(yl0, yl1);
      ohi[w] = pack_bf16(yh0, yh1);
    } else {
      float ya, yb;
      rot(bf_lo(lo[w]), bf_hi(lo[w]), c[w], s[w], ya, yb);
      olo[w] = pack_bf16(ya, yb);
      rot(bf_lo(hi[w]), bf_hi(hi[w]), c[4 + w], s[4 + w], ya, yb);
      ohi[w] = pack_bf16(ya, yb);
    }
  }
}

// Streaming store: system-scope, non-temporal (sc0 sc1 nt).  The line is written through instead of
// staying dirty in L2 for a later kernel to flush; measured best for the page kernels' scattered
// 32 KB writes when they run back to back with the compare kernel.
template <bool NT>
__device__ __forceinline__ void st16(u32x4* p, u32x4 v) {
  // The two idle cycles keep a following VALU write of the data registers clear of the store's read
  // of them (16-byte stores need two wait states on gfx940+; the compiler cannot see into the asm).
  if (NT) asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1 nt\n\ts_nop 1" : : "v"(p), "v"(v) : "memory");
  else *p = v;
}

template <bool NT>
__device__ __forceinline__ u32x4 ld16(const u32x4* p) {
  return NT ? __builtin_nontemporal_load(p) : *p;
}

// ---------------------------------------------------------------------------------------------
// per-workgroup staging
// ---------------------------------------------------------------------------------------------

struct GroupShared {
  float   tab[kMaxGroup][2 * kHalf];  // cos[64], sin[64] of each agent of the group
  longlong2 b[kMaxGroup];             // byte of row 0 of the page in a pool plane: for the rows on its first physical page, and for
                                      // those on the next one (where row 0 would lie)
  int32_t cut[kMaxGroup];             // first row on the next one
  int32_t aux[kMaxGroup];             // flag kernel: OR of the waves; decode: 1 if the page is listed
};

// The same for rounds with per-agent block layouts: a master page can meet two segments of an agent
// (two position deltas), and its rows can land anywhere, so the pool row of every row is staged.
struct GroupSharedSeg {
  float    tab[kMaxGroup][2][2 * kHalf];
  int32_t  row[kMaxGroup][32];       // pool row of each row of the page
  uint32_t sel[kMaxGroup];           // bit r set: row r uses the second table
  int32_t  aux[kMaxGroup];
};

// A work item in scalar registers.
struct Item {
  ItemDev d;
  __device__ __forceinline__ Item(const ItemDev* list, int item) : d(scalar_read(list + __builtin_amdgcn_readfirstlane(item))) {}
  __device__ __forceinline__ int count() const { return d.counts & 255; }
  __device__ __forceinline__ int rows() const { return d.counts >> 8; }
  // agent g of the group; its (agent, page) pair; its (agent, token) pair of the page's first token
  __device__ __forceinline__ int agent(const RoundDev& rd, int g) const { return d.agent0 >= 0 ? d.agent0 + g : rd.order[d.order0 + g]; }
  __device__ __forceinline__ int flat(const RoundDev& rd, int g) const { return d.agent0 >= 0 ? d.flat0 + g * d.pages : rd.oagents[d.order0 + g].flag_off + d.page; }
  __device__ __forceinline__ int score(const RoundDev& rd, int g) const {
    return d.agent0 >= 0 ? d.score0 + g * d.span : rd.oagents[d.order0 + g].score_off + d.page * rd.page_tokens;
  }
};

// A group is staged in two steps, so that its reads and those of the master page are in flight together: what an item's first store
// waits for is the item (one scalar read), then everything else at once.  (One after the other, as branches around the loads make
// the compiler wait, it was nine vector reads; a read that no cache holds takes 0.65 us on an idle chip and 2 to 4 on a busy one: 25 agents
// x 5000 tokens, collect, restore and store 301.4 -> 297.9 us; 37 x 2999, 4 heads, one plane after the other 123.7 -> 121.5; 48 agents
// with own orders and 32-token pages, restore 104 -> 102; drawn rounds up to 1.08 times.)
struct AskedGroup { u32x4 place; float4 tab[2]; };

// Wavefronts of a page kernel's workgroup: eight with two rows of every page each where that is faster (wide_reads, wide_writes), else four.
__device__ __host__ constexpr int waves_of(int rpw, bool pack) { return !pack && rpw == 2 ? 2 * kWaves : kWaves; }

template <int W>
__device__ __forceinline__ void ask_group(const RoundDev& rd, const Item& it, const int, const GroupShared&, AskedGroup& a) {
  const int tid = threadIdx.x, n = it.count() - 1, q = tid & 31;
  a.place = reinterpret_cast<const u32x4*>(rd.places)[it.flat(rd, min(tid, n))];
  const float4* tab = reinterpret_cast<const float4*>(rd.tab);
  a.tab[0] = tab[(size_t)it.agent(rd, min(tid >> 5, n)) * (kHalf / 2) + q];
  a.tab[1] = a.tab[0];
  if (n >= 2 * W) a.tab[1] = tab[(size_t)it.agent(rd, min(2 * W + (tid >> 5), n)) * (kHalf / 2) + q];
}

template <int W>
__device__ __forceinline__ void put_group(const RoundDev& rd, const Item& it, const int T, GroupShared& sh, const AskedGroup& a) {
  const int tid = threadIdx.x, n = it.count(), q = tid & 31, g = tid >> 5;
  if (g < n) reinterpret_cast<float4*>(sh.tab[g])[q] = a.tab[0];
  if (g + 2 * W < n) reinterpret_cast<float4*>(sh.tab[g + 2 * W])[q] = a.tab[1];
  for (int g2 = g + 4 * W; g2 < n; g2 += 2 * W)
    reinterpret_cast<float4*>(sh.tab[g2])[q] = reinterpret_cast<const float4*>(rd.tab)[(size_t)it.agent(rd, g2) * (kHalf / 2) + q];
  if (tid < n) {
    const uint32_t row_bytes = (uint32_t)rd.heads * (kHeadDim * 2);
    const int off = (int)a.place[2];
    sh.b[tid] = make_longlong2(((int64_t)(int32_t)a.place[0] * T + off) * row_bytes, ((int64_t)(int32_t)a.place[1] * T + off - T) * row_bytes);
    sh.cut[tid] = T - off;
  }
}

struct AskedGroupSeg { u32x4 pt; int32_t row, sel; };

template <int W>
__device__ __forceinline__ void ask_group(const RoundDev& rd, const Item& it, const int T, const GroupSharedSeg&, AskedGroupSeg& a) {
  const int tid = threadIdx.x, n = it.count() - 1, lg = T == 16 ? 4 : 5;
  a.pt = reinterpret_cast<const u32x4*>(rd.pagetab)[it.flat(rd, min(tid >> 6, n))];
  a.sel = rd.pagetab[it.flat(rd, min(tid, n))].z;
  a.row = rd.rowmap[it.score(rd, min(tid >> lg, n)) + min(tid & (T - 1), it.rows() - 1)];
}

template <int W>
__device__ __forceinline__ void put_group(const RoundDev& rd, const Item& it, const int T, GroupSharedSeg& sh, const AskedGroupSeg& a) {
  const int tid = threadIdx.x, n = it.count(), lg = T == 16 ? 4 : 5, which = (tid >> 5) & 1, q = tid & 31;
  const float4* tab = reinterpret_cast<const float4*>(rd.segtab);
  u32x4 pt = a.pt;
  for (int g = tid >> 6; g < n; g += W) {
    if (g >= W) pt = reinterpret_cast<const u32x4*>(rd.pagetab)[it.flat(rd, g)];
    reinterpret_cast<float4*>(sh.tab[g][which])[q] = tab[(size_t)(which ? pt[1] : pt[0]) * (kHalf / 2) + q];
  }
  int32_t row = a.row;
  for (int i = tid; i < n << lg; i += 64 * W) {
    if (i >= 64 * W) row = rd.rowmap[it.score(rd, i >> lg) + min(i & (T - 1), it.rows() - 1)];
    sh.row[i >> lg][i & (T - 1)] = row;            // (a row past the span repeats the last one; nobody uses it)
  }
  if (tid < n) sh.sel[tid] = (uint32_t)a.sel;
}

template <bool SEG> using Shared = std::conditional_t<SEG, GroupSharedSeg, GroupShared>;
template <bool SEG> using Asked = std::conditional_t<SEG, AskedGroupSeg, AskedGroup>;

// Where each page of each agent lies: a workgroup per agent, once per round.
__global__ __launch_bounds__(kBlock) void tdk_places_kernel(const RoundDev rd, PlaceDev* __restrict__ places) {
  const AgentDev ad = rd.agents[blockIdx.x];
  const int T = rd.page_tokens, lg = T == 16 ? 4 : 5, pages = rd.sess[ad.session].pages;
  for (int p = threadIdx.x; p < pages; p += kBlock) {
    const int a0 = ad.pos0 + p * T, lp = (a0 >> lg) - ad.lp_first;       // (positions are not negative)
    places[ad.flag_off + p] = PlaceDev{rd.bt[ad.bt_off + lp], lp + 1 < ad.bt_len ? rd.bt[ad.bt_off + lp + 1] : -1, a0 & (T - 1), 0};
  }
}

// lane geometry inside a row of H heads x 128 bf16 (= H*16 chunks of 16 bytes)
struct Lane {
  int klo, khi;      // chunk index of this lane's low-half / high-half K chunk
  int v0, v1;        // chunk indices of its two V chunks
  bool kok, v0ok, v1ok;
  int jb;            // which 8-element block of the half this lane rotates
  int rk, rv0, rv1;  // which of the rows that share an instruction the chunks belong to (0 unless PACK)
};

// Rows that share an instruction.  A row of H heads is 8 H lanes wide (K: two chunks per lane) or 16 H chunks (V: two
// per lane), so 8 / H rows fill a wavefront; the four wavefronts of a workgroup divide the page's rows among them,
// so a 16-token page gives a wavefront at most 4 rows.
__device__ __host__ __forceinline__ int rows_per_access(int H, int T) { const int n = 8 / H; return n < T / kWaves ? n : T / kWaves; }

// PACK: H is 1, 2 or 4
template <bool PACK>
__device__ __forceinline__ Lane lane_geometry(int H, int T) {
  const int lane = threadIdx.x & 63;
  Lane L;
  L.jb = lane & 7;
  L.rk = L.rv0 = L.rv1 = 0;
  if (!PACK) {
    L.klo = (lane >> 3) * 16 + L.jb;
    L.khi = L.klo + 8;
    L.kok = (lane >> 3) < H;
    L.v0 = lane;
    L.v1 = lane + 64;
    L.v0ok = L.v0 < H * 16;
    L.v1ok = L.v1 < H * 16;
  } else {
    const int n = rows_per_access(H, T), lgh = H == 4 ? 2 : H - 1;
    L.rk = (lane >> 3) >> lgh;
    L.klo = ((lane >> 3) & (H - 1)) * 16 + L.jb;
    L.khi = L.klo + 8;
    L.kok = L.rk < n;
    L.rv0 = lane >> (4 + lgh);
    L.rv1 = (lane + 64) >> (4 + lgh);
    L.v0 = lane & (16 * H - 1);
    L.v1 = lane & (16 * H - 1);
    L.v0ok = L.rv0 < n;
    L.v1ok = L.rv1 < n;
  }
  return L;
}

// The k-th group of rows of a wavefront: the first row of the page it covers.
template <bool PACK, int W = kWaves>
__device__ __forceinline__ int group_row(int k, int H, int T) {
  const int wave = threadIdx.x >> 6;
  return PACK ? (wave + kWaves * k) * rows_per_access(H, T) : wave + W * k;
}

__device__ __forceinline__ const float* tab_of(const GroupShared& sh, int g, int) { return sh.tab[g]; }
__device__ __forceinline__ const float* tab_of(const GroupSharedSeg& sh, int g, int r) {
  return sh.tab[g][(sh.sel[g] >> r) & 1u];
}

// cos/sin a lane needs for row r of agent g (r matters only with per-agent block layouts)
template <bool IL, class Shared>
__device__ __forceinline__ void load_tab(const Shared& sh, int g, int r, int jb, float (&c)[8], float (&s)[8]) {
  const float* t = tab_of(sh, g, r);
  if (!IL) {
#pragma unroll
    for (int e = 0; e < 8; ++e) { c[e] = t[jb * 8 + e]; s[e] = t[kHalf + jb * 8 + e]; }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      c[e] = t[jb * 4 + e];          s[e] = t[kHalf + jb * 4 + e];
      c[4 + e] = t[32 + jb * 4 + e]; s[4 + e] = t[kHalf + 32 + jb * 4 + e];
    }
  }
}

template <int RPW>
struct MasterRows {
  u32x4 kl[RPW], kh[RPW], v0[RPW], v1[RPW];
  bool  valid[RPW];                          // some row of the group lies inside the span
  bool  kin[RPW], v0in[RPW], v1in[RPW];      // PACK: the rows of this lane's chunks do
  template <bool PACK> __device__ __forceinline__ bool kok(const Lane& L, int k) const { return PACK ? L.kok && kin[k] : L.kok; }
  template <bool PACK> __device__ __forceinline__ bool v0ok(const Lane& L, int k) const { return PACK ? L.v0ok && v0in[k] : L.v0ok; }
  template <bool PACK> __device__ __forceinline__ bool v1ok(const Lane& L, int k) const { return PACK ? L.v1ok && v1in[k] : L.v1ok; }
};

// No branch stands around a load: a row or a chunk that does not exist reads another one of the page, and is not used.
template <int RPW, bool PACK, bool LOADV = true, bool LOADK = true>
__device__ __forceinline__ void load_master(const RoundDev& rd, const LayerDev& io, const Item& it, const int T,
                                            const Lane& L, MasterRows<RPW>& M) {
  constexpr int W = waves_of(RPW, PACK);
  const int rows = it.rows();
  const uint32_t row_u4 = (uint32_t)rd.heads * 16u;
  const u32x4* mk = io.master_k + it.d.row0 * row_u4;
  const u32x4* mv = io.master_v + it.d.row0 * row_u4;
  const uint32_t klo = L.kok ? L.klo : L.jb, v0 = L.v0ok ? L.v0 : 0, v1 = L.v1ok ? L.v1 : 0;
#pragma unroll
  for (int k = 0; k < RPW; ++k) {
    const int r = group_row<PACK, W>(k, rd.heads, T);
    M.valid[k] = r < rows;
    if (PACK) { M.kin[k] = r + L.rk < rows; M.v0in[k] = r + L.rv0 < rows; M.v1in[k] = r + L.rv1 < rows; }
    const u32x4 z = {0, 0, 0, 0};
    M.kl[k] = z; M.kh[k] = z; M.v0[k] = z; M.v1[k] = z;
    const uint32_t rk = min(PACK ? r + L.rk : r, rows - 1) * row_u4;
    if (LOADK) { M.kl[k] = mk[rk + klo]; M.kh[k] = mk[rk + klo + 8]; }
    if (LOADV) {
      M.v0[k] = mv[(PACK ? min(r + L.rv0, rows - 1) * row_u4 : rk) + v0];
      M.v1[k] = mv[(PACK ? min(r + L.rv1, rows - 1) * row_u4 : rk) + v1];
    }
  }
}

// Waits for the master page here.  Left to its first uses, the wait for the V rows stands in the loop over the agents, where the
// compiler does not see the streaming stores that count with the loads: every agent then waits for the stores of the one before.  Worth
// it for one access per page and wavefront (174 agents x 233 tokens, 1 head, restore 8.8 -> 7.4 us; 40 x 8000, 2 heads, collect 66.8 -> 66.2);
// with more of them that wait costs nothing or helps, as fewer pages are being written at a time (25 agents x 5000 tokens, restore 102.3
// against 100.5 us; ten sessions 0.998 times).
template <int RPW, bool V, bool K>
__device__ __forceinline__ void have_master(MasterRows<RPW>& M) {
#pragma unroll
  for (int k = 0; k < RPW; ++k) {
    if (K) asm volatile("" : "+v"(M.kl[k]), "+v"(M.kh[k]));
    if (V) asm volatile("" : "+v"(M.v0[k]), "+v"(M.v1[k]));
  }
}

// The compiler takes the K rows apart into fp32 in front of the loop over the agents, which costs 16 registers per row on top of the 8 that
// hold it: 128 with eight rows per wavefront, and the kernels of the master's order then need more than 256 (one wavefront per SIMD), the
// paired compare with own orders scratch.  KEEP: the rows are taken apart again for every agent.  8 heads, 32-token pages, 25 agents x 5000
// tokens: check layer 66.1 -> 61.9 us, store with own orders 121.5 -> 113.8; 100 agents x 5000, collect 388.5 -> 378.0; 16 x 850, collect,
// restore and store 64.1 -> 59.5.  Where two wavefronts per SIMD fit without it, it costs up to 1.3 % (own orders, collect of 100 x 5000
// 381.7 -> 386.9), but for the paired compare kernel with two accesses of several rows, where it is what makes the third fit: 4 heads, 16-token
// pages, store of 40 x 4000 69.8 -> 66.3 us, 200 x 1500 119.6 -> 117.9, 37 x 9000 133.0 -> 131.0 (launches with fewer than two items per
// place gain nothing: 64 x 700 25.7 -> 26.4); 2 heads, 32-token pages, 100 x 3000 67.7 -> 64.7.
template <bool KEEP>
__device__ __forceinline__ void keep_packed(u32x4& lo, u32x4& hi) {
  if (KEEP) asm("" : "+v"(lo), "+v"(hi));
}

// Where the rows of the master page lie for an agent of the group, read once per agent (a read of b0 or b1 behind every row's comparison, as
// a conditional expression on LDS compiles, makes every row wait for LDS twice).
struct Origin { longlong2 b; int32_t cut; };
__device__ __forceinline__ Origin origin_of(const GroupShared& sh, int g) { return Origin{sh.b[g], sh.cut[g]}; }
struct OriginSeg { const int32_t* row; };
__device__ __forceinline__ OriginSeg origin_of(const GroupSharedSeg& sh, int g) { return OriginSeg{sh.row[g]}; }

// byte of row r (0..T-1) of the page in a pool plane
__device__ __forceinline__ int64_t dest_row(const OriginSeg& o, uint32_t row_bytes, int r) { return (int64_t)o.row[r] * row_bytes; }
__device__ __forceinline__ int64_t dest_row(const Origin& o, uint32_t row_bytes, int r) { return (r < o.cut ? o.b.x : o.b.y) + (uint32_t)r * row_bytes; }

// where a row group's rows lie: one row for all lanes, or (PACK) each chunk's own
struct Dest { int64_t k, v0, v1; };
template <bool PACK, class O>
__device__ __forceinline__ Dest dest_of(const O& o, uint32_t row_bytes, int r, const Lane& L) {
  Dest d;
  d.k = dest_row(o, row_bytes, PACK ? r + L.rk : r);
  d.v0 = PACK ? dest_row(o, row_bytes, r + L.rv0) : d.k;
  d.v1 = PACK ? dest_row(o, row_bytes, r + L.rv1) : d.k;
  return d;
}
// chunk c of the row at that byte
template <class P> __device__ __forceinline__ P* chunk_at(P* pool, int64_t row, int c) {
  return reinterpret_cast<P*>(reinterpret_cast<std::conditional_t<std::is_const_v<P>, const char, char>*>(pool) + row) + c;
}

// ---------------------------------------------------------------------------------------------
// rerotate: pool_k <- bf16(R(delta_i) master_k), pool_v <- master_v       [Sec. 4.2]
// ---------------------------------------------------------------------------------------------

constexpr int kPrefetchBlocks = 1024;   // workgroups that take part in the master sweep (about one dispatch wave)

// The workgroups that start first sweep the masters once, in address order, before any of them
// writes: the reads then come from DRAM as one sequential stream into the memory-side cache instead
// of arriving one page at a time among the writes (a read among writes costs DRAM a bus turnaround;
// measured at about twice its byte share).
// Not in launches of at most three workgroups per compute unit, those that stand by for the tail and those that copy listed pages among them:
// nearly all their master reads stand before the writes anyway, and the sweep is a wait in front of them (4 agents x 256 tokens, collect,
// restore and store 24.0 -> 23.7 us).  Of the forms with eight wavefronts or 32-token pages only two fit a compute unit, but the line at two
// was no better for them: 691 workgroups of eight wavefronts, collect of 16 agents x 1536 tokens 21.8 us without the sweep and 22.8 with it,
// five heads 15.8 and 16.2, own orders 23.9 and 23.7, six restores 0.99 to 1.00; 32-token pages, six launches within 0.3 %.
template <bool LOOPING, int W>
__device__ __forceinline__ void sweep_masters(const RoundDev& rd, const LayerDev& io, bool k, bool v) {
  if (blockIdx.x >= kPrefetchBlocks || (!LOOPING && (int)gridDim.x <= 3 * rd.n_cus)) return;
  const size_t n16 = (size_t)rd.master_rows * rd.heads * 16;
  const unsigned nb = min((unsigned)gridDim.x, (unsigned)kPrefetchBlocks);
  u32x4 acc = {0, 0, 0, 0};
  for (size_t i = (size_t)blockIdx.x * (64 * W) + threadIdx.x; i < n16; i += (size_t)nb * (64 * W)) {
    if (k) acc ^= io.master_k[i];
    if (v) acc ^= io.master_v[i];
  }
  asm volatile("" : : "v"(acc));      // keeps the loads alive; the values are not used
}

// Optional timeline of a launch (measurement only): when the round carries a stamp buffer, the clock is
// recorded when a work item is taken up and when the last wavefront has issued its last access for it.
__device__ __forceinline__ int xcd_id() { return (int)(__builtin_amdgcn_s_getreg((3 << 11) | 20) & 7u); }   // XCC_ID, bits 3:0

__device__ __forceinline__ void stamp_begin(const RoundDev& rd, int item) {
  // (the low four bits carry the XCD the workgroup runs on)
  if (rd.stamps && threadIdx.x == 0) rd.stamps[4 * (size_t)item] = (wall_clock64() & ~15ull) | (unsigned)xcd_id();
}
__device__ __forceinline__ void stamp_end(const RoundDev& rd, int item) {
  if (rd.stamps && (threadIdx.x & 63) == 0) atomicMax(&rd.stamps[4 * (size_t)item + 1], (unsigned long long)wall_clock64());
}
// which = 2: the item's staging is in LDS; which = 3: the first wavefront has handled its rows of the first agent
__device__ __forceinline__ void stamp_mid(const RoundDev& rd, int item, int which) {
  if (rd.stamps && threadIdx.x == 0) rd.stamps[4 * (size_t)item + which] = wall_clock64();
}

// Which work items a workgroup processes.
//   Static: workgroup b owns item b, dispatched by the hardware round-robin over the XCDs.
//   Queued (TDK_TUNE_XCD_QUEUES, the kernels that write): the launch holds two workgroups per compute unit, and each
//   takes items until none is left: first from the queue of the XCD it runs on (the items that the static form
//   would have run there, so re-reads of a master page still meet in that XCD's L2), then from the other XCDs'
//   queues.  The XCDs do not write to memory at the same rate (measured: four of the eight finish a static
//   rerotate launch 15 % earlier and then idle); with queues the fast ones take over what the slow ones have left.
// Queue state in device memory: next[8], then the count of workgroups that have left the loop; the last one to
// leave puts everything back to zero, so every launch finds the state as the round's creation left it.
// Barrier for data exchanged through LDS only: waits for this wavefront's LDS traffic, not for its global stores
// (__syncthreads() would also wait until every store issued so far has been acknowledged by memory, which stalls
// a wavefront for microseconds at every item border while the chip is writing at full rate).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <bool queued>
struct Items {
  int home, k, ahead;
  __device__ __forceinline__ Items() : home(queued ? xcd_id() : 0), k(0), ahead(-1) {}

  // The first item of every workgroup is fixed by its number (workgroup b starts with entry b / 8 of queue b % 8, the
  // XCD the hardware places it on): no atomic stands between the launch and the first access, and the queues hand
  // out what lies behind those entries.
  __device__ __forceinline__ int reserved(int x) const { return ((int)gridDim.x - x + 7) >> 3; }   // workgroups b with b % 8 == x

  // thread 0 only: the next item for this workgroup, or -1 when every queue is empty
  __device__ __forceinline__ int fetch(const RoundDev& rd) {
    while (k < 8) {
      const int x = (home + k) & 7;
      const int n = rd.q_begin[x + 1] - rd.q_begin[x] - reserved(x);
      const int i = n > 0 ? atomicAdd(&rd.q_state[x], 1) : 0;
      if (i < n) return rd.q_begin[x] + reserved(x) + i;
      ++k;             // that queue is empty for good
    }
    return -1;
  }

  // Asks for the item after the current one (thread 0; an atomic whose answer is a round trip to memory among
  // the writes).  Called once per item, after the item's own loads have been issued: answers come back in issue
  // order, so a load issued behind the atomic would wait for it, while the stores of the data phase do not.
  __device__ __forceinline__ void prefetch(const RoundDev& rd) {
    if (queued) { if (threadIdx.x == 0) ahead = fetch(rd); }
  }

  // Hands the prefetched item to the whole workgroup.
  __device__ __forceinline__ int publish(int* s_item) {
    lds_barrier();     // every wavefront is through with the previous item: its staging in LDS may be replaced
    if (threadIdx.x == 0) *s_item = ahead;
    lds_barrier();
    return *s_item;
  }

  __device__ __forceinline__ int first(const RoundDev& rd, int* s_item) {
    if (!queued) {
      // Static launch: workgroup b owns item b, except for a shared tail (TDK_TUNE_SHARED_TAIL): the last items
      // go, in order, to whichever of the launch's last workgroups start first (there are twice as many of those
      // as items left, the late ones leave at once).  An XCD that writes faster gets through its share of the
      // workgroup ids sooner and so takes more of the tail, which evens out the end of a launch too short for
      // the looping form.  Every such workgroup does one atomic; the one that draws the last ticket puts the
      // counter back to zero.
      const int b = (int)blockIdx.x;
      if (b < rd.dyn_begin) return b;
      if (b >= rd.dyn_begin + rd.dyn_count) return -1;
      if (threadIdx.x == 0) {
        const int i = atomicAdd(&rd.q_state[12], 1);
        if (i == rd.dyn_count - 1) atomicExch(&rd.q_state[12], 0);
        *s_item = rd.dyn_begin + i < rd.n_work ? rd.dyn_begin + i : -1;
      }
      lds_barrier();
      return *s_item;
    }
    const int x = (int)blockIdx.x & 7, i = (int)blockIdx.x >> 3;
    return i < rd.q_begin[x + 1] - rd.q_begin[x] ? rd.q_begin[x] + i : -1;
  }
  __device__ __forceinline__ int next(const RoundDev& rd, int* s_item) {
    if (!queued) return -1;
    return publish(s_item);
  }
  __device__ __forceinline__ const ItemDev* list(const RoundDev& rd) const { return queued ? rd.qwork : rd.work; }
  __device__ __forceinline__ void leave(const RoundDev& rd) {
    if (queued) if (threadIdx.x == 0) {
      const int gone = atomicAdd(&rd.q_state[8], 1);
      if (gone == (int)gridDim.x - 1) {       // nobody takes items any more
#pragma unroll
        for (int x = 0; x < 8; ++x) atomicExch(&rd.q_state[x], 0);
        __threadfence();
        atomicExch(&rd.q_state[8], 0);
      }
    }
  }
};

template <int RPW, bool PACK, bool IL, bool NT, bool SEG, bool Q>
__global__ __launch_bounds__(64 * waves_of(RPW, PACK)) void tdk_rerotate_kernel(const RoundDev rd, const LayerDev io) {
  constexpr int W = waves_of(RPW, PACK);
  const int T = PACK ? rd.page_tokens : RPW * W;
  __shared__ Shared<SEG> sh;
  __shared__ int s_item;
  const Lane L = lane_geometry<PACK>(rd.heads, T);
  if (rd.nontemporal & 32) sweep_masters<Q, W>(rd, io, true, true);
  const uint32_t row_bytes = (uint32_t)rd.heads * (kHeadDim * 2);
  u32x4* pk = io.pool_k;
  u32x4* pv = io.pool_v;
  Items<Q> items;
  for (int item = items.first(rd, &s_item); item >= 0; item = items.next(rd, &s_item)) {
    stamp_begin(rd, item);
    const Item w(items.list(rd), item);
    Asked<SEG> asked;
    ask_group<W>(rd, w, T, sh, asked);
    MasterRows<RPW> M;
    load_master<RPW, PACK>(rd, io, w, T, L, M);
    put_group<W>(rd, w, T, sh, asked);
    if (RPW == 1) have_master<RPW, true, true>(M);
    lds_barrier();
    items.prefetch(rd);
    stamp_mid(rd, item, 2);
    for (int g = 0; g < w.count(); ++g) {
      if (g == 1) stamp_mid(rd, item, 3);
      float c[8], s[8];
      const auto from = origin_of(sh, g);
      if (!SEG) load_tab<IL>(sh, g, 0, L.jb, c, s);
#pragma unroll
      for (int k = 0; k < RPW; ++k) {
        if (!M.valid[k]) continue;
        const int r = group_row<PACK, W>(k, rd.heads, T);
        const Dest to = dest_of<PACK>(from, row_bytes, r, L);
        if (M.template kok<PACK>(L, k)) {
          if (SEG) load_tab<IL>(sh, g, PACK ? r + L.rk : r, L.jb, c, s);
          u32x4 olo, ohi;
          keep_packed<RPW == 8 && !SEG>(M.kl[k], M.kh[k]);
          rotate16<IL>(M.kl[k], M.kh[k], c, s, olo, ohi);
          st16<NT>(chunk_at(pk, to.k, L.klo), olo);
          st16<NT>(chunk_at(pk, to.k, L.khi), ohi);
        }
        if (M.template v0ok<PACK>(L, k)) st16<NT>(chunk_at(pv, to.v0, L.v0), M.v0[k]);
        if (M.template v1ok<PACK>(L, k)) st16<NT>(chunk_at(pv, to.v1, L.v1), M.v1[k]);
      }
    }
    stamp_end(rd, item);
  }
  items.leave(rd);
}

// ---------------------------------------------------------------------------------------------
// flag: per (agent, master page) compare against the re-rotated master     [Sec. 4.3]
// ---------------------------------------------------------------------------------------------

// differ <=> not (|a - ref| <= eps) in fp32; NaN on either side differs
__device__ __forceinline__ bool word_differs(uint32_t a, uint32_t r, float eps) {
  const bool lo = !(__builtin_fabsf(bf_lo(a) - bf_lo(r)) <= eps);
  const bool hi = !(__builtin_fabsf(bf_hi(a) - bf_hi(r)) <= eps);
  return lo | hi;
}

__device__ __forceinline__ bool chunk_differs(const u32x4 a, const u32x4 r, float eps) {
  bool d = false;
#pragma unroll
  for (int w = 0; w < 4; ++w) d |= word_differs(a[w], r[w], eps);
  return d;
}

__device__ __forceinline__ uint32_t chunk_xor(const u32x4 a, const u32x4 r) {
  const u32x4 x = a ^ r;
  return x[0] | x[1] | x[2] | x[3];
}

// Largest magnitude (as its 15 bits) in each half of the words of a chunk and of what came before.
__device__ __forceinline__ uint32_t chunk_largest(const u32x4 m, uint32_t so_far) {
  typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
  u16x2 v = __builtin_bit_cast(u16x2, so_far);
#pragma unroll
  for (int w = 0; w < 4; ++w) v = __builtin_elementwise_max(v, __builtin_bit_cast(u16x2, m[w] & 0x7fff7fffu));
  return __builtin_bit_cast(uint32_t, v);
}

// true if some bf16 of them is non-finite or so large (|x| >= 2^126) that a rotation could
// overflow: only then can a reference that is bit-identical to the agent's value still "differ"
// (|inf - inf| and NaN compare false), so such pages always take the full fp32 compare.  (Two packed instructions per word; with
// four comparisons per word and a verdict per row it was 1.4 of the 8.5 us that 4 agents x 256 tokens take; collect, restore and store 24.9 -> 24.0.)
__device__ __forceinline__ bool special_values(uint32_t largest) { return (largest & 0xffffu) >= 0x7e80u || largest >= 0x7e800000u; }

// PM: planes that take part (bit 0 = K, bit 1 = V); 3 is the paired diff, 1 / 2 the single-plane diffs
template <int RPW, bool PACK, bool IL, int PM, bool SEG, bool NTL>
__global__ __launch_bounds__(64 * waves_of(RPW, PACK)) void tdk_flag_kernel(const RoundDev rd, const LayerDev io, const float eps) {
  constexpr int W = waves_of(RPW, PACK);
  const int T = PACK ? rd.page_tokens : RPW * W;
  constexpr bool DOK = (PM & 1) != 0, DOV = (PM & 2) != 0;
  __shared__ Shared<SEG> sh;
  const Lane L = lane_geometry<PACK>(rd.heads, T);
  const uint32_t row_bytes = (uint32_t)rd.heads * (kHeadDim * 2);
  const u32x4* pk = io.pool_k;
  const u32x4* pv = io.pool_v;
  const int item = blockIdx.x;
  stamp_begin(rd, item);
  const Item w(rd.rwork, item);
  const int count = w.count();
  Asked<SEG> asked;
  ask_group<W>(rd, w, T, sh, asked);
  MasterRows<RPW> M;
  load_master<RPW, PACK, DOV, DOK>(rd, io, w, T, L, M);
  put_group<W>(rd, w, T, sh, asked);
  if ((int)threadIdx.x < count) sh.aux[threadIdx.x] = 0;
  lds_barrier();
  // Rolling requests (see tdk_keydiff_kernel): the rows of the next agent are asked for as the rows of this one
  // are used up; no branch stands around a load, a request with nothing to fetch reads the first row of the
  // master page and its result is ignored.
  const int64_t first_row = w.d.row0 * ((int64_t)rd.heads * 16);
  const u32x4* idle_k = DOK ? io.master_k + first_row + L.jb : nullptr;
  const u32x4* idle_v = DOV ? io.master_v + first_row + (threadIdx.x & 15) : nullptr;
  const u32x4 z = {0, 0, 0, 0};
  u32x4 akl[RPW], akh[RPW], av0[RPW], av1[RPW];
  auto request = [&](const auto& from, int g, int k) {
    const Dest at = dest_of<PACK>(from, row_bytes, group_row<PACK, W>(k, rd.heads, T), L);
    const bool ok = g < count && M.valid[k];
    akl[k] = z; akh[k] = z; av0[k] = z; av1[k] = z;
    if (DOK) {
      akl[k] = ld16<NTL>(ok && M.template kok<PACK>(L, k) ? chunk_at(pk, at.k, L.klo) : idle_k);
      akh[k] = ld16<NTL>(ok && M.template kok<PACK>(L, k) ? chunk_at(pk, at.k, L.khi) : idle_k + 8);
    }
    if (DOV) {
      av0[k] = ld16<NTL>(ok && M.template v0ok<PACK>(L, k) ? chunk_at(pv, at.v0, L.v0) : idle_v);
      av1[k] = ld16<NTL>(ok && M.template v1ok<PACK>(L, k) ? chunk_at(pv, at.v1, L.v1) : idle_v);
    }
  };
#pragma unroll
  for (int k = 0; k < RPW; ++k) { request(origin_of(sh, 0), 0, k); __builtin_amdgcn_sched_barrier(0); }   // in the order the loop uses them
  uint32_t largest = 0;
#pragma unroll
  for (int k = 0; k < RPW; ++k) {
    if (DOK) largest = chunk_largest(M.kh[k], chunk_largest(M.kl[k], largest));
    if (DOV) largest = chunk_largest(M.v1[k], chunk_largest(M.v0[k], largest));
  }
  const bool special = special_values(largest);
  for (int g = 0; g < count; ++g) {
    float c[8], s[8];
    const auto next = origin_of(sh, min(g + 1, count - 1));
    if (DOK && !SEG) load_tab<IL>(sh, g, 0, L.jb, c, s);
    bool differs = false;
#pragma unroll
    for (int k = 0; k < RPW; ++k) {
      if (M.valid[k]) {
        u32x4 rlo = z, rhi = z;
        if (DOK && SEG) load_tab<IL>(sh, g, group_row<PACK, W>(k, rd.heads, T) + (PACK ? L.rk : 0), L.jb, c, s);
        if (DOK) keep_packed<(RPW == 8 && (PM == 3 || !SEG)) || (RPW == 2 && PACK && PM == 3 && !SEG)>(M.kl[k], M.kh[k]);
        if (DOK) rotate16<IL>(M.kl[k], M.kh[k], c, s, rlo, rhi);
        // rows whose bits all match the reference (the common case) need no fp32 compare
        uint32_t x = 0;
        if (DOV) x |= (M.template v0ok<PACK>(L, k) ? chunk_xor(av0[k], M.v0[k]) : 0u) | (M.template v1ok<PACK>(L, k) ? chunk_xor(av1[k], M.v1[k]) : 0u);
        if (DOK) x |= M.template kok<PACK>(L, k) ? chunk_xor(akl[k], rlo) | chunk_xor(akh[k], rhi) : 0u;
        if (__any((int)(x != 0) | (int)special)) {
          if (DOK && M.template kok<PACK>(L, k)) {
            differs |= chunk_differs(akl[k], rlo, eps);
            differs |= chunk_differs(akh[k], rhi, eps);
          }
          if (DOV && M.template v0ok<PACK>(L, k)) differs |= chunk_differs(av0[k], M.v0[k], eps);
          if (DOV && M.template v1ok<PACK>(L, k)) differs |= chunk_differs(av1[k], M.v1[k], eps);
        }
      }
      request(next, g + 1, k);
    }
    if (__any(differs) && (threadIdx.x & 63) == 0) atomicOr(&sh.aux[g], 1);
  }
  lds_barrier();
  if ((int)threadIdx.x < count) rd.flags[w.flat(rd, threadIdx.x)] = (uint8_t)sh.aux[threadIdx.x];
  stamp_end(rd, item);
}

// ---------------------------------------------------------------------------------------------
// compaction: count, exclusive prefix, ascending index list                [Sec. 5]
// One launch.  A workgroup of 16 wavefronts takes 16 consecutive agents, one per wavefront: ballot over
// 64 page flags at a time, popcount, prefix by lane mask.  The flag bytes of all agents lie one after
// another in agent order, so the number of listed pages of all earlier agents (the exclusive prefix the
// offsets need) is the number of non-zero bytes before the workgroup's first agent: every workgroup
// counts that range itself with 16-byte loads (the flags of a round are a few hundred KB, L2-resident),
// and no workgroup waits for another.
// ---------------------------------------------------------------------------------------------

constexpr int kCompactBlock = 1024;
constexpr int kCompactWaves = kCompactBlock / 64;

__device__ __forceinline__ int nonzero_bytes(uint32_t w) {
  const uint32_t t = (((w & 0x7f7f7f7fu) + 0x7f7f7f7fu) | w) & 0x80808080u;
  return __popc(t);
}

__global__ __launch_bounds__(kCompactBlock) void tdk_compact_kernel(const RoundDev rd, const DiffDev d) {
  __shared__ int64_t s_part[kCompactWaves];
  __shared__ int32_t s_cnt[kCompactWaves];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (rd.n_agents == 0) {
    if (blockIdx.x == 0 && threadIdx.x == 0) { d.offset[0] = 0; d.overflow[0] = 0; }
    return;
  }
  const int a0 = blockIdx.x * kCompactWaves;
  const int a = a0 + wave;
  // listed pages of all agents before a0: non-zero bytes of flags[0, flag_off(a0))
  const int64_t n_before = rd.agents[a0].flag_off;
  const uint8_t* fl = rd.flags;
  int64_t part = 0;
  const int64_t n16 = n_before >> 4;
  for (int64_t i = threadIdx.x; i < n16; i += kCompactBlock) {
    const u32x4 w = reinterpret_cast<const u32x4*>(fl)[i];
    part += nonzero_bytes(w[0]) + nonzero_bytes(w[1]) + nonzero_bytes(w[2]) + nonzero_bytes(w[3]);
  }
  for (int64_t i = (n16 << 4) + threadIdx.x; i < n_before; i += kCompactBlock) part += fl[i] != 0;
#pragma unroll
  for (int sft = 32; sft > 0; sft >>= 1) part += __shfl_xor(part, sft);
  // this wavefront's agent: its count
  int n = 0;
  int P = 0, flag_off = 0;
  if (a < rd.n_agents) {
    const AgentDev ad = rd.agents[a];
    P = rd.sess[ad.session].pages;
    flag_off = ad.flag_off;
    for (int p0 = 0; p0 < P; p0 += 64) {
      const int p = p0 + lane;
      const bool f = p < P && fl[flag_off + p] != 0;
      n += __popcll(__ballot(f));
    }
  }
  if (lane == 0) { s_part[wave] = part; s_cnt[wave] = n; }
  __syncthreads();
  int64_t base = 0;
#pragma unroll
  for (int q = 0; q < kCompactWaves; ++q) { base += s_part[q]; if (q < wave) base += s_cnt[q]; }
  if (a >= rd.n_agents) return;
  if (lane == 0) {
    d.count[a] = n;
    d.offset[a] = base;
    if (a == rd.n_agents - 1) {
      const int64_t total = base + n;
      d.offset[a + 1] = total;
      d.overflow[0] = total > d.capacity ? 1 : 0;
    }
  }
  int64_t run = base;
  for (int p0 = 0; p0 < P; p0 += 64) {
    const int p = p0 + lane;
    const bool f = p < P && fl[flag_off + p] != 0;
    const uint64_t b = __ballot(f);
    const int rank = __popcll(b & ((1ull << lane) - 1ull));
    if (f && run + rank < d.capacity) d.idx[run + rank] = p;
    run += __popcll(b);
  }
}

// ---------------------------------------------------------------------------------------------
// gather: K/V values of the listed pages, as they sit in the agent's cache   [Sec. 5]
// A workgroup copies one payload slot (the selected planes back to back); grid-stride over the slots that
// exist, so the host never needs the count.
// ---------------------------------------------------------------------------------------------

// Shared by gather and scatter.  Prologue: all threads search offset[] in parallel for the agent that owns the slot
// (one memory round trip per 256 agents instead of a serial binary search), then T threads resolve the pool
// row of each row of the page through the block table.
struct SlotShared {
  int32_t owner, page;
  int64_t row[32];     // pool row of each row of the page, -1 past the span / not listed
};

template <int W = kWaves>
__device__ __forceinline__ void find_owner(const DiffDev& d, int A, int64_t slot, SlotShared& sh) {
  for (int a = threadIdx.x; a < A; a += 64 * W)
    if (d.offset[a] <= slot && slot < d.offset[a + 1]) sh.owner = a;
}

// pool row of master token page * T + r for an agent, -1 past the span
__device__ __forceinline__ int64_t slot_row(const RoundDev& rd, const AgentDev& ad, int page, int r) {
  const int T = rd.page_tokens, m = page * T + r;
  if (m >= rd.sess[ad.session].span) return -1;
  if (rd.seg) return (int64_t)rd.rowmap[ad.score_off + m];
  const int a0 = ad.pos0 + m;
  return (int64_t)rd.bt[ad.bt_off + (T == 16 ? a0 >> 4 : a0 >> 5) - ad.lp_first] * T + (a0 & (T - 1));
}

// 16-byte accesses per thread in flight in gather / scatter: a K and a V page are 16 accesses per thread, so a slot is
// two round trips to memory (with 4 in flight, and a branch around each, it was four: payload copies of 64 agents x 12800
// tokens with a tenth of the pages listed 141 -> 137 us, with streamed reads; 48 agents with moved mirrors and
// their own block orders, whose K rows are turned four at a time now instead of one, 148 -> 124 us).
constexpr int kCopyBatch = 8;

// Planes p0 .. p1 - 1 (0 = K, 1 = V) of one slot between pool and payload; slot_data: the payload of plane p0.  A row past
// the span (row < 0) is zero in the payload and not written in the pool.  No branch stands around a load: a load with
// nothing to fetch repeats one of its page.  NT: streaming stores; NTL: non-temporal loads.  (The gather streams both:
// with caches that change from call to call a store of 180 agents x 2166 tokens, one page in ten listed, took 277 us with
// ordinary loads and 263 streamed; 30 agents x 2000, one in five, 69 and 70.)  share: this workgroup's part of the slot, of 1 << lg_shares.
template <bool TO_PAYLOAD, bool NT, bool NTL, int W = kWaves>
__device__ __forceinline__ void copy_slot(const RoundDev& rd, const LayerDev& io, u32x4* slot_data, int p0, int p1, const SlotShared& sh,
                                          int share = 0, int lg_shares = 0) {
  const int row_u4 = rd.heads * 16, page_u4 = rd.page_tokens * row_u4, all = (p1 - p0) * page_u4;
  const int n = (all * (share + 1)) >> lg_shares;
  const uint32_t inv = 0xffffffffu / (uint32_t)row_u4 + 1u;      // i / row_u4 == __umulhi(i, inv) for i < 2^13 (row_u4 <= 128)
  for (int i0 = ((all * share) >> lg_shares) + threadIdx.x; i0 < n; i0 += 64 * W * kCopyBatch) {
    u32x4 v[kCopyBatch];
    u32x4* at[kCopyBatch];
    bool there[kCopyBatch];
#pragma unroll
    for (int j = 0; j < kCopyBatch; ++j) {
      const int i = min(i0 + j * (64 * W), n - 1);
      const int plane = p0 + (i >= page_u4), q = i >= page_u4 ? i - page_u4 : i;
      const int r = (int)__umulhi((uint32_t)q, inv);
      const int64_t row = sh.row[r];
      there[j] = row >= 0;
      at[j] = (plane ? io.pool_v : io.pool_k) + (row >= 0 ? row : max(sh.row[0], (int64_t)0)) * row_u4 + (q - r * row_u4);
      v[j] = ld16<NTL>(TO_PAYLOAD ? at[j] : slot_data + i);
    }
#pragma unroll
    for (int j = 0; j < kCopyBatch; ++j) {
      const int i = i0 + j * (64 * W);
      if (TO_PAYLOAD) {
        if (!there[j]) v[j] = u32x4{0, 0, 0, 0};
        if (i < n) st16<NT>(slot_data + i, v[j]);
      } else {
        if (i < n && there[j]) st16<NT>(at[j], v[j]);
      }
    }
  }
}

// batches of accesses in a slot (copy_slot)
__device__ __host__ __forceinline__ int slot_batches(const RoundDev& rd, int planes, int waves = kWaves) {
  return (planes == 3 ? 2 : 1) * rd.page_tokens * rd.heads * 16 / (64 * waves * kCopyBatch);
}

// does a restore share its slots out? (scatter_slots)
__device__ __host__ __forceinline__ bool slots_shared(const RoundDev& rd) { return !rd.diff_moved; }

// planes: bit 0 = K, bit 1 = V; a slot holds the selected planes back to back
__device__ __forceinline__ void gather_slot(const RoundDev& rd, const LayerDev& io, const DiffDev& d, const int planes, int64_t slot,
                                            const SlotShared& sh, int share = 0, int lg_shares = 0) {
  const int p0 = planes == 2 ? 1 : 0, p1 = planes == 1 ? 1 : 2;
  u32x4* data = d.payload + slot * (p1 - p0) * (int64_t)(rd.page_tokens * rd.heads * 16);
  if (rd.nontemporal & 16) copy_slot<true, true, true>(rd, io, data, p0, p1, sh, share, lg_shares);
  else copy_slot<true, false, false>(rd, io, data, p0, p1, sh, share, lg_shares);
}

__global__ __launch_bounds__(kBlock) void tdk_gather_kernel(const RoundDev rd, const LayerDev io, const DiffDev d,
                                                            const int planes) {
  __shared__ SlotShared sh;
  const int A = rd.n_agents;
  if (A == 0) return;
  int64_t total = d.offset[A];
  if (total > d.capacity) total = d.capacity;
  for (int64_t slot = blockIdx.x; slot < total; slot += gridDim.x) {
    find_owner(d, A, slot, sh);
    __syncthreads();
    if (threadIdx.x < rd.page_tokens) sh.row[threadIdx.x] = slot_row(rd, rd.agents[sh.owner], d.idx[slot], threadIdx.x);
    __syncthreads();
    gather_slot(rd, io, d, planes, slot, sh);
    __syncthreads();
  }
}

// Compaction and gather in one launch, for rounds with at most kListPages (agent, page) pairs: a workgroup needs neither
// the counts nor the index list of another, because it finds the page of its slot in the flag bytes itself (64 bytes
// per thread at most, one round trip, L2-resident).  What it saves is a launch of a few workgroups between two
// larger ones and half of the gather's chain of dependent reads (4 agents x 256 tokens: 3.5 + 9.8 -> 8.2 us, the whole
// collect, restore and store 36 -> 28; 37 agents, one plane: 4.8 + 9.0 -> 11.3 us); with more flags the count that every
// workgroup repeats costs more than the launch.  The workgroups that own a slot write its index, workgroup 0
// the counts and offsets.
constexpr int kListPages = 64 * kBlock;

// non-zero bytes among the first `lim` of 16, and the same as a mask word by word (bit 7 of each such byte)
__device__ __forceinline__ uint32_t set_bytes(uint32_t w, int lim) {
  const uint32_t t = (((w & 0x7f7f7f7fu) + 0x7f7f7f7fu) | w) & 0x80808080u;
  return lim >= 4 ? t : lim <= 0 ? 0u : t & ((1u << (8 * lim)) - 1u);
}
__device__ __forceinline__ int count_set(const u32x4 w, int lim) {
  return __popc(set_bytes(w[0], lim)) + __popc(set_bytes(w[1], lim - 4)) + __popc(set_bytes(w[2], lim - 8)) + __popc(set_bytes(w[3], lim - 12));
}

__global__ __launch_bounds__(kBlock) void tdk_list_gather_kernel(const RoundDev rd, const LayerDev io, const DiffDev d, const int planes) {
  __shared__ SlotShared sh;
  __shared__ int s_wave[kWaves], s_before[kBlock], s_flat;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, A = rd.n_agents;
  const int n = (int)rd.agent_pages;                          // at most kListPages
  const int per = ((n + 16 * kBlock - 1) / (16 * kBlock)) * 16;        // consecutive flag bytes per thread: 0, 16, 32, 48 or 64
  u32x4 w[4];
  int own = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int at = tid * per + 16 * q;
    w[q] = u32x4{0, 0, 0, 0};
    if (16 * q < per && at < n) w[q] = *reinterpret_cast<const u32x4*>(rd.flags + at);
    own += count_set(w[q], n - at);
  }
  int inc = own;
#pragma unroll
  for (int sft = 1; sft < 64; sft <<= 1) {
    const int v = __shfl_up(inc, sft);
    if (lane >= sft) inc += v;
  }
  if (lane == 63) s_wave[wave] = inc;
  __syncthreads();
  int before = inc - own, total = 0;
#pragma unroll
  for (int q = 0; q < kWaves; ++q) { if (q < wave) before += s_wave[q]; total += s_wave[q]; }
  if (blockIdx.x == 0) {
    s_before[tid] = before;
    __syncthreads();
    // listed pages of all agents before the flat page index `at`
    auto listed_before = [&](int at) {
      if (at >= n) return total;
      const int t = at / per;
      int c = s_before[t];
      for (int q = t * per; q < at; q += 16) c += count_set(*reinterpret_cast<const u32x4*>(rd.flags + q), at - q);
      return c;
    };
    for (int a = tid; a < A; a += kBlock) {
      const AgentDev ad = rd.agents[a];
      const int lo = listed_before(ad.flag_off), hi = listed_before(ad.flag_off + rd.sess[ad.session].pages);
      d.count[a] = hi - lo;
      d.offset[a] = lo;
    }
    if (tid == 0) { d.offset[A] = total; d.overflow[0] = total > d.capacity ? 1 : 0; }
  }
  const int slots = (int)min((int64_t)total, d.capacity);
  // Few slots are shared out further, down to one batch of accesses per thread: a workgroup's batches are round trips to memory one
  // after the other (4 agents x 256 tokens, the whole collect, restore and store 27.3 -> 25.5 us).
  int lg_shares = 0;
  while ((2 << lg_shares) <= slot_batches(rd, planes) && (int64_t)slots << (lg_shares + 1) <= gridDim.x) ++lg_shares;
  for (int unit = blockIdx.x; unit < slots << lg_shares; unit += gridDim.x) {
    const int slot = unit >> lg_shares, share = unit & ((1 << lg_shares) - 1);
    // the slot-th listed page: one thread holds its flag
    if (slot >= before && slot < before + own) {
      int k = slot - before, found = -1;
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          uint32_t t = set_bytes(w[q][j], n - (tid * per + 16 * q + 4 * j));
          const int c = __popc(t);
          if (found < 0 && k < c) {
            for (; k > 0; --k) t &= t - 1u;
            found = tid * per + 16 * q + 4 * j + ((__ffs((int)t) - 1) >> 3);
          }
          if (found < 0) k -= c;
        }
      s_flat = found;
    }
    __syncthreads();
    const int flat = s_flat;
    for (int a = tid; a < A; a += kBlock) {
      const AgentDev ad = rd.agents[a];
      if (flat >= ad.flag_off && flat < ad.flag_off + rd.sess[ad.session].pages) { sh.owner = a; sh.page = flat - ad.flag_off; }
    }
    __syncthreads();
    if (tid < rd.page_tokens) sh.row[tid] = slot_row(rd, rd.agents[sh.owner], sh.page, tid);
    if (tid == 0 && share == 0) d.idx[slot] = sh.page;
    __syncthreads();
    gather_slot(rd, io, d, planes, slot, sh, share, lg_shares);
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------------------------
// decode: diff pages from the payload, all others from the re-rotated master   [Sec. 4.4, Alg. 1]
// ---------------------------------------------------------------------------------------------

// The "correct" half of skip-or-correct: pages listed in a diff are copied from the payload to the
// agent's rows (the mirror image of the gather kernel).  Every pool row is written exactly once by
// either this kernel or the page kernel above, so their order does not matter.
struct ScatterShared {
  SlotShared sh;
  float s_tab[2][2 * kHalf];    // cos/sin of the payload re-rotation: up to two segments meet a page
  uint32_t s_sel, s_moved;      // bit r of s_sel: row r uses table 1; bit t of s_moved: table t is not the identity
};

// Workgroup `first` of `stride` workgroups: walks the payload slots first, first + stride, ...
template <bool IL, int W = kWaves>
__device__ __forceinline__ void scatter_slots(const RoundDev& rd, const LayerDev& io, const DiffDev& d, const int planes,
                                              ScatterShared& ss, const int64_t first, const int64_t stride) {
  SlotShared& sh = ss.sh;
  float (&s_tab)[2][2 * kHalf] = ss.s_tab;
  uint32_t& s_sel = ss.s_sel;
  uint32_t& s_moved = ss.s_moved;
  constexpr int kRows = 4 * kWaves / W;            // rows of a wavefront in flight: 16 of the workgroup, which divide the page
  const int T = rd.page_tokens;
  const int A = rd.n_agents;
  if (A == 0) return;
  int64_t total = d.offset[A];
  if (total > d.capacity) total = d.capacity;
  const int row_u4 = rd.heads * 16;
  const int page_u4 = T * row_u4;
  const Lane L = lane_geometry<false>(rd.heads, T);
  // Payload reads are streamed where the call's inputs are too many to be found in the 256 MB memory-side cache by the time
  // they are read: there ordinary reads find nothing and push the masters out, which are read more than once.  What the call
  // leaves in that cache is counted: payload and masters, and for moved diffs the K rows once more, whose stores are
  // ordinary ones.  Measured with inputs that change from call to call, ordinary -> streamed: 20, 41, 61 MB 43.6 -> 48.6,
  // 82.4 -> 88.0, 121 -> 127 us; 73 MB 150 -> 155; 84 MB 125 -> 122; 92 MB 96.7 -> 101; 94 MB 297 -> 282; 102 MB 218 -> 209;
  // 133 MB 155 -> 146; 184 MB 205 -> 193; 306 MB 293 -> 266; moved diffs 55 MB 70.4 -> 74.8, 75 MB 91.3 -> 93.4, 83 MB
  // 110 -> 105 and 107 -> 102.  (One set of inputs over and over stays with ordinary reads up to 256 MB: 180 MB 634 us, streamed
  // 650.)  A call on one plane counts both: a program restores them in turn.
  const int64_t u4s = total * page_u4 * (rd.diff_moved ? 3 : 2) + rd.master_rows * row_u4 * 2;
  const bool stream = (rd.nontemporal & 8) && u4s * 16 > (int64_t)80 << 20;
  // Few slots are shared out further (see tdk_list_gather_kernel), but for K rows that are turned: 4 agents x 256 tokens, the whole
  // collect, restore and store 25.5 -> 25.1 us, restore of 4 x 8 agents x 2306 tokens 66.0 -> 64.8.  (With divisions in place of
  // the shifts small calls on one plane lost 1 to 3 %.)
  int lg_shares = 0;
  if (slots_shared(rd))
    while ((2 << lg_shares) <= slot_batches(rd, planes, W) && total << (lg_shares + 1) <= stride) ++lg_shares;
  for (int64_t unit = first; unit < total << lg_shares; unit += stride) {
    const int64_t slot = unit >> lg_shares;
    const int share = (int)unit & ((1 << lg_shares) - 1);
    if (threadIdx.x == 0) sh.owner = -1;
    __syncthreads();
    find_owner<W>(d, A, slot, sh);
    __syncthreads();
    bool rot = false;
    int t0 = 0, t1 = 0;
    const float* tabs = rd.tab_diff;
    if (sh.owner >= 0 && rd.agents[sh.owner].diff_rot != 0) {
      // which stored-frame -> current-frame rotations this page needs
      const AgentDev ad = rd.agents[sh.owner];
      const int p = d.idx[slot];
      uint32_t sel = 0, moved = 1;
      t0 = t1 = sh.owner;
      if (rd.seg) {
        moved = 0;
        if (p >= 0 && p < rd.sess[ad.session].pages) {
          const PageTab pt = rd.pagetab[ad.flag_off + p];
          t0 = pt.x; t1 = pt.y; sel = (uint32_t)pt.z; moved = (uint32_t)pt.w;
          tabs = rd.segtab_diff;
        }
      }
      rot = moved != 0;
      if (threadIdx.x == 0) { s_sel = sel; s_moved = moved; }
    }
    if (threadIdx.x < T) {
      int64_t row = -1;
      if (sh.owner >= 0) {                       // an inconsistent offset[] leaves the slot unowned
        const AgentDev ad = rd.agents[sh.owner];
        const int p = d.idx[slot];
        if (p >= 0 && p < rd.sess[ad.session].pages) row = slot_row(rd, ad, p, threadIdx.x);   // anything else is not an index this round produces
      }
      sh.row[threadIdx.x] = row;
    }
    if (rot && threadIdx.x < 4 * kHalf) {
      const int which = threadIdx.x >> 7, e = threadIdx.x & (2 * kHalf - 1);
      s_tab[which][e] = tabs[(size_t)(which ? t1 : t0) * (2 * kHalf) + e];
    }
    __syncthreads();
    int p0 = planes == 2 ? 1 : 0;
    const int p1 = planes == 1 ? 1 : 2;
    u32x4* data = d.payload + slot * (p1 - p0) * (int64_t)page_u4;
    if (p0 == 0 && rot) {
      // stored at another position: K rows are re-rotated, a wavefront per row, both members of a pair in one lane
      // (the page kernels' lane layout); four rows of the wavefront (two where it is one of eight) are requested before the first is used
      for (int r0 = threadIdx.x >> 6; r0 < T; r0 += kRows * W) {
        u32x4 lo[kRows], hi[kRows];
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
          const u32x4* src = data + (r0 + W * k) * row_u4;          // (T is a multiple of 16)
          lo[k] = src[L.kok ? L.klo : 0];
          hi[k] = src[L.kok ? L.khi : 0];
        }
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
          const int r = r0 + W * k;
          const int64_t row = sh.row[r];
          const int which = (s_sel >> r) & 1u;
          if ((s_moved >> which) & 1u) {           // a run that did not move is a bit copy
            const float* t = s_tab[which];
            float c[8], sn[8];
            if (!IL) {
#pragma unroll
              for (int e = 0; e < 8; ++e) { c[e] = t[L.jb * 8 + e]; sn[e] = t[kHalf + L.jb * 8 + e]; }
            } else {
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                c[e] = t[L.jb * 4 + e];          sn[e] = t[kHalf + L.jb * 4 + e];
                c[4 + e] = t[32 + L.jb * 4 + e]; sn[4 + e] = t[kHalf + 32 + L.jb * 4 + e];
              }
            }
            rotate16<IL>(lo[k], hi[k], c, sn, lo[k], hi[k]);
          }
          if (row >= 0 && L.kok) {
            io.pool_k[row * row_u4 + L.klo] = lo[k];
            io.pool_k[row * row_u4 + L.khi] = hi[k];
          }
        }
      }
      p0 = 1;
      data += page_u4;
    }
    if (p0 < p1) {
      if (stream) copy_slot<false, true, true, W>(rd, io, data, p0, p1, sh, share, lg_shares);
      else if (rd.nontemporal & 8) copy_slot<false, true, false, W>(rd, io, data, p0, p1, sh, share, lg_shares);
      else copy_slot<false, false, false, W>(rd, io, data, p0, p1, sh, share, lg_shares);
    }
    __syncthreads();
  }
}

template <bool IL>
__global__ __launch_bounds__(kBlock) void tdk_scatter_kernel(const RoundDev rd, const LayerDev io, const DiffDev d,
                                                             const int planes) {
  __shared__ ScatterShared ss;
  scatter_slots<IL>(rd, io, d, planes, ss, blockIdx.x, gridDim.x);
}

// Skip-or-correct decision of a work item: listed[g] = 1 where the item's page is in the index list of agent g of its group.
// All threads of the workgroup take part, 64 lanes per agent in groups of up to four, 32 in groups of up to eight and so on:
// each round of reads divides what is left of a list by that number.  One agent per thread halves it, and every read is a memory
// latency in front of the item's first store: 37 agents x 2999 tokens, 4 heads, one plane after the other 127.5 -> 125.6 us,
// 4 x 12 agents x 3001 tokens with moved diffs and own orders 104.2 -> 101.9, 13 agents x 19322 tokens, 4 heads 292 -> 275.
__device__ __forceinline__ void find_listed(const RoundDev& rd, const DiffDev& d, const Item& w, int32_t* listed) {
  const int count = w.count(), page = w.d.page, lg = count <= 4 ? 6 : count <= 8 ? 5 : count <= 16 ? 4 : 3;      // (four wavefronts reach kMaxGroup agents; of eight the rest has none)
  const int g = threadIdx.x >> lg, lanes = 1 << lg, l = threadIdx.x & (lanes - 1), shift = threadIdx.x & 63 & ~(lanes - 1);
  const uint64_t mine = (lanes == 64 ? ~0ull : (1ull << lanes) - 1ull) << shift;
  const int32_t* v = d.idx;
  int n = 0;
  if (g < count) {
    const int a = w.agent(rd, g);
    int64_t lo = d.offset[a];
    int64_t hi = lo + d.count[a];
    if (lo < 0) lo = 0;
    if (hi > d.capacity) hi = d.capacity;
    v += lo;
    n = hi > lo ? (int)min<int64_t>(hi - lo, 1 << 30) : 0;
  }
  bool found = false;
  while (__any(n > 0)) {
    const int stride = (n + lanes - 1) >> lg, i = l * stride;
    const int x = i < n ? v[i] : 0x7fffffff;
    const uint64_t below = __ballot(x < page) & mine;
    found |= (__ballot(x == page) & mine) != 0;
    const int c = __popcll(below), skip = c ? (c - 1) * stride + 1 : n;
    v += skip;
    n = found ? 0 : max(min(stride - 1, n - skip), 0);
  }
  if (l == 0 && g < count) listed[g] = found;
}

template <int RPW, bool PACK, bool IL, bool NT, int PM, bool SEG, bool Q>
__global__ __launch_bounds__(64 * waves_of(RPW, PACK)) void tdk_decode_kernel(const RoundDev rd, const LayerDev io, const DiffDev d,
                                                            const int n_scatter) {
  constexpr int W = waves_of(RPW, PACK);
  const int T = PACK ? rd.page_tokens : RPW * W;
  __shared__ Shared<SEG> sh;
  __shared__ int s_item;
  constexpr bool DOK = (PM & 1) != 0, DOV = (PM & 2) != 0;
  if (!Q && (int)blockIdx.x >= rd.dyn_begin + rd.dyn_count) {
    // Small rounds only (static launches that do not fill the chip for long): the workgroups that copy the listed
    // pages from the payload ride behind the page items of the same launch, n_scatter of them, and run while the
    // page items drain, instead of paying for a launch of their own.  (On large rounds two launches are faster:
    // payload reads among the page items' writes cost more than the second launch.)
    __shared__ ScatterShared ss;
    scatter_slots<IL, W>(rd, io, d, PM, ss, (int64_t)blockIdx.x - (rd.dyn_begin + rd.dyn_count), n_scatter);
    return;
  }
  const Lane L = lane_geometry<PACK>(rd.heads, T);
  if (rd.nontemporal & 64) sweep_masters<Q, W>(rd, io, DOK, DOV);
  const uint32_t row_bytes = (uint32_t)rd.heads * (kHeadDim * 2);
  u32x4* pk = io.pool_k;
  u32x4* pv = io.pool_v;
  Items<Q> items;
  for (int item = items.first(rd, &s_item); item >= 0; item = items.next(rd, &s_item)) {
    stamp_begin(rd, item);
    const Item w(items.list(rd), item);
    Asked<SEG> asked;
    ask_group<W>(rd, w, T, sh, asked);
    MasterRows<RPW> M;
    load_master<RPW, PACK, DOV, DOK>(rd, io, w, T, L, M);
    find_listed(rd, d, w, sh.aux);
    put_group<W>(rd, w, T, sh, asked);
    if (RPW == 1) have_master<RPW, DOV, DOK>(M);
    lds_barrier();
    items.prefetch(rd);
    for (int g = 0; g < w.count(); ++g) {
      if (sh.aux[g] != 0) continue;   // listed in the diff: the scatter kernel writes this page
      float c[8], s[8];
      const auto from = origin_of(sh, g);
      if (DOK && !SEG) load_tab<IL>(sh, g, 0, L.jb, c, s);
#pragma unroll
      for (int k = 0; k < RPW; ++k) {
        if (!M.valid[k]) continue;
        const int r = group_row<PACK, W>(k, rd.heads, T);
        const Dest to = dest_of<PACK>(from, row_bytes, r, L);
        if (DOK && M.template kok<PACK>(L, k)) {
          if (SEG) load_tab<IL>(sh, g, PACK ? r + L.rk : r, L.jb, c, s);
          u32x4 olo, ohi;
          keep_packed<RPW == 8 && !SEG>(M.kl[k], M.kh[k]);
          rotate16<IL>(M.kl[k], M.kh[k], c, s, olo, ohi);
          st16<NT>(chunk_at(pk, to.k, L.klo), olo);
          st16<NT>(chunk_at(pk, to.k, L.khi), ohi);
        }
        if (DOV && M.template v0ok<PACK>(L, k)) st16<NT>(chunk_at(pv, to.v0, L.v0), M.v0[k]);
        if (DOV && M.template v1ok<PACK>(L, k)) st16<NT>(chunk_at(pv, to.v1, L.v1), M.v1[k]);
      }
    }
    stamp_end(rd, item);
  }
  items.leave(rd);
}

// ---------------------------------------------------------------------------------------------
// plain copy / fill (bandwidth ceiling and traffic-counter reference)
// ---------------------------------------------------------------------------------------------

// Plain copy with the streaming policy on both sides (the fastest copy measured on this chip).
__global__ __launch_bounds__(kBlock) void tdk_copy_kernel(u32x4* __restrict__ dst, const u32x4* __restrict__ src, size_t n) {
  for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (size_t)gridDim.x * kBlock)
    st16<true>(dst + i, ld16<true>(src + i));
}

__global__ __launch_bounds__(kBlock) void tdk_fill_kernel(u32x4* __restrict__ dst, uint32_t word, size_t n) {
  const u32x4 v = {word, word, word, word};
  for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (size_t)gridDim.x * kBlock) dst[i] = v;
}

// ---------------------------------------------------------------------------------------------
// check layer: batched key-difference pass, important positions, master choice   [Sec. 4.2]
// ---------------------------------------------------------------------------------------------

// Sum of v over the `width` lanes of a row (64; or 8, 16, 32 with several rows per wavefront) with DPP row shifts and
// row broadcasts (no LDS traffic); the total is valid in the last lane of each row only.
__device__ __forceinline__ float row_sum_to_last_lane(float v, int width) {
  auto dpp = [](float x, auto ctrl, auto row_mask) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value,
                                                                   decltype(row_mask)::value, 0xf, false));
  };
  v += dpp(v, std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xf>{});   // row_shr:1
  v += dpp(v, std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xf>{});   // row_shr:2
  v += dpp(v, std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xf>{});   // row_shr:4
  if (width > 8) v += dpp(v, std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xf>{});   // row_shr:8 -> lane 15 of each row
  if (width > 16) v += dpp(v, std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});   // row_bcast:15 into rows 1, 3
  if (width > 32) v += dpp(v, std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});   // row_bcast:31 into rows 2, 3
  return v;
}

// Per (agent, token): sum over the row of (fresh K - rotated cached K)^2, fp32.  Same traversal as
// the compare kernel, K plane only.  Twice the arithmetic per byte of the compare kernel and only half a
// page per agent in flight, so the loads of one agent must overlap the arithmetic of the one before: see the
// rolling requests below (482 -> 415 us on 250 agents x 5000 tokens; at a budget of 128 registers the compiler
// spills, and a reload from scratch waits for every load issued before it, so the kernel runs at 3 waves per SIMD).
template <int RPW, bool PACK, bool IL, bool SEG, bool NTL>
__global__ __launch_bounds__(64 * waves_of(RPW, PACK)) __attribute__((amdgpu_waves_per_eu(RPW <= 4 ? 3 : 1))) void tdk_keydiff_kernel(const RoundDev rd, const LayerDev io, const PlanDev pl) {
  constexpr int W = waves_of(RPW, PACK);
  const int T = PACK ? rd.page_tokens : RPW * W;
  __shared__ Shared<SEG> sh;
  __shared__ float s_score[kMaxGroup][PACK ? 32 : RPW * waves_of(RPW, PACK)];
  const Lane L = lane_geometry<PACK>(rd.heads, T);
  const uint32_t row_bytes = (uint32_t)rd.heads * (kHeadDim * 2);
  const u32x4* pk = io.pool_k;
  const Item w(rd.rwork, blockIdx.x);
  const int count = w.count();
  Asked<SEG> asked;
  ask_group<W>(rd, w, T, sh, asked);
  MasterRows<RPW> M;
  load_master<RPW, PACK, false>(rd, io, w, T, L, M);
  put_group<W>(rd, w, T, sh, asked);
  if ((int)threadIdx.x < count) sh.aux[threadIdx.x] = w.score(rd, threadIdx.x);
  lds_barrier();
  // Rolling requests: row k of the next agent is asked for as soon as row k of this one has been used, into the
  // registers that just became free, so a wavefront keeps its eight 16-byte loads per lane in flight all the
  // time instead of only between two arithmetic phases.  The loop body has no branch around a load: a request
  // that has nothing to fetch (a row past the span, a lane past the heads, the agent after the last) reads the
  // first row of the master page instead, and its result is not used; with straight-line code the compiler
  // counts the outstanding loads exactly and waits for the oldest pair only.
  const u32x4* idle = io.master_k + w.d.row0 * ((int64_t)rd.heads * 16) + L.jb;
  u32x4 akl[RPW], akh[RPW];
  auto request = [&](const auto& from, int g, int k) {
    const int64_t base = dest_row(from, row_bytes, group_row<PACK, W>(k, rd.heads, T) + (PACK ? L.rk : 0));
    const bool ok = g < count && M.valid[k] && M.template kok<PACK>(L, k);
    const u32x4* lo = ok ? chunk_at(pk, base, L.klo) : idle;
    const u32x4* hi = ok ? chunk_at(pk, base, L.khi) : idle + 8;
    akl[k] = ld16<NTL>(lo); akh[k] = ld16<NTL>(hi);
  };
#pragma unroll
  for (int k = 0; k < RPW; ++k) { request(origin_of(sh, 0), 0, k); __builtin_amdgcn_sched_barrier(0); }   // in the order the loop uses them
  for (int g = 0; g < count; ++g) {
    float c[8], s[8];
    const auto next = origin_of(sh, min(g + 1, count - 1));
    if (!SEG) load_tab<IL>(sh, g, 0, L.jb, c, s);
#pragma unroll
    for (int k = 0; k < RPW; ++k) {
      if (SEG) load_tab<IL>(sh, g, group_row<PACK, W>(k, rd.heads, T) + (PACK ? L.rk : 0), L.jb, c, s);
      u32x4 rlo, rhi;
      keep_packed<RPW == 8 && !SEG>(M.kl[k], M.kh[k]);
      rotate16<IL>(M.kl[k], M.kh[k], c, s, rlo, rhi);
      float acc = 0.f;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float d0 = bf_lo(akl[k][q]) - bf_lo(rlo[q]), d1 = bf_hi(akl[k][q]) - bf_hi(rlo[q]);
        float d2 = bf_lo(akh[k][q]) - bf_lo(rhi[q]), d3 = bf_hi(akh[k][q]) - bf_hi(rhi[q]);
        acc = __builtin_fmaf(d0, d0, acc); acc = __builtin_fmaf(d1, d1, acc);
        acc = __builtin_fmaf(d2, d2, acc); acc = __builtin_fmaf(d3, d3, acc);
      }
      request(next, g + 1, k);
      const int width = PACK ? 8 * rd.heads : 64;
      acc = row_sum_to_last_lane(L.kok ? acc : 0.f, width);
      if ((threadIdx.x & (width - 1)) == width - 1 && (!PACK || L.kok)) s_score[g][group_row<PACK, W>(k, rd.heads, T) + (PACK ? L.rk : 0)] = acc;   // (no store to memory among the loads: the count of outstanding accesses stays exact)
    }
  }
  lds_barrier();
  const int rows = w.rows();
  for (int i = threadIdx.x; i < count * T; i += 64 * W) {
    const int g = T == 16 ? i >> 4 : i >> 5, r = i & (T - 1);
    if (r < rows) pl.score[sh.aux[g] + r] = s_score[g][r];
  }
}

// Important positions of one agent: the k = ceil(ratio * S) tokens with the largest score among those
// with !(score <= min_score), ties towards the lower token index, listed in ascending token order.
// Radix select on the fp32 bit patterns (non-negative floats order like unsigned integers; NaN sorts
// above everything), then an ordered compaction.  Also the agent's total deviation, and, by the workgroup that
// delivers a session's last total, the session's master.
// One workgroup per agent, so the launch lasts as long as one agent takes: a chain of passes over the agent's
// scores with barriers between them.  16 wavefronts instead of 4 shorten every pass; the scores are read from memory
// once and their keys stay in LDS (64 KB = 16384 tokens, longer spans read the rest again); the compaction gives
// every thread consecutive tokens, so that one scan over the workgroup serves the whole span.  (250 agents x 5000
// tokens, under the profiler: 36 + 5 us with 4 wavefronts, keys read again in every pass and a launch of its own for the
// masters; 21 us now; the whole check-layer call 441 -> 426 us.)
// Spans of up to 512 tokens leave most of 16 wavefronts without work at every barrier: 4 wavefronts there (call with 144,
// 242 and 500 tokens: 12.8, 15.4 and 21.1 us with 16, 11.8, 14.4 and 20.6 with 4; 600, 800 and 1024 tokens: 12.2, 13.9 and
// 13.1 with 16, 12.9, 15.0 and 14.0 with 4).
constexpr int kSelBlock = 1024, kSelKeys = 16384;
constexpr int kSelSmall = 256, kSelShort = 512;

// Master of a session: the agent with the lowest total deviation (NaN counts as +inf; ties go to the agent listed
// first).  One wavefront; the totals were delivered by other workgroups, so they are read at device scope.
__device__ __forceinline__ void choose_master(const RoundDev& rd, const PlanDev& pl, int session) {
  const SessionDev sd = rd.sess[session];
  const int lane = threadIdx.x & 63;
  float best = __builtin_inff();
  int best_i = 0x7fffffff;
  for (int q = lane; q < sd.n_agents; q += 64) {
    const int a = rd.order[sd.order_begin + q];
    float t = __hip_atomic_load(&pl.total[a], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (t != t) t = __builtin_inff();
    if (t < best || (t == best && a < best_i)) { best = t; best_i = a; }
  }
#pragma unroll
  for (int sft = 32; sft > 0; sft >>= 1) {
    const float ob = __shfl_xor(best, sft);
    const int oi = __shfl_xor(best_i, sft);
    if (ob < best || (ob == best && oi < best_i)) { best = ob; best_i = oi; }
  }
  if (lane == 0) pl.master[session] = sd.n_agents ? best_i : -1;
}

template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void tdk_select_kernel(const RoundDev rd, const PlanDev pl) {
  constexpr int kSelWaves = BLOCK / 64, kKeys = BLOCK == kSelBlock ? kSelKeys : kSelShort;
  __shared__ uint32_t keys[kKeys];
  __shared__ uint32_t hist[4][256];             // one histogram per pass: a pass costs one barrier
  __shared__ double s_sum[kSelWaves];
  __shared__ int s_a[kSelWaves], s_b[kSelWaves];
  __shared__ int s_last;
  const int a = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  if (a == 0)                                   // sessions without agents have no workgroup of their own
    for (int s = tid; s < rd.n_sessions; s += BLOCK)
      if (rd.sess[s].n_agents == 0) pl.master[s] = -1;
  if (a >= rd.n_agents) return;
  const AgentDev ad = rd.agents[a];
  const int S = rd.sess[ad.session].span;
  const float* sc = pl.score + ad.score_off;
  const float min_score = pl.min_score;
  auto to_key = [&](float v) -> uint32_t { return !(v <= min_score) ? (__float_as_uint(v) & 0x7fffffffu) : 0u; };
  auto key_of = [&](int m) -> uint32_t { return m < kKeys ? keys[m] : to_key(sc[m]); };
  for (int q = tid; q < 4 * 256; q += BLOCK) hist[q >> 8][q & 255] = 0u;
  __syncthreads();
  // total deviation, number of candidates, keys, and the first pass's histogram
  double part = 0.0;
  int cand = 0;
  // (eight scores per thread in flight: one after the other they are five memory latencies at 5000 tokens; 4 x 3 agents x
  // 5776 tokens, 2 heads, 23.0 -> 22.2 us for the call, 21 x 8773 41.0 -> 39.7)
  constexpr int kAhead = 8;
  for (int m0 = tid; m0 < S; m0 += kAhead * BLOCK) {
    float v[kAhead];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) v[q] = sc[min(m0 + q * BLOCK, S - 1)];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) {
      const int m = m0 + q * BLOCK;
      if (m >= S) break;
      const uint32_t key = to_key(v[q]);
      part += (double)v[q];
      cand += key != 0u;
      if (key != 0u) atomicAdd(&hist[0][key >> 24], 1u);
      if (m < kKeys) keys[m] = key;
    }
  }
#pragma unroll
  for (int sft = 32; sft > 0; sft >>= 1) { part += __shfl_xor(part, sft); cand += __shfl_xor(cand, sft); }
  if (lane == 0) { s_sum[wave] = part; s_a[wave] = cand; }
  __syncthreads();
  double sum = 0.0;
  int n_cand = 0;
#pragma unroll
  for (int q = 0; q < kSelWaves; ++q) { sum += s_sum[q]; n_cand += s_a[q]; }
  const float total = (float)sum;
  if (tid == 0) {
    // The exchange's answer means that the total has reached memory; only then does the ticket count it.  The
    // workgroup that draws a session's last ticket puts the counter back to zero.
    const float old = atomicExch(&pl.total[a], total);
    asm volatile("" : : "v"(old) : "memory");
    const int ticket = atomicAdd(&rd.tickets[ad.session], 1);
    s_last = ticket == rd.sess[ad.session].n_agents - 1;
    if (s_last) atomicExch(&rd.tickets[ad.session], 0);
  }
  int64_t k = (int64_t)ceil((double)pl.ratio * (double)S);
  if (k > S) k = S;
  if (k > pl.k_stride) k = pl.k_stride;
  if (k > n_cand) k = n_cand;
  if (k <= 0) {
    if (tid == 0) pl.n_important[a] = 0;
    __syncthreads();
    if (s_last && wave == 0) choose_master(rd, pl, ad.session);
    return;
  }
  // radix select: the key of the k-th largest candidate, 8 bits at a time from the top
  uint32_t mask = 0u, prefix = 0u, need = (uint32_t)k;
#pragma unroll
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = 24 - 8 * pass;
    if (pass > 0) {
      for (int m = tid; m < S; m += BLOCK) {
        const uint32_t key = key_of(m);
        if (key != 0u && (key & mask) == prefix) atomicAdd(&hist[pass][(key >> shift) & 255u], 1u);
      }
      __syncthreads();
    }
    // the bin that holds the need-th largest key: every wavefront looks at all 256 counts, lane l at bins
    // 4 l .. 4 l + 3, with a suffix scan over the lanes; exactly one bin has above < need <= above + own
    const uint4 c = reinterpret_cast<const uint4*>(hist[pass])[lane];
    const uint32_t own = c.x + c.y + c.z + c.w;
    uint32_t inc = own;                                   // own + the bins of the higher lanes
#pragma unroll
    for (int sft = 1; sft < 64; sft <<= 1) {
      const uint32_t v = __shfl_down(inc, sft);
      if (lane + sft < 64) inc += v;
    }
    uint32_t above = inc - own;
    int bin = -1;
    uint32_t left = 0u;
    const uint32_t cnt[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
    for (int q = 3; q >= 0; --q) {
      if (above < need && above + cnt[q] >= need) { bin = 4 * lane + q; left = need - above; }
      above += cnt[q];
    }
    const int src = __ffsll((unsigned long long)__ballot(bin >= 0)) - 1;
    need = __shfl(left, src);
    prefix |= (uint32_t)__shfl(bin, src) << shift;
    mask |= 255u << shift;
  }
  const uint32_t tkey = prefix;
  const int need_eq = (int)need;       // how many tokens equal to the threshold key are taken (the first ones)
  // ordered compaction: thread t takes tokens [t c, (t + 1) c)
  const int per = (S + BLOCK - 1) / BLOCK, m0 = min(tid * per, S), m1 = min(m0 + per, S);
  int gt = 0, eq = 0;
  for (int m = m0; m < m1; ++m) {
    const uint32_t key = key_of(m);
    gt += key > tkey;
    eq += key == tkey;                 // (tkey is a candidate's key, never zero)
  }
  int gt_before = gt, eq_before = eq;
#pragma unroll
  for (int sft = 1; sft < 64; sft <<= 1) {
    const int u = __shfl_up(gt_before, sft), v = __shfl_up(eq_before, sft);
    if (lane >= sft) { gt_before += u; eq_before += v; }
  }
  if (lane == 63) { s_a[wave] = gt_before; s_b[wave] = eq_before; }
  gt_before -= gt;
  eq_before -= eq;
  __syncthreads();
  int all_gt = 0;
#pragma unroll
  for (int q = 0; q < kSelWaves; ++q) {
    if (q < wave) { gt_before += s_a[q]; eq_before += s_b[q]; }
    all_gt += s_a[q];
  }
  int32_t* out = pl.important + (int64_t)a * pl.k_stride;
  for (int m = m0; m < m1; ++m) {
    const uint32_t key = key_of(m);
    const bool is_gt = key > tkey, is_eq = key == tkey;
    if (is_gt || (is_eq && eq_before < need_eq)) out[gt_before + min(eq_before, need_eq)] = m;
    gt_before += is_gt;
    eq_before += is_eq;
  }
  if (tid == 0) pl.n_important[a] = all_gt + need_eq;
  if (s_last && wave == 0) choose_master(rd, pl, ad.session);
}

// Access-pattern probes: the page kernels' memory accesses with no arithmetic and no master.
// Plain form: one workgroup per page, contiguous 4 KB per step, ordinary stores / dependent loads.
__global__ __launch_bounds__(kBlock) void tdk_page_fill_kernel(u32x4* __restrict__ dst, const int32_t* __restrict__ ids,
                                                              int page_u4, uint32_t word) {
  const u32x4 v = {word, word, word, word};
  u32x4* p = dst + (size_t)ids[blockIdx.x] * page_u4;
  for (int i = threadIdx.x; i < page_u4; i += kBlock) p[i] = v;
}

__global__ __launch_bounds__(kBlock) void tdk_page_read_kernel(const u32x4* __restrict__ src, const int32_t* __restrict__ ids,
                                                              int page_u4, u32x4* __restrict__ sink) {
  const u32x4* p = src + (size_t)ids[blockIdx.x] * page_u4;
  u32x4 acc = {0, 0, 0, 0};
  for (int i = threadIdx.x; i < page_u4; i += kBlock) acc ^= p[i];
  // never true for the probe's fill pattern; keeps the loads alive
  if (acc[0] == 0x9e3779b9u && acc[1] == 0x7f4a7c15u) sink[0] = acc;
}

// Product form: exactly the traversal of the page kernels.  A workgroup takes `group` pages of the id list (as
// a work item takes a group of agents); its four wavefronts own interleaved rows; a lane touches the two
// halves of a head row in the K plane and two chunks 1 KB apart in the V plane; streaming stores / non-temporal
// loads; all 16 accesses of a wavefront's rows of one page are issued before anything waits for them.
template <int RPW>
__global__ __launch_bounds__(kBlock) void tdk_page_fill_product_kernel(u32x4* __restrict__ pk, u32x4* __restrict__ pv,
                                                                      const int32_t* __restrict__ ids, int n_pages, int group,
                                                                      int heads, uint32_t word) {
  constexpr int T = RPW * kWaves;
  const Lane L = lane_geometry<false>(heads, T);
  const int wave = threadIdx.x >> 6;
  const int64_t row_u4 = (int64_t)heads * 16;
  const u32x4 v = {word, word ^ threadIdx.x, word, blockIdx.x};
  for (int g = 0; g < group; ++g) {
    const int64_t q = (int64_t)blockIdx.x * group + g;
    if (q >= n_pages) break;
    const int64_t page = ids[q];
#pragma unroll
    for (int k = 0; k < RPW; ++k) {
      const int64_t base = (page * T + wave + kWaves * k) * row_u4;
      if (L.kok) { st16<true>(pk + base + L.klo, v); st16<true>(pk + base + L.khi, v); }
      if (L.v0ok) st16<true>(pv + base + L.v0, v);
      if (L.v1ok) st16<true>(pv + base + L.v1, v);
    }
  }
}

template <int RPW>
__global__ __launch_bounds__(kBlock) void tdk_page_read_product_kernel(const u32x4* __restrict__ pk, const u32x4* __restrict__ pv,
                                                                      const int32_t* __restrict__ ids, int n_pages, int group,
                                                                      int heads, u32x4* __restrict__ sink) {
  constexpr int T = RPW * kWaves;
  const Lane L = lane_geometry<false>(heads, T);
  const int wave = threadIdx.x >> 6;
  const int64_t row_u4 = (int64_t)heads * 16;
  u32x4 acc = {0, 0, 0, 0};
  for (int g = 0; g < group; ++g) {
    const int64_t q = (int64_t)blockIdx.x * group + g;
    if (q >= n_pages) break;
    const int64_t page = ids[q];
    u32x4 a[RPW][4];
    const u32x4 z = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < RPW; ++k) {
      const int64_t base = (page * T + wave + kWaves * k) * row_u4;
      a[k][0] = z; a[k][1] = z; a[k][2] = z; a[k][3] = z;
      if (L.kok) { a[k][0] = ld16<true>(pk + base + L.klo); a[k][1] = ld16<true>(pk + base + L.khi); }
      if (L.v0ok) a[k][2] = ld16<true>(pv + base + L.v0);
      if (L.v1ok) a[k][3] = ld16<true>(pv + base + L.v1);
    }
#pragma unroll
    for (int k = 0; k < RPW; ++k) acc ^= a[k][0] ^ a[k][1] ^ a[k][2] ^ a[k][3];
  }
  if (acc[0] == 0x9e3779b9u && acc[1] == 0x7f4a7c15u) sink[0] = acc;
}

// ---------------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------------

// Launch of a page kernel that writes (rerotate, decode).  Static distribution: one workgroup per work item.
// Queued (TDK_TUNE_XCD_QUEUES, and only for long launches, see plan_loops: a short one is over before an imbalance between the XCDs can build
// up, and the hardware's own dispatch of fresh workgroups fills freed wavefront slots sooner than a looping workgroup does): two workgroups
// per compute unit that loop over the items (see below).  `queued_kernel` / `static_kernel` are the two instantiations; `large`: a long launch.
// `half_pages`: the call writes one of the two planes only.
// `extra` static workgroups behind the page items (decode's payload copies on small rounds); returns whether they
// were launched (only the static form takes them).
template <class KernelQ, class KernelS, class... Args>
static bool launch_write_pages(const RoundDev& rd, KernelQ queued_kernel, KernelS static_kernel, int threads, bool large, bool half_pages, int extra, hipStream_t st, Args... args) {
  if ((rd.nontemporal & 128) && (large || (threads == kBlock && (rd.nontemporal & 512)))) {
    // Two looping workgroups per compute unit, although three may fit: memory is saturated with one per unit already,
    // and the fewer pages are being written at a time, the better DRAM takes it (batched250: decode 876 us with
    // three per unit, 868 with two, 860 with one; rerotate 958 / 953 / 962; `long` loses 7 % with one).
    const int64_t looping = 2 * (int64_t)std::max(rd.n_cus, 1);
    hipLaunchKernelGGL(queued_kernel, dim3((unsigned)std::min<int64_t>(rd.n_work, looping)), dim3(kBlock), 0, st, rd, args...);
    return false;
  }
  const bool ride = extra > 0 && !large && (rd.nontemporal & 1024);
  RoundDev rs = rd;
  if (half_pages) {
    rs.work = rd.pwork;
    rs.n_work = rd.n_pwork;
  }
  rs.dyn_begin = rs.n_work;
  rs.dyn_count = 0;
  if ((rd.nontemporal & 2048) && rs.n_work >= 64) {
    // the last fifth of the items is shared (see Items::first); twice as many workgroups as items stand by for it
    const int tail = rs.n_work / 5;
    rs.dyn_begin = rs.n_work - tail;
    rs.dyn_count = 2 * tail;
  }
  hipLaunchKernelGGL(static_kernel, dim3((unsigned)(rs.dyn_begin + rs.dyn_count) + (ride ? (unsigned)extra : 0u)), dim3((unsigned)threads), 0, st, rs, args...);
  return ride;
}

template <int V> using ic = std::integral_constant<int, V>;

template <class F> static void with_rpw(int page_tokens, F f) { if (page_tokens == 16) f(ic<4>{}); else f(ic<8>{}); }
// Row groups per wavefront, and whether a group holds several rows.  With 1, 2 or 4 KV heads a row alone would leave
// seven eighths, three quarters or half of a wavefront idle in every access and as many requests less in flight
// (37 agents x 2999 tokens, 4 heads, both planes stored and restored one at a time: 169 us with one row per access, 149
// with two; drawn rounds with 1 or 2 heads up to 1.8 times); 3 heads keep one row (rows of 24 lanes do not divide the
// page), 5 and more fill the wavefront by themselves.
template <class F> static void with_rows(const RoundDev& rd, bool wide, F f) {
  const int H = rd.heads, T = rd.page_tokens;
  if (H != 1 && H != 2 && H != 4) {
    if (wide) f(ic<2>{}, std::false_type{});
    else with_rpw(T, [&](auto rpw) { f(rpw, std::false_type{}); });
    return;
  }
  switch (T / (kWaves * rows_per_access(H, T))) {
    case 1: f(ic<1>{}, std::true_type{}); break;
    case 2: f(ic<2>{}, std::true_type{}); break;
    default: f(ic<4>{}, std::true_type{}); break;
  }
}
// Eight wavefronts per workgroup, two rows of every page each, instead of four with four rows?  16-token pages whose rows fill an access.
//   Kernels that read: while every item has a compute unit to itself.  What an item takes is then what one of its wavefronts does one
//   after the other (store of 40 to 100 pairs 14.1 -> 13.0 us, check layer of 40 to 270 13.0 -> 12.7; from one and a half items per unit on
//   0.95 to 1.06 times, no rule found).
//   Kernels that write both planes: launches of 6 (agent, page) pairs per compute unit and more whose items have several agents, up to
//   those that loop.  Twice the wavefronts hide the items' starts, and an item's pages are written by as many (25 agents x 5000 tokens, collect
//   98.1 -> 96.2 us, restore 100.5 -> 99.1; 2 x 35 x 949 57.5 -> 56.2; over 40 such launches 1.00 to 1.05).  Items of two agents end too
//   soon for it (ten sessions of 2 x 1040 tokens 27.2 -> 28.6), and smaller launches have too few items (12 agents x 600 tokens, restore 9.5 -> 11.3).
static bool wide_item_rows(const RoundDev& rd) { const int H = rd.heads; return H != 1 && H != 2 && H != 4 && rd.page_tokens == 16; }
static bool wide_reads(const RoundDev& rd) { return wide_item_rows(rd) && rd.n_rwork <= rd.n_cus; }
static bool wide_writes(const RoundDev& rd) {
  const int64_t cus = rd.n_cus;
  return wide_item_rows(rd) && !(rd.nontemporal & 512) && rd.agent_pages >= 6 * cus && rd.agent_pages < 64 * cus && 2 * rd.agent_pages >= 5 * (int64_t)rd.n_work;
}
template <class F> static void with_bool(bool b, F f) { if (b) f(std::true_type{}); else f(std::false_type{}); }
template <class F> static void with_planes(int planes, F f) {
  if (planes == 1) f(ic<1>{}); else if (planes == 2) f(ic<2>{}); else f(ic<3>{});
}

hipError_t launch_places(const RoundDev& rd, PlaceDev* places, hipStream_t st) {
  if (rd.n_agents == 0) return hipSuccess;
  // (its own status: an error that the caller's calls have left behind is not this one's)
  RoundDev r = rd;
  void* args[] = {&r, &places};
  return hipLaunchKernel(reinterpret_cast<const void*>(tdk_places_kernel), dim3((unsigned)rd.n_agents), dim3(kBlock), args, 0, st);
}

hipError_t launch_rerotate(const RoundDev& rd, const LayerDev& io, hipStream_t st) {
  if (rd.n_work == 0) return hipSuccess;
  with_rows(rd, wide_writes(rd), [&](auto rpw, auto pack) { with_bool(rd.interleaved != 0, [&](auto il) { with_bool((rd.nontemporal & 1) != 0, [&](auto nt) {
    with_bool(rd.seg != 0, [&](auto sg) {
      constexpr int R = decltype(rpw)::value;
      constexpr bool P = decltype(pack)::value, I = decltype(il)::value, N = decltype(nt)::value, G = decltype(sg)::value;
      constexpr bool kQueues = waves_of(R, P) == kWaves;
      const bool large = kQueues && plan_loops(rd.n_work, rd.agent_pages, rd.n_cus, R, P, 3, G);
      launch_write_pages(rd, tdk_rerotate_kernel<R, P, I, N, G, kQueues>, tdk_rerotate_kernel<R, P, I, N, G, false>, 64 * waves_of(R, P), large, false, 0, st, io);
    });
  }); }); });
  return hipGetLastError();
}

hipError_t launch_flag(const RoundDev& rd, const LayerDev& io, float eps, int planes, hipStream_t st) {
  if (rd.n_work == 0) return hipSuccess;
  with_rows(rd, wide_reads(rd), [&](auto rpw, auto pack) { with_bool(rd.interleaved != 0, [&](auto il) { with_planes(planes, [&](auto pm) {
    with_bool(rd.seg != 0, [&](auto sg) { with_bool((rd.nontemporal & 4) != 0, [&](auto ntl) {
      hipLaunchKernelGGL((tdk_flag_kernel<decltype(rpw)::value, decltype(pack)::value, decltype(il)::value, decltype(pm)::value, decltype(sg)::value,
                                          decltype(ntl)::value>), dim3(rd.n_rwork), dim3(64 * waves_of(decltype(rpw)::value, decltype(pack)::value)), 0, st, rd, io, eps);
    }); });
  }); }); });
  return hipGetLastError();
}

hipError_t launch_compact(const RoundDev& rd, const DiffDev& d, hipStream_t st) {
  const dim3 grid(rd.n_agents ? (rd.n_agents + kCompactWaves - 1) / kCompactWaves : 1);
  hipLaunchKernelGGL(tdk_compact_kernel, grid, dim3(kCompactBlock), 0, st, rd, d);
  return hipGetLastError();
}

hipError_t launch_gather(const RoundDev& rd, const LayerDev& io, const DiffDev& d, int planes, int grid_size, hipStream_t st) {
  if (rd.n_agents == 0 || d.capacity == 0 || grid_size <= 0) return hipSuccess;
  hipLaunchKernelGGL(tdk_gather_kernel, dim3(grid_size), dim3(kBlock), 0, st, rd, io, d, planes);
  return hipGetLastError();
}

bool lists_in_gather(const RoundDev& rd) { return rd.agent_pages <= kListPages; }

hipError_t launch_list_gather(const RoundDev& rd, const LayerDev& io, const DiffDev& d, int planes, int grid_size, hipStream_t st) {
  // (capacities are mostly generous: workgroups without a slot repeat the count for nothing, so no more than four per
  // compute unit are launched)
  const int blocks = std::min(plan_copy_workgroups(grid_size, slot_batches(rd, planes), rd.n_cus, 1 << 30), 4 * std::max(rd.n_cus, 1));
  hipLaunchKernelGGL(tdk_list_gather_kernel, dim3((unsigned)std::max(1, blocks)), dim3(kBlock), 0, st, rd, io, d, planes);
  return hipGetLastError();
}

// scatter_blocks > 0: so many workgroups may ride behind the page items to copy the listed pages; *scattered says
// whether they did (then no separate scatter launch is needed)
hipError_t launch_decode(const RoundDev& rd, const LayerDev& io, const DiffDev& d, int planes, int scatter_blocks, bool* scattered,
                         hipStream_t st) {
  *scattered = false;
  if (rd.n_work == 0) return hipSuccess;
  const bool wide = planes == 3 && wide_writes(rd);
  if (rd.n_agents == 0 || d.capacity == 0) scatter_blocks = 0;
  if (slots_shared(rd)) {
    // (Three workgroups of the kernels for both planes fit a compute unit; the page items are launched with those that stand by for the last
    // fifth.  Only two fit of the kernels with eight wavefronts and of those for 32-token pages whose rows fill an access, but the limit is for
    // slots of two batches: with eight wavefronts a slot is one batch, and 32-token pages have two with five heads only.  Of the kernels for one
    // plane more fit, and no limit showed: 60 agents x 700 tokens, pages of 32, stored and restored one plane at a time 109.7 us, 111.9 with a
    // limit of four.)
    const int left = planes == 3 ? 3 * rd.n_cus - rd.n_work - rd.n_work / 5 : -1;
    scatter_blocks = plan_copy_workgroups(scatter_blocks, slot_batches(rd, planes, wide ? 2 * kWaves : kWaves), rd.n_cus, left);
  }
  with_rows(rd, wide, [&](auto rpw, auto pack) { with_bool(rd.interleaved != 0, [&](auto il) { with_bool((rd.nontemporal & 2) != 0, [&](auto nt) {
    with_planes(planes, [&](auto pm) { with_bool(rd.seg != 0, [&](auto sg) {
      constexpr int R = decltype(rpw)::value, M = decltype(pm)::value;
      constexpr bool P = decltype(pack)::value, I = decltype(il)::value, N = decltype(nt)::value, G = decltype(sg)::value;
      constexpr bool kQueues = waves_of(R, P) == kWaves;
      if constexpr (kQueues || M == 3) {        // (eight wavefronts: both planes only)
        const bool large = kQueues && plan_loops(rd.n_work, rd.agent_pages, rd.n_cus, R, P, M, G);
        *scattered = launch_write_pages(rd, tdk_decode_kernel<R, P, I, N, M, G, kQueues>, tdk_decode_kernel<R, P, I, N, M, G, false>, 64 * waves_of(R, P),
                                        large, planes != 3, scatter_blocks, st, io, d, scatter_blocks);
      }
    }); });
  }); }); });
  return hipGetLastError();
}

hipError_t launch_scatter(const RoundDev& rd, const LayerDev& io, const DiffDev& d, int planes, int grid_size, hipStream_t st) {
  if (rd.n_agents == 0 || d.capacity == 0 || grid_size <= 0) return hipSuccess;
  if (rd.interleaved) hipLaunchKernelGGL(tdk_scatter_kernel<true>, dim3(grid_size), dim3(kBlock), 0, st, rd, io, d, planes);
  else hipLaunchKernelGGL(tdk_scatter_kernel<false>, dim3(grid_size), dim3(kBlock), 0, st, rd, io, d, planes);
  return hipGetLastError();
}

hipError_t launch_keydiff(const RoundDev& rd, const LayerDev& io, const PlanDev& pl, hipStream_t st) {
  if (rd.n_work == 0) return hipSuccess;
  with_rows(rd, wide_reads(rd), [&](auto rpw, auto pack) { with_bool(rd.interleaved != 0, [&](auto il) { with_bool(rd.seg != 0, [&](auto sg) {
    with_bool((rd.nontemporal & 4) != 0, [&](auto ntl) {
      hipLaunchKernelGGL((tdk_keydiff_kernel<decltype(rpw)::value, decltype(pack)::value, decltype(il)::value, decltype(sg)::value, decltype(ntl)::value>),
                         dim3(rd.n_rwork), dim3(64 * waves_of(decltype(rpw)::value, decltype(pack)::value)), 0, st, rd, io, pl);
    });
  }); }); });
  return hipGetLastError();
}

hipError_t launch_select(const RoundDev& rd, const PlanDev& pl, hipStream_t st) {
  if (rd.n_agents == 0 && rd.n_sessions == 0) return hipSuccess;
  const dim3 grid(std::max(rd.n_agents, 1));
  if (rd.max_span <= kSelShort) hipLaunchKernelGGL(tdk_select_kernel<kSelSmall>, grid, dim3(kSelSmall), 0, st, rd, pl);
  else hipLaunchKernelGGL(tdk_select_kernel<kSelBlock>, grid, dim3(kSelBlock), 0, st, rd, pl);
  return hipGetLastError();
}

hipError_t launch_copy(u32x4* dst, const u32x4* src, size_t n16, hipStream_t st) {
  if (n16 == 0) return hipSuccess;
  // one 4 KB chunk per workgroup while the grid allows: workgroups are dispatched in order, so the chip
  // sweeps memory in one narrow sequential window, which is what DRAM serves fastest
  size_t blocks = (n16 + kBlock - 1) / kBlock;
  if (blocks > ((size_t)1 << 30)) blocks = (size_t)1 << 30;
  hipLaunchKernelGGL(tdk_copy_kernel, dim3((unsigned)blocks), dim3(kBlock), 0, st,
                     dst, src, n16);
  return hipGetLastError();
}

hipError_t launch_fill(u32x4* dst, uint32_t word, size_t n16, hipStream_t st) {
  if (n16 == 0) return hipSuccess;
  size_t blocks = (n16 + kBlock - 1) / kBlock;
  if (blocks > ((size_t)1 << 30)) blocks = (size_t)1 << 30;
  hipLaunchKernelGGL(tdk_fill_kernel, dim3((unsigned)blocks), dim3(kBlock), 0, st,
                     dst, word, n16);
  return hipGetLastError();
}

hipError_t launch_page_fill(u32x4* dst, const int32_t* ids, int n_pages, int page_u4, uint32_t word, hipStream_t st) {
  if (n_pages <= 0) return hipSuccess;
  hipLaunchKernelGGL(tdk_page_fill_kernel, dim3(n_pages), dim3(kBlock), 0, st, dst, ids, page_u4, word);
  return hipGetLastError();
}

hipError_t launch_page_read(const u32x4* src, const int32_t* ids, int n_pages, int page_u4, u32x4* sink, hipStream_t st) {
  if (n_pages <= 0) return hipSuccess;
  hipLaunchKernelGGL(tdk_page_read_kernel, dim3(n_pages), dim3(kBlock), 0, st, src, ids, page_u4, sink);
  return hipGetLastError();
}

hipError_t launch_page_fill_product(u32x4* pk, u32x4* pv, const int32_t* ids, int n_pages, int group, int heads, int page_tokens,
                                    uint32_t word, hipStream_t st) {
  if (n_pages <= 0) return hipSuccess;
  const dim3 grid((n_pages + group - 1) / group);
  if (page_tokens == 16) hipLaunchKernelGGL(tdk_page_fill_product_kernel<4>, grid, dim3(kBlock), 0, st, pk, pv, ids, n_pages, group, heads, word);
  else hipLaunchKernelGGL(tdk_page_fill_product_kernel<8>, grid, dim3(kBlock), 0, st, pk, pv, ids, n_pages, group, heads, word);
  return hipGetLastError();
}

hipError_t launch_page_read_product(const u32x4* pk, const u32x4* pv, const int32_t* ids, int n_pages, int group, int heads,
                                    int page_tokens, u32x4* sink, hipStream_t st) {
  if (n_pages <= 0) return hipSuccess;
  const dim3 grid((n_pages + group - 1) / group);
  if (page_tokens == 16) hipLaunchKernelGGL(tdk_page_read_product_kernel<4>, grid, dim3(kBlock), 0, st, pk, pv, ids, n_pages, group, heads, sink);
  else hipLaunchKernelGGL(tdk_page_read_product_kernel<8>, grid, dim3(kBlock), 0, st, pk, pv, ids, n_pages, group, heads, sink);
  return hipGetLastError();
}

}  // namespace tdk
