// CPU-only test of the host side of the queue protocol against the device stand-in
// (device_standin.cpp), meant to be built with -fsanitize=thread.  Prints one line per check and
// exits non-zero on the first failure.
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <thread>
#include <vector>

#include <hip/hip_runtime_api.h>

#include "../../include/gpuos.h"
#include "../../paper_2604_17861_amd/csrc/gpuos_internal.h"

extern "C" uint64_t standin_errors();
extern "C" void standin_leave_before(uint64_t ticket);
extern "C" void standin_stall_ms(uint32_t ms);
extern "C" uint64_t standin_records();
extern "C" uint64_t standin_links();
extern "C" uint64_t standin_streams();
extern "C" uint64_t standin_alloc_calls();
extern "C" void standin_scratch_dirty();
extern "C" uint64_t standin_scratch_nonzero(uint64_t n);

#define CHECK(cond) do { if (!(cond)) { std::printf("FAILED %s:%d: %s\n", __FILE__, __LINE__, #cond); std::exit(1); } } while (0)

static gpuos_task add_task(uint16_t op, uint32_t numel, uint16_t dep = 0) {
  gpuos_task t;
  std::memset(&t, 0, sizeof(t));
  t.op_id = op; t.ndim = 1; t.n_inputs = 2; t.size[0] = numel;
  for (int k = 0; k < 2; ++k) { t.in[k].ptr = (void*)(uintptr_t)(0x100000 * (k + 1)); t.in[k].stride[0] = 1; t.in[k].dtype = GPUOS_F32; }
  t.out.ptr = (void*)(uintptr_t)0x900000; t.out.stride[0] = 1; t.out.dtype = GPUOS_F32;
  t.dep[0] = dep;
  return t;
}

static gpuos_ctx* make(uint32_t cap, bool nonblocking = false, bool harvester = false) {
  gpuos_config cfg;
  gpuos_default_config(&cfg);
  cfg.nonblocking_submit = nonblocking;
  cfg.harvester_thread = harvester;
  cfg.wait_timeout_ms = 20000;
  gpuos_ctx* c = nullptr;
  CHECK(gpuos_init(&c, cap, &cfg) == GPUOS_OK);
  CHECK(gpuos_register_op(c, 7, GPUOS_IMPL_ADD, nullptr) == GPUOS_OK);
  CHECK(gpuos_register_op(c, 9, GPUOS_IMPL_MUL, nullptr) == GPUOS_OK);
  return c;
}

// The ring record's check word must reject every mixture of the record a slot held on the previous
// lap and the record being written into it (write-combined stores land piecewise, in any order):
// all 8-byte pieces in which two same-shaped tasks differ, in every old / new combination.
static void check_word_rejects_mixtures() {
  using gpuos::Record;
  auto seal = [](Record& r, uint64_t ticket) {          // what gpuos_submit does to a packed record
    r.ticket = 0;
    r.check = gpuos::record_check_seed(ticket) - gpuos::record_check_sum(reinterpret_cast<const uint32_t*>(&r), 63);
  };
  auto verifies = [](const Record& r, uint64_t ticket) { // what the dispatcher does
    return gpuos::record_check_sum(reinterpret_cast<const uint32_t*>(&r), 64) == gpuos::record_check_seed(ticket);
  };
  for (uint64_t cap : {2ull, 64ull, 4096ull, 65536ull})
    for (uint64_t t : {0ull, 1ull, 63ull, 4095ull, 123456789ull, (1ull << 32) - 1, (1ull << 40) + 17}) {
      Record oldr, newr;
      std::memset(&oldr, 0, sizeof(oldr));
      oldr.op_id = 7; oldr.path = 1; oldr.ndim = 1; oldr.n_inputs = 2; oldr.nchunks = 1; oldr.chunk = 8192; oldr.numel = 2048;
      oldr.size[0] = 2048;
      newr = oldr;
      for (int k = 0; k < 4; ++k) { oldr.ptr[k] = 0x7f0000000000ull + 0x10000000ull * k + 8192ull * 77; newr.ptr[k] = 0x7f0000000000ull + 0x10000000ull * k + 8192ull * 1234; }
      seal(oldr, t);
      seal(newr, t + cap);
      CHECK(verifies(newr, t + cap) && verifies(oldr, t));
      CHECK(!verifies(oldr, t + cap) && !verifies(newr, t));
      const uint64_t* po = reinterpret_cast<const uint64_t*>(&oldr);
      const uint64_t* pn = reinterpret_cast<const uint64_t*>(&newr);
      int diff[32], nd = 0;
      for (int k = 0; k < 32; ++k) if (po[k] != pn[k]) diff[nd++] = k;
      CHECK(nd >= 2 && nd <= 8);
      for (unsigned mask = 0; mask + 1 < (1u << nd); ++mask) {     // every mixture except "all new"
        Record mix = newr;
        uint64_t* pm = reinterpret_cast<uint64_t*>(&mix);
        for (int j = 0; j < nd; ++j) if (!((mask >> j) & 1u)) pm[diff[j]] = po[diff[j]];   // bit clear: the old piece is still there
        CHECK(!verifies(mix, t + cap));
      }
    }
  std::printf("ok: check word rejects every old/new mixture of a slot's records\n");
}

// However large the chunks a context asks for, every chunk lies within what 32-bit byte offsets reach
// (the stand-in looks at each record): integer and float tensors, rows of whole vectors and ragged ones.
static void chunks_stay_addressable() {
  for (uint32_t elems : {1u << 24, 1u << 29, 800000000u, 0xffffffffu}) {
    gpuos_config cfg;
    gpuos_default_config(&cfg);
    cfg.chunk_elems = elems;
    cfg.wait_timeout_ms = 20000;
    gpuos_ctx* c = nullptr;
    CHECK(gpuos_init(&c, 64, &cfg) == GPUOS_OK);
    CHECK(gpuos_register_op(c, 7, GPUOS_IMPL_ADD, nullptr) == GPUOS_OK);
    CHECK(gpuos_register_op(c, 8, GPUOS_IMPL_SOFTMAX_LAST, nullptr) == GPUOS_OK);
    for (uint32_t dt : {GPUOS_F32, GPUOS_I32}) {
      gpuos_task t = add_task(7, 2147483647u - 1024u);
      t.in[0].dtype = t.in[1].dtype = t.out.dtype = (uint8_t)dt;
      CHECK(gpuos_submit(c, &t, 1, nullptr) == GPUOS_OK);
    }
    for (uint32_t n : {1024u, 1021u, 536870908u}) {
      gpuos_task t = add_task(8, 0);
      t.ndim = 2; t.n_inputs = 1;
      t.size[0] = 2147483647u / n; t.size[1] = n;
      t.in[0].stride[0] = t.out.stride[0] = n;
      t.in[0].stride[1] = t.out.stride[1] = 1;
      CHECK(gpuos_submit(c, &t, 1, nullptr) == GPUOS_OK);
    }
    CHECK(gpuos_flush(c) == GPUOS_OK && gpuos_wait(c, GPUOS_ALL, 0) == GPUOS_OK);
    CHECK(gpuos_shutdown(c) == GPUOS_OK);
  }
  CHECK(standin_errors() == 0);
  std::printf("chunks within 32-bit offsets: ok\n");
}

// Rows cut at memory's 16-byte blocks: the resource covers the whole chunk, and no store that is to do nothing (kNoLoad) falls
// inside it, up to the longest rows that the ragged executors take.
static void block_cuts_stay_below_the_offset_that_does_nothing() {
  for (uint32_t es : {2u, 4u})
    for (uint32_t skew = 0; skew < 16; skew += es)
      for (uint32_t bytes : {65540u, 128012u, gpuos::kNoLoad - 32, gpuos::kNoLoad - 16 - es, gpuos::kNoLoad - 16, gpuos::kNoLoad - 12, gpuos::kNoLoad - 8,
                             gpuos::kNoLoad - es, gpuos::kNoLoad}) {
        const uint64_t x = 0x7f0000000000ull + skew, o = 0x7e0000000000ull + skew;
        const gpuos::BlockCut c = gpuos::block_cut(x, o, bytes);
        CHECK(c.window <= gpuos::kNoLoad && c.window >= c.front + bytes);
        CHECK(c.blocks ? c.front == skew && c.window % 16 == 0 : c.front == 0 && c.window == bytes);
        CHECK(c.blocks == (skew + bytes <= gpuos::kNoLoad));
        CHECK(!gpuos::block_cut(x, o + es, bytes).blocks);
      }
  std::printf("ok: rows cut at blocks stay below the offset that does nothing\n");
}

// Which tasks of a submit the host marks as links of a run: whoever reads what the task right before it wrote, over
// buffers that are the same or apart, and nobody else.
static void runs_are_marked() {
  gpuos_ctx* c = make(256);
  CHECK(gpuos_register_op(c, 11, GPUOS_IMPL_MAX_LAST, nullptr) == GPUOS_OK);
  const uint32_t n = 1000;
  auto ptr = [](int k) { return (void*)(uintptr_t)(0x1000000 + 0x100000 * k); };
  auto link = [&](int in, int other, int out, uint16_t dep = 1) {
    gpuos_task t = add_task(7, n, dep);
    t.in[0].ptr = ptr(in); t.in[1].ptr = ptr(other); t.out.ptr = ptr(out);
    return t;
  };
  auto links_of = [&](std::vector<gpuos_task> v) {
    const uint64_t before = standin_links();
    v[0].dep[0] = 0;
    CHECK(gpuos_submit_flush(c, v.data(), (uint32_t)v.size(), nullptr) == GPUOS_OK);
    CHECK(gpuos_wait(c, GPUOS_ALL, 0) == GPUOS_OK);
    return standin_links() - before;
  };
  std::vector<gpuos_task> v = {link(0, 1, 2), link(2, 1, 3), link(3, 1, 2), link(2, 1, 2)};   // two buffers in turn, then in place
  CHECK(links_of(v) == 3);
  auto with = [&](int k, auto change) { std::vector<gpuos_task> w = v; change(w[k]); return links_of(w); };
  CHECK(with(1, [&](gpuos_task& t) { t.dep[0] = 0; }) == 2);                                  // names nothing
  CHECK(with(2, [&](gpuos_task& t) { t.dep[1] = 2; }) == 2);                                  // names another one too (and heads the next run)
  CHECK(with(1, [&](gpuos_task& t) { t.flags = GPUOS_FLAG_FENCE; }) == 2);
  CHECK(with(1, [&](gpuos_task& t) { t.size[0] = n - 4; }) == 1);                             // another length: neither before nor behind it
  CHECK(with(3, [&](gpuos_task& t) { t.in[0].ptr = ptr(1); }) == 2);                          // does not read what the one before wrote
  CHECK(with(1, [&](gpuos_task& t) { t.in[1].ptr = (char*)ptr(1) + 16; }) == 1);              // overlaps a buffer of the run in part
  CHECK(with(2, [&](gpuos_task& t) { t.out.ptr = (char*)ptr(1) - 16; }) == 1);
  CHECK(with(1, [&](gpuos_task& t) { t.in[0].ptr = (char*)t.in[0].ptr + 4; }) == 1);          // not aligned to a vector
  CHECK(with(1, [&](gpuos_task& t) { for (auto* q : {&t.in[0], &t.in[1], &t.out}) q->dtype = GPUOS_F16; }) == 1);
  std::vector<gpuos_task> big = v;                                                            // more chunks than a waiting task may have
  for (auto& t : big) t.size[0] = 200000;
  CHECK(links_of(big) == 0);
  std::vector<gpuos_task> many(150, link(2, 1, 2));
  CHECK(links_of(many) == 150 - 3);                                                           // runs of at most 64: three heads
  // a reduction over rows and what reads its scalars: 250 rows of 4, and rows of 5 that are no whole vectors
  auto rows = [&](int64_t r, int64_t len) {
    gpuos_task m = add_task(11, 1, 1), d = add_task(7, 1, 1);
    m.n_inputs = 1; m.ndim = 2; m.size[0] = r; m.size[1] = len;
    m.in[0].ptr = ptr(2); m.in[0].stride[0] = len; m.in[0].stride[1] = 1; m.out.ptr = ptr(5);
    d.ndim = 2; d.size[0] = r; d.size[1] = len;
    d.in[0].ptr = ptr(2); d.in[0].stride[0] = len; d.in[0].stride[1] = 1;
    d.in[1].ptr = ptr(5); d.in[1].stride[0] = 1; d.in[1].stride[1] = 0;
    d.out.ptr = ptr(3); d.out.stride[0] = len; d.out.stride[1] = 1;
    return std::vector<gpuos_task>{link(0, 1, 2), m, d};
  };
  CHECK(links_of(rows(250, 4)) == 2);
  for (uint32_t dt : {GPUOS_F16, GPUOS_BF16}) {                                               // the scalars read as what they were written as, or not
    std::vector<gpuos_task> h = rows(250, 4);
    h[1].out.dtype = GPUOS_F16;
    h[2].in[1].dtype = (uint8_t)dt;
    CHECK(links_of(h) == (dt == GPUOS_F16 ? 2 : 1));
  }
  CHECK(links_of(rows(200, 5)) == 0);
  // a task that is refused changes nothing: three large adds, the last one's bias 24 wide, stay by themselves whether a reduction
  // over rows of 16, which does not go with that bias, follows or not; nor does a refused one's bias keep another out
  {
    std::vector<gpuos_task> h = {link(0, 1, 2), link(2, 1, 3), link(3, 4, 2)};
    for (auto& t : h) t.size[0] = 240000;
    gpuos_task& bias = h[2];
    bias.ndim = 2; bias.size[0] = 10000; bias.size[1] = 24;
    for (auto* q : {&bias.in[0], &bias.in[1], &bias.out}) { q->stride[0] = q == &bias.in[1] ? 0 : 24; q->stride[1] = 1; }
    for (int k = 0; k < 3; ++k) for (auto* q : {&h[k].in[0], &h[k].in[1], &h[k].out}) q->ptr = (void*)((uintptr_t)q->ptr * 16);
    CHECK(links_of(h) == 0);
    gpuos_task max16 = rows(15000, 16)[1];
    max16.in[0].ptr = h[2].out.ptr;
    h.push_back(max16);
    CHECK(links_of(h) == 0);
  }
  // scalars that a task of the run wrote are not in registers any more behind other scalars of the rows: who reads or writes them
  // then begins a run of its own (add m, add k, add m again; the same with a reduction into m at the end)
  {
    std::vector<gpuos_task> h = rows(250, 4);
    gpuos_task by_m = h[2], by_k = h[2];
    by_m.in[0].ptr = by_m.out.ptr = by_k.in[0].ptr = by_k.out.ptr = ptr(3);
    by_k.in[1].ptr = ptr(6);
    gpuos_task again = h[1];
    again.in[0].ptr = ptr(3);
    CHECK(links_of({h[0], h[1], h[2], by_m, by_k, by_k}) == 5);
    CHECK(links_of({h[0], h[1], h[2], by_k, by_m}) == 3);
    CHECK(links_of({h[0], h[1], h[2], by_k, by_m, by_k}) == 4);
    CHECK(links_of({h[0], h[1], h[2], by_k, again}) == 3);
    CHECK(links_of({h[0], h[1], h[2], again, by_m}) == 4);
  }
  // a run's tasks complete at its end: together they are at most 2^30 elements
  for (int64_t r : {1ll << 22, 1ll << 23}) {
    std::vector<gpuos_task> h = rows(r, 64);
    h[0].size[0] = r * 64;
    for (auto& t : h) for (auto* q : {&t.in[0], &t.in[1], &t.out}) q->ptr = (void*)((uintptr_t)q->ptr << 16);
    CHECK(links_of(h) == (r == 1 << 22 ? 2 : 1));
  }
  CHECK(gpuos_shutdown(c) == GPUOS_OK);
  std::printf("ok: links of runs are marked, and nothing else\n");
}

// Calls of more than two batches are checked first and then packed batch by batch: whatever a descriptor is, such a call answers as
// a single submit of it does, enqueues nothing if one is refused, and marks the same links.
static void large_calls_answer_as_small_ones() {
  gpuos_ctx* c = make(512);
  const uint16_t impls[] = {GPUOS_IMPL_ADD, GPUOS_IMPL_RELU, GPUOS_IMPL_SUM_LAST, GPUOS_IMPL_MAX_LAST, GPUOS_IMPL_SOFTMAX_LAST, GPUOS_IMPL_LAYERNORM_LAST};
  const int arity[] = {2, 1, 1, 1, 1, 3};
  for (int k = 0; k < 6; ++k) CHECK(gpuos_register_op(c, (uint16_t)(20 + k), impls[k], nullptr) == GPUOS_OK);
  uint32_t seed = 12345;
  auto rnd = [&](uint32_t n) { seed = seed * 1664525u + 1013904223u; return (seed >> 8) % n; };
  int refused = 0;
  uint64_t head = 0;
  for (int trial = 0; trial < 600; ++trial) {
    const int k = (int)rnd(6);
    gpuos_task t = add_task((uint16_t)(20 + k), 0);
    t.n_inputs = (uint8_t)arity[k];
    t.ndim = (uint8_t)(1 + rnd(GPUOS_MAX_DIMS));
    const uint8_t dt = (uint8_t)rnd(4) ? GPUOS_F32 : GPUOS_BF16;
    for (int d = 0; d < t.ndim; ++d) t.size[d] = rnd(12) ? 1 + rnd(9) : 0;
    for (int j = 0; j < 4; ++j) {
      auto& q = j < 3 ? t.in[j] : t.out;
      q.ptr = (void*)(uintptr_t)(0x1000000 * (j + 1) + (rnd(3) ? 0 : 4));
      q.dtype = dt;
      int64_t s = 1;
      for (int d = t.ndim - 1; d >= 0; --d) { q.stride[d] = s; s *= t.size[d] ? t.size[d] : 1; }
      if (j < 3 && !rnd(4)) q.stride[rnd(t.ndim)] = 0;
      if (j < 3 && t.ndim > 1 && !rnd(4)) std::swap(q.stride[0], q.stride[1]);
    }
    switch (rnd(24)) {                                    // one fault in half of them
      case 0: t.n_inputs ^= 1; break;
      case 1: t.ndim = 0; break;
      case 2: t.ndim = GPUOS_MAX_DIMS + 1; break;
      case 3: t.size[0] = -1; break;
      case 4: t.size[0] = 1ll << 40; break;
      case 5: t.in[0].ptr = nullptr; break;
      case 6: t.out.dtype = GPUOS_I32; break;
      case 7: t.in[0].dtype = 77; break;
      case 8: t.out.stride[0] = 0; break;
      case 9: t.op_id = 60; break;
      case 10: t.flags = 0x80; break;
      case 11: t.dep[1] = 512; break;
      case 12: t.out.ptr = (void*)(uintptr_t)0x900001; break;
      default: break;
    }
    uint64_t tk = 0;
    const int one = gpuos_submit_flush(c, &t, 1, &tk);
    if (one == GPUOS_OK) { CHECK(tk == head); ++head; }
    else ++refused;
    const uint32_t n = 129 + rnd(300);
    std::vector<gpuos_task> v(n, add_task(7, 256));
    v[rnd(n)] = t;
    const int many = gpuos_submit_flush(c, v.data(), n, &tk);
    CHECK(many == one);
    if (many == GPUOS_OK) { CHECK(tk == head); head += n; }
    gpuos_queue_state q;
    CHECK(gpuos_peek_queue(c, &q) == GPUOS_OK && q.head_submitted == head);
  }
  CHECK(refused > 100 && refused < 500);
  std::vector<gpuos_task> v(300, add_task(7, 256));
  v[5].dep[0] = 511;                                      // one fault of each pass: the earlier pass answers
  CHECK(head >= 511);
  v[299].op_id = 60;
  CHECK(gpuos_submit_flush(c, v.data(), 300, nullptr) == GPUOS_E_BADOP);
  CHECK(gpuos_wait(c, GPUOS_ALL, 0) == GPUOS_OK);
  for (uint32_t n : {129u, 191u, 192u, 193u, 450u}) {     // runs across the ends of batches, and tasks that are none
    std::vector<gpuos_task> w(n, add_task(7, 1000, 1));
    for (uint32_t i = 0; i < n; ++i) { w[i].in[0].ptr = w[i].out.ptr; if (rnd(40) == 0 || i == 0) w[i].dep[0] = 0; }
    const uint64_t a = standin_links();
    CHECK(gpuos_submit(c, w.data(), n, nullptr) == GPUOS_OK && gpuos_flush(c) == GPUOS_OK && gpuos_wait(c, GPUOS_ALL, 0) == GPUOS_OK);
    const uint64_t b = standin_links();
    CHECK(gpuos_submit_flush(c, w.data(), n, nullptr) == GPUOS_OK && gpuos_wait(c, GPUOS_ALL, 0) == GPUOS_OK);
    CHECK(b > a && standin_links() - b == b - a);
  }
  CHECK(gpuos_shutdown(c) == GPUOS_OK);
  CHECK(standin_errors() == 0);
  std::printf("ok: large calls answer as small ones (%d of 600 refused)\n", refused);
}

// What reads past the memory-side cache (RF_STREAM): by the bytes of each operand, in its own dtype, what is broadcast counted once.
static void large_reads_are_marked() {
  gpuos_ctx* c = make(64);
  CHECK(gpuos_register_op(c, 40, GPUOS_IMPL_COPY, nullptr) == GPUOS_OK);
  CHECK(gpuos_register_op(c, 41, GPUOS_IMPL_SUM_LAST, nullptr) == GPUOS_OK);
  CHECK(gpuos_register_op(c, 42, GPUOS_IMPL_EXP, nullptr) == GPUOS_OK);
  struct In { uint8_t dtype; int64_t s0, s1; uint64_t ptr; };
  auto marked = [&](uint16_t op, int64_t rows, int64_t cols, std::vector<In> in, uint8_t out_dtype) {
    gpuos_task t = add_task(op, 1);
    t.ndim = 2; t.n_inputs = (uint8_t)in.size();
    t.size[0] = rows; t.size[1] = cols;
    for (size_t k = 0; k < in.size(); ++k) {
      t.in[k].ptr = (void*)(uintptr_t)in[k].ptr; t.in[k].dtype = in[k].dtype;
      t.in[k].stride[0] = in[k].s0; t.in[k].stride[1] = in[k].s1;
    }
    t.out.ptr = (void*)(uintptr_t)0x90000000; t.out.dtype = out_dtype;
    t.out.stride[0] = op == 41 ? 1 : cols; t.out.stride[1] = op == 41 ? 0 : 1;
    const uint64_t before = standin_streams();
    uint64_t tk = 0;
    CHECK(gpuos_submit_flush(c, &t, 1, &tk) == GPUOS_OK && gpuos_wait(c, tk, 0) == GPUOS_OK);
    return standin_streams() != before;
  };
  const uint64_t A = 0x10000000, B = 0x30000000;
  const int64_t M = 1 << 20;
  // rows of 513: by rows, from 1 MB on
  for (auto rows : {300, 600}) {                          // 0.6 and 1.2 MB of fp32
    const bool big = rows == 600;
    CHECK(marked(7, rows, 513, {{GPUOS_F32, 513, 1, A}, {GPUOS_F32, 0, 1, B}}, GPUOS_F32) == big);           // + a row vector
    CHECK(marked(7, rows, 513, {{GPUOS_F32, 0, 1, B}, {GPUOS_F32, 513, 1, A}}, GPUOS_F32) == big);
    CHECK(marked(7, rows, 513, {{GPUOS_F32, 513, 1, A}, {GPUOS_F32, 1, 0, B}}, GPUOS_F32) == big);           // + a scalar per row
    CHECK(marked(7, 2 * rows, 513, {{GPUOS_BF16, 513, 1, A}, {GPUOS_F32, 1, 0, B}}, GPUOS_BF16) == big);
    CHECK(marked(7, 2 * rows, 513, {{GPUOS_F32, 1, 0, B}, {GPUOS_BF16, 513, 1, A}}, GPUOS_BF16) == big);     // (the first input's dtype is not all there is)
    CHECK(marked(7, rows, 513, {{GPUOS_F32, 513, 1, A + 4}, {GPUOS_F32, 513, 1, B}}, GPUOS_F32));            // two full operands, unaligned
  }
  // contiguous and aligned: from 4 MB on
  CHECK(!marked(7, 1, M / 2 - 4, {{GPUOS_F32, M, 1, A}, {GPUOS_F32, M, 1, B}}, GPUOS_F32));
  CHECK(marked(7, 1, M / 2, {{GPUOS_F32, M, 1, A}, {GPUOS_F32, M, 1, B}}, GPUOS_F32));
  CHECK(!marked(41, 1024, 1020, {{GPUOS_F32, 1020, 1, A}}, GPUOS_F32));
  CHECK(marked(41, 1024, 1024, {{GPUOS_F32, 1024, 1, A}}, GPUOS_F32));
  // EXP, DIV and SUB_EXP, and reductions of rows of up to 64 vectors: from 16 MB on
  CHECK(!marked(42, 1, 4 * M - 4, {{GPUOS_F32, M, 1, A}}, GPUOS_F32) && marked(42, 1, 4 * M, {{GPUOS_F32, M, 1, A}}, GPUOS_F32));
  CHECK(!marked(41, 16383, 256, {{GPUOS_F32, 256, 1, A}}, GPUOS_F32) && marked(41, 16384, 256, {{GPUOS_F32, 256, 1, A}}, GPUOS_F32));
  // casts, by rows whatever their alignment: what is read counts
  CHECK(!marked(40, 1, M / 4 - 8, {{GPUOS_F32, M, 1, A}}, GPUOS_BF16));
  CHECK(marked(40, 1, M / 4, {{GPUOS_F32, M, 1, A}}, GPUOS_BF16));
  CHECK(!marked(40, 1, M / 2 - 8, {{GPUOS_BF16, M, 1, A}}, GPUOS_F32));
  CHECK(marked(40, 1, M / 2, {{GPUOS_BF16, M, 1, A}}, GPUOS_F32));
  CHECK(gpuos_shutdown(c) == GPUOS_OK);
  CHECK(standin_errors() == 0);
  std::printf("ok: large reads are marked\n");
}

// A large call is packed and written while other threads wait, flush, swap and submit: nothing of theirs waits for it but what
// needs the room that it takes.
static void other_calls_pass_a_large_one() {
  using clock = std::chrono::steady_clock;
  auto ms_since = [](clock::time_point t) { return std::chrono::duration<double, std::milli>(clock::now() - t).count(); };
  {                                                       // ... that waits for room on a device that is busy
    gpuos_ctx* c = make(64);
    std::vector<gpuos_task> many(200, add_task(7, 256));
    uint64_t first = ~0ull;
    std::atomic<bool> done{false};
    standin_stall_ms(1500);
    std::thread large([&] { CHECK(gpuos_submit_flush(c, many.data(), 200, &first) == GPUOS_OK); done.store(true); });
    gpuos_queue_state q;
    do CHECK(gpuos_peek_queue(c, &q) == GPUOS_OK); while (q.tail_published < 64);
    std::this_thread::sleep_for(std::chrono::milliseconds(20));
    const auto t0 = clock::now();
    CHECK(gpuos_flush(c) == GPUOS_OK);
    CHECK(gpuos_wait(c, 0, 30ull * 1000 * 1000) == GPUOS_E_TIMEOUT);
    CHECK(gpuos_wait(c, GPUOS_ALL, 30ull * 1000 * 1000) == GPUOS_E_TIMEOUT);
    CHECK(gpuos_swap_op(c, 9, GPUOS_IMPL_SUB, nullptr) == GPUOS_OK);
    CHECK(ms_since(t0) < 700 && !done.load());
    gpuos_task t = add_task(9, 256, 1);
    uint64_t tk = 0;
    CHECK(gpuos_submit_flush(c, &t, 1, &tk) == GPUOS_OK && tk == 200);       // (waits for its room)
    large.join();
    CHECK(first == 0 && gpuos_wait(c, GPUOS_ALL, 0) == GPUOS_OK);
    std::vector<gpuos_completion> comp(201);
    CHECK(gpuos_get_completions(c, 0, 201, comp.data()) == GPUOS_OK);
    for (uint64_t i = 0; i <= 200; ++i) CHECK(comp[i].ticket == i && comp[i].status == 0 && comp[i].op_version == (i < 200 ? 1u : 2u));
    CHECK(gpuos_shutdown(c) == GPUOS_OK);
  }
  {                                                       // ... that is being written: a call behind it returns first
    gpuos_ctx* c = make(65536);
    std::vector<gpuos_task> many(60000, add_task(7, 256));
    uint64_t head = 0;
    bool passed = false;
    for (int trial = 0; trial < 20 && !passed; ++trial) {
      std::atomic<bool> done{false};
      std::thread large([&] { uint64_t tk = 0; CHECK(gpuos_submit_flush(c, many.data(), 60000, &tk) == GPUOS_OK && tk == head); done.store(true); });
      gpuos_queue_state q;
      do CHECK(gpuos_peek_queue(c, &q) == GPUOS_OK); while (q.head_submitted == head);
      gpuos_task t[3] = {add_task(9, 256, 1), add_task(9, 256, 1), add_task(9, 256, 1)};
      uint64_t tk = 0;
      CHECK((trial & 1 ? gpuos_submit(c, t, 3, &tk) : gpuos_submit_flush(c, t, 3, &tk)) == GPUOS_OK && tk == head + 60000);
      passed = !done.load();
      CHECK(gpuos_wait(c, tk + 2, 0) == GPUOS_OK);
      large.join();
      head += 60003;
    }
    CHECK(passed);
    CHECK(gpuos_wait(c, GPUOS_ALL, 0) == GPUOS_OK);
    CHECK(gpuos_shutdown(c) == GPUOS_OK);
  }
  {                                                       // ... that gives up: what is written keeps its tickets
    gpuos_config cfg;
    gpuos_default_config(&cfg);
    cfg.wait_timeout_ms = 400;
    gpuos_ctx* c = nullptr;
    CHECK(gpuos_init(&c, 64, &cfg) == GPUOS_OK);
    CHECK(gpuos_register_op(c, 7, GPUOS_IMPL_ADD, nullptr) == GPUOS_OK);
    std::vector<gpuos_task> many(200, add_task(7, 256));
    uint64_t tk = ~0ull;
    standin_stall_ms(1600);
    CHECK(gpuos_submit_flush(c, many.data(), 200, &tk) == GPUOS_E_TIMEOUT && tk == 0);
    gpuos_queue_state q;
    CHECK(gpuos_peek_queue(c, &q) == GPUOS_OK && q.head_submitted == 64 && q.tail_published == 64);
    CHECK(gpuos_wait(c, GPUOS_ALL, 5000ull * 1000 * 1000) == GPUOS_OK);
    standin_leave_before(150);                            // (64 are done)
    CHECK(gpuos_submit_flush(c, many.data(), 200, &tk) == GPUOS_E_DEAD && tk == 64);
    CHECK(gpuos_peek_queue(c, &q) == GPUOS_OK && q.completed == 150 && q.head_submitted >= 150 && q.head_submitted <= 150 + 64);
    CHECK(q.tail_published == q.head_submitted);
    CHECK(gpuos_start_worker(c) == GPUOS_OK);
    CHECK(gpuos_submit_flush(c, many.data(), 200, &tk) == GPUOS_OK && tk == q.head_submitted);
    CHECK(gpuos_wait(c, GPUOS_ALL, 5000ull * 1000 * 1000) == GPUOS_OK);
    CHECK(gpuos_shutdown(c) == GPUOS_OK);
  }
  CHECK(standin_errors() == 0);
  std::printf("ok: other calls pass a large one\n");
}

// Producers of small and of large calls, waits and swaps beside them: every ticket once, in one piece per call, versions in order.
static void large_and_small_producers() {
  for (uint32_t cap : {64u, 512u, 4096u})
    for (int harv = 0; harv < 2; ++harv) {
      gpuos_ctx* c = make(cap, false, harv != 0);
      const int n_threads = 4, per_thread = 6000;
      std::vector<std::vector<std::pair<uint64_t, uint32_t>>> calls(n_threads);
      std::vector<std::thread> th;
      std::atomic<int> failures{0}, running{n_threads};
      for (int k = 0; k < n_threads; ++k)
        th.emplace_back([&, k] {
          unsigned s = 71u * (unsigned)k + 5u;
          uint32_t left = per_thread;
          while (left > 0) {
            s = s * 1664525u + 1013904223u;
            uint32_t m = k % 2 ? 129 + (s >> 16) % 400u : 1 + (s >> 16) % 5u;
            if (m > left) m = left;
            std::vector<gpuos_task> v(m, add_task(9, 300 + (s >> 20), 1));
            v[0].dep[0] = 0;
            for (uint32_t i = 0; i < m; i += 1 + (s >> 28)) v[i].op_id = 7;
            uint64_t first = ~0ull;
            if (((s >> 4) % 3u ? gpuos_submit_flush(c, v.data(), m, &first) : gpuos_submit(c, v.data(), m, &first)) != GPUOS_OK) { failures++; break; }
            calls[k].push_back({first, m});
            if ((s >> 8) % 7u == 0 && gpuos_wait(c, first + m - 1, 0) != GPUOS_OK) { failures++; break; }
            left -= m;
          }
          running--;
        });
      uint32_t v = 1;
      std::vector<uint64_t> own;
      while (running.load() > 0) {
        CHECK(gpuos_swap_op(c, 7, v % 2 ? GPUOS_IMPL_SUB : GPUOS_IMPL_ADD, &v) == GPUOS_OK);
        gpuos_task t = add_task(7, 256);
        own.push_back(0);
        CHECK(gpuos_submit_flush(c, &t, 1, &own.back()) == GPUOS_OK);
        // (the stand-in has read this version then, and reads no entry while the next is written)
        CHECK((v % 2 ? gpuos_wait(c, own.back(), 0) : gpuos_wait(c, GPUOS_ALL, 0)) == GPUOS_OK);
      }
      for (auto& t : th) t.join();
      CHECK(failures.load() == 0);
      CHECK(gpuos_wait(c, GPUOS_ALL, 0) == GPUOS_OK);
      const uint64_t total = (uint64_t)n_threads * per_thread + own.size();
      std::vector<int> seen(total, 0);
      for (uint64_t t : own) { CHECK(t < total); seen[t]++; }
      for (auto& q : calls) for (auto& f : q) for (uint64_t t = f.first; t < f.first + f.second; ++t) { CHECK(t < total); seen[t]++; }
      for (uint64_t t = 0; t < total; ++t) CHECK(seen[t] == 1);
      gpuos_queue_state q;
      CHECK(gpuos_peek_queue(c, &q) == GPUOS_OK && q.head_submitted == total && q.tail_published == total && q.completed == total);
      std::vector<gpuos_completion> comp(total);
      CHECK(gpuos_get_completions(c, 0, (uint32_t)total, comp.data()) == GPUOS_OK);
      uint32_t last = 1;
      for (uint64_t t = 0; t < total; ++t) {
        CHECK(comp[t].ticket == t && comp[t].status == 0 && comp[t].t_done_ns >= comp[t].t_submit_ns);
        if (comp[t].op_version != 1) { CHECK(comp[t].op_version >= last); last = comp[t].op_version; }
      }
      uint64_t n_log = 0;
      CHECK(gpuos_audit_log(c, 0, 0, nullptr, &n_log) == GPUOS_OK);
      std::vector<gpuos_audit_record> log(n_log);
      CHECK(gpuos_audit_log(c, 0, (uint32_t)n_log, log.data(), nullptr) == GPUOS_OK);
      // (operator 9 keeps version 1; a task of operator 7 from a swap's ticket on has that version or a later one)
      for (size_t i = 1; i < log.size(); ++i) {
        CHECK(log[i].head_ticket >= log[i - 1].head_ticket);
        if (log[i].kind == GPUOS_AUDIT_SWAP)
          for (uint64_t t = log[i].head_ticket; t < total && t < log[i].head_ticket + 600; ++t) CHECK(comp[t].op_version == 1 || comp[t].op_version >= log[i].version);
      }
      CHECK(gpuos_shutdown(c) == GPUOS_OK);
      CHECK(standin_errors() == 0);
    }
  std::printf("ok: producers of small and of large calls\n");
}

int main() {
  check_word_rejects_mixtures();
  block_cuts_stay_below_the_offset_that_does_nothing();
  runs_are_marked();
  chunks_stay_addressable();
  large_calls_answer_as_small_ones();
  large_reads_are_marked();
  other_calls_pass_a_large_one();
  large_and_small_producers();
  // 1. many producers, tiny rings: every ticket exactly once, consecutive inside a call, in-order log
  for (uint32_t cap : {2u, 8u, 64u}) {
    for (int harv = 0; harv < 2; ++harv) {
      gpuos_ctx* c = make(cap, false, harv != 0);
      const int n_threads = 6, per_thread = 3000;
      std::vector<std::vector<uint64_t>> firsts(n_threads);
      std::vector<std::thread> th;
      std::atomic<int> failures{0};
      for (int k = 0; k < n_threads; ++k)
        th.emplace_back([&, k] {
          unsigned s = 17u * (unsigned)k + 1u;
          int left = per_thread;
          while (left > 0) {
            s = s * 1664525u + 1013904223u;
            int m = 1 + (int)((s >> 16) % 5u);
            if (m > left) m = left;
            gpuos_task batch[5];
            for (int i = 0; i < m; ++i) batch[i] = add_task(k % 2 ? 7 : 9, 1000 + (uint32_t)i, i > 0 ? 1 : 0);   // chain inside the call
            uint64_t first = ~0ull;
            // (every third call as submit + flush in one: records and doorbell leave with one flush)
            const int rc = (s >> 4) % 3u == 0 ? gpuos_submit_flush(c, batch, (uint32_t)m, &first) : gpuos_submit(c, batch, (uint32_t)m, &first);
            if (rc != GPUOS_OK) { failures++; return; }
            for (int i = 0; i < m; ++i) firsts[k].push_back(first + (uint64_t)i);
            if ((s >> 8) % 7u == 0 && gpuos_wait(c, first + (uint64_t)m - 1, 0) != GPUOS_OK) { failures++; return; }
            if ((s >> 8) % 11u == 0) gpuos_flush(c);
            left -= m;
          }
        });
      for (auto& t : th) t.join();
      CHECK(failures.load() == 0);
      CHECK(gpuos_wait(c, GPUOS_ALL, 0) == GPUOS_OK);
      const uint64_t total = (uint64_t)n_threads * per_thread;
      std::vector<int> seen(total, 0);
      for (auto& v : firsts) for (uint64_t t : v) { CHECK(t < total); seen[t]++; }
      for (uint64_t t = 0; t < total; ++t) CHECK(seen[t] == 1);
      std::vector<gpuos_completion> comp(total);
      CHECK(gpuos_get_completions(c, 0, (uint32_t)total, comp.data()) == GPUOS_OK);
      for (uint64_t t = 0; t < total; ++t) {
        CHECK(comp[t].ticket == t && comp[t].status == 0 && comp[t].op_version == 1);
        CHECK(comp[t].t_done_ns >= comp[t].t_submit_ns);
      }
      gpuos_queue_state q;
      CHECK(gpuos_peek_queue(c, &q) == GPUOS_OK);
      CHECK(q.head_submitted == total && q.tail_published == total && q.claimed == total && q.completed == total);
      CHECK(gpuos_worker_alive(c) == 1);
      CHECK(gpuos_shutdown(c) == GPUOS_OK);
      std::printf("ok: %d producers x %d tasks, capacity %u, harvester thread %d\n", n_threads, per_thread, cap, harv);
    }
  }
  // 2. a full ring in non-blocking mode: E_FULL and nothing enqueued; a dependency that reaches
  //    before the first ticket or beyond the ring is rejected
  {
    gpuos_ctx* c = make(4, true);
    gpuos_task five[5];
    for (int i = 0; i < 5; ++i) five[i] = add_task(7, 64);
    uint64_t first = 0;
    CHECK(gpuos_submit(c, five, 5, &first) == GPUOS_E_FULL);
    gpuos_queue_state q;
    CHECK(gpuos_peek_queue(c, &q) == GPUOS_OK && q.head_submitted == 0);
    gpuos_task bad = add_task(7, 64, 1);
    CHECK(gpuos_submit(c, &bad, 1, nullptr) == GPUOS_E_INVAL);          // ticket 0 has nothing before it
    CHECK(gpuos_submit(c, five, 4, &first) == GPUOS_OK && first == 0);
    CHECK(gpuos_wait(c, GPUOS_ALL, 0) == GPUOS_OK);
    bad = add_task(7, 64, 4);
    CHECK(gpuos_submit(c, &bad, 1, nullptr) == GPUOS_E_INVAL);          // back-distance >= capacity
    bad = add_task(200, 64);
    CHECK(gpuos_submit(c, &bad, 1, nullptr) == GPUOS_E_BADOP);          // never registered
    CHECK(gpuos_shutdown(c) == GPUOS_OK);
    std::printf("ok: non-blocking ring, dependency and op-id checks\n");
  }
  // 3. swaps while producers run: versions never go back in ticket order, the kill switch shows,
  //    a swap returns only versions that later tasks observe
  {
    gpuos_ctx* c = make(16);
    std::atomic<bool> stop{false};
    std::atomic<uint64_t> after_swap_first{0};
    std::thread prod([&] {
      gpuos_task t = add_task(7, 128);
      while (!stop.load()) CHECK(gpuos_submit(c, &t, 1, nullptr) == GPUOS_OK);
    });
    uint32_t v = 0;
    for (int i = 0; i < 40; ++i) {
      CHECK(gpuos_swap_op(c, 7, i % 2 ? GPUOS_IMPL_ADD : GPUOS_IMPL_SUB, &v) == GPUOS_OK);
      CHECK(v == (uint32_t)i + 2);
    }
    CHECK(gpuos_swap_op(c, 7, GPUOS_IMPL_RELU, &v) == GPUOS_E_INVAL);   // arity differs
    stop.store(true);
    prod.join();
    gpuos_task t = add_task(7, 128);
    uint64_t tk = 0;
    CHECK(gpuos_submit(c, &t, 1, &tk) == GPUOS_OK);
    CHECK(gpuos_wait(c, tk, 0) == GPUOS_OK);
    std::vector<gpuos_completion> comp(tk + 1);
    // the log holds at least the last 2^20 tickets
    const uint64_t lo = tk + 1 > (1u << 20) ? tk + 1 - (1u << 20) : 0;
    CHECK(gpuos_get_completions(c, lo, (uint32_t)(tk + 1 - lo), comp.data()) == GPUOS_OK);
    for (uint64_t i = 1; i + lo <= tk; ++i) CHECK(comp[i].op_version >= comp[i - 1].op_version);
    CHECK(comp[tk - lo].op_version == 41);
    CHECK(gpuos_kill_op(c, 7, &v) == GPUOS_OK && v == 42);
    CHECK(gpuos_submit(c, &t, 1, &tk) == GPUOS_OK);
    CHECK(gpuos_wait(c, tk, 0) == GPUOS_E_BADOP);
    CHECK(gpuos_wait(c, GPUOS_ALL, 0) == GPUOS_E_BADOP);                // first error, reported once
    CHECK(gpuos_wait(c, GPUOS_ALL, 0) == GPUOS_OK);
    // the audit log has every change, in order: one register (make()), 40 swaps, the kill
    uint64_t total = 0;
    CHECK(gpuos_audit_log(c, 0, 0, nullptr, &total) == GPUOS_OK);
    std::vector<gpuos_audit_record> log(total);
    CHECK(gpuos_audit_log(c, 0, (uint32_t)total, log.data(), nullptr) == GPUOS_OK);
    CHECK(gpuos_audit_log(c, 1, (uint32_t)total, log.data(), nullptr) == GPUOS_E_INVAL);
    size_t swaps = 0, kills = 0, regs = 0;
    uint32_t last_v = 0;
    for (size_t i = 0; i < log.size(); ++i) {
      if (i) CHECK(log[i].t_ns >= log[i - 1].t_ns && log[i].head_ticket >= log[i - 1].head_ticket);
      if (log[i].op_id != 7) { regs += log[i].kind == GPUOS_AUDIT_REGISTER; continue; }
      CHECK(log[i].version == last_v + 1);
      last_v = log[i].version;
      if (log[i].kind == GPUOS_AUDIT_REGISTER) { regs++; CHECK(log[i].version == 1 && log[i].head_ticket == 0); }
      else if (log[i].kind == GPUOS_AUDIT_SWAP) { swaps++; CHECK(log[i].impl_id == (log[i].version % 2 ? GPUOS_IMPL_ADD : GPUOS_IMPL_SUB)); }
      else if (log[i].kind == GPUOS_AUDIT_KILL) { kills++; CHECK(log[i].impl_id == GPUOS_IMPL_FAIL && log[i].version == 42 && log[i].head_ticket == tk); }
    }
    CHECK(swaps == 40 && kills == 1 && regs >= 1 && last_v == 42);
    CHECK(gpuos_shutdown(c) == GPUOS_OK);
    std::printf("ok: 40 swaps under load, kill switch, audit log\n");
  }
  // 4. shutdown with tasks in flight drains them; use after stop is refused; programs are table entries
  {
    gpuos_ctx* c = make(32);
    gpuos_instr code[2] = {{GPUOS_PC_ADD, 0, 0, 1, 0.f}, {GPUOS_PC_MUL, 0, 0, 3, 0.f}};
    uint32_t impl = 0;
    CHECK(gpuos_define_program(c, code, 2, 2, &impl) == GPUOS_OK && impl == GPUOS_IMPL_PROGRAM_BASE);
    CHECK(gpuos_register_op(c, 30, impl, nullptr) == GPUOS_OK);
    CHECK(gpuos_register_op(c, 31, impl + 1, nullptr) == GPUOS_E_BADOP);
    {
      uint64_t total = 0;
      CHECK(gpuos_audit_log(c, 0, 0, nullptr, &total) == GPUOS_OK && total >= 2);
      gpuos_audit_record two[2];
      CHECK(gpuos_audit_log(c, total - 2, 2, two, nullptr) == GPUOS_OK);
      uint64_t h = 0xcbf29ce484222325ull;
      for (size_t b = 0; b < sizeof(code); ++b) h = (h ^ reinterpret_cast<const unsigned char*>(code)[b]) * 0x100000001b3ull;
      CHECK(two[0].kind == GPUOS_AUDIT_DEFINE_PROGRAM && two[0].impl_id == impl && two[0].n_instr == 2 && two[0].n_inputs == 2 && two[0].code_hash == h);
      CHECK(two[1].kind == GPUOS_AUDIT_REGISTER && two[1].op_id == 30 && two[1].impl_id == impl && two[1].code_hash == h && two[1].version == 1);
    }
    code[1].a = 9;
    CHECK(gpuos_define_program(c, code, 2, 2, &impl) == GPUOS_E_INVAL);
    std::vector<gpuos_task> many(500, add_task(30, 4096));
    CHECK(gpuos_submit(c, many.data(), 500, nullptr) == GPUOS_OK);
    CHECK(gpuos_stop_worker(c) == GPUOS_OK);
    gpuos_queue_state q;
    CHECK(gpuos_peek_queue(c, &q) == GPUOS_OK && q.completed == 500);
    CHECK(gpuos_submit(c, many.data(), 1, nullptr) == GPUOS_E_DEAD);
    CHECK(gpuos_worker_alive(c) == 0);
    CHECK(gpuos_shutdown(c) == GPUOS_OK);
    std::printf("ok: shutdown drains, use after stop refused, program ids\n");
  }
  // 5. the worker stopped and started again several times: tickets, the completion log, the
  //    operator table (a swap made while stopped) and the ring position all continue
  for (int harv = 0; harv < 2; ++harv) {
    gpuos_ctx* c = make(8, false, harv != 0);
    uint64_t expect = 0;
    uint32_t v = 0;
    for (int round = 0; round < 5; ++round) {
      std::vector<gpuos_task> some(13 + 7 * round, add_task(7, 256));
      uint64_t first = ~0ull;
      CHECK(gpuos_submit(c, some.data(), (uint32_t)some.size(), &first) == GPUOS_OK && first == expect);
      expect += some.size();
      CHECK(gpuos_start_worker(c) == GPUOS_OK);                          // running: nothing to do
      CHECK(gpuos_stop_worker(c) == GPUOS_OK);                           // drains
      gpuos_queue_state q;
      CHECK(gpuos_peek_queue(c, &q) == GPUOS_OK && q.completed == expect && q.claimed == expect);
      CHECK(gpuos_worker_alive(c) == 0);
      CHECK(gpuos_submit(c, some.data(), 1, nullptr) == GPUOS_E_DEAD);
      CHECK(gpuos_swap_op(c, 7, round % 2 ? GPUOS_IMPL_ADD : GPUOS_IMPL_SUB, &v) == GPUOS_OK && v == (uint32_t)round + 2);
      CHECK(gpuos_start_worker(c) == GPUOS_OK);
      CHECK(gpuos_worker_alive(c) == 1);
      uint64_t tk = 0;
      CHECK(gpuos_submit(c, some.data(), 1, &tk) == GPUOS_OK && tk == expect);
      expect += 1;
      CHECK(gpuos_wait(c, tk, 0) == GPUOS_OK);
      gpuos_completion comp;
      CHECK(gpuos_get_completions(c, tk, 1, &comp) == GPUOS_OK && comp.ticket == tk && comp.op_version == (uint32_t)round + 2);
    }
    CHECK(gpuos_shutdown(c) == GPUOS_OK);
    std::printf("ok: worker stopped and started 5 times, harvester thread %d\n", harv);
  }
  // 5b. an idle exit that races with a submit: the worker leaves without having seen the last
  //     doorbell; the wait says so, and the worker started again executes what was left in the ring
  {
    gpuos_ctx* c = make(16);
    std::vector<gpuos_task> some(10, add_task(7, 256));
    uint64_t tk = 0;
    CHECK(gpuos_submit(c, some.data(), 4, &tk) == GPUOS_OK && tk == 0);
    CHECK(gpuos_wait(c, 3, 0) == GPUOS_OK);
    standin_leave_before(6);                                          // tickets 4, 5 will be served, 6.. not
    CHECK(gpuos_submit(c, some.data(), 10, &tk) == GPUOS_OK && tk == 4);
    CHECK(gpuos_wait(c, 5, 0) == GPUOS_OK);
    CHECK(gpuos_wait(c, GPUOS_ALL, 0) == GPUOS_E_DEAD);
    CHECK(gpuos_worker_alive(c) == 0);
    gpuos_queue_state q;
    CHECK(gpuos_peek_queue(c, &q) == GPUOS_OK && q.completed == 6 && q.claimed == 6 && q.head_submitted == 14);
    CHECK(gpuos_start_worker(c) == GPUOS_OK);
    CHECK(gpuos_wait(c, GPUOS_ALL, 0) == GPUOS_OK);
    CHECK(gpuos_peek_queue(c, &q) == GPUOS_OK && q.completed == 14 && q.claimed == 14);
    std::vector<gpuos_completion> comp(14);
    CHECK(gpuos_get_completions(c, 0, 14, comp.data()) == GPUOS_OK);
    for (uint64_t t = 0; t < 14; ++t) CHECK(comp[t].ticket == t && comp[t].status == 0);
    CHECK(gpuos_submit(c, some.data(), 3, &tk) == GPUOS_OK && tk == 14);
    CHECK(gpuos_wait(c, GPUOS_ALL, 0) == GPUOS_OK);
    CHECK(gpuos_shutdown(c) == GPUOS_OK);
    std::printf("ok: tasks stranded by an idle exit are executed after a restart\n");
  }
  // 5c. a wait with a time limit on a device that is busy: GPUOS_E_TIMEOUT, nothing lost, the same
  //     wait without a limit succeeds; a ticket that was never issued is refused
  {
    gpuos_ctx* c = make(16);
    gpuos_task t = add_task(7, 256);
    uint64_t tk = 0;
    standin_stall_ms(400);
    CHECK(gpuos_submit(c, &t, 1, &tk) == GPUOS_OK);
    const auto t0 = std::chrono::steady_clock::now();
    CHECK(gpuos_wait(c, tk, 30ull * 1000 * 1000) == GPUOS_E_TIMEOUT);
    const double waited = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    CHECK(waited > 0.025 && waited < 0.3);
    CHECK(gpuos_worker_alive(c) == 1);
    CHECK(gpuos_wait(c, tk + 1, 0) == GPUOS_E_INVAL);
    CHECK(gpuos_wait(c, tk, 0) == GPUOS_OK);
    CHECK(gpuos_wait(c, GPUOS_ALL, 1) == GPUOS_OK);                     // complete already: no time is needed
    CHECK(gpuos_shutdown(c) == GPUOS_OK);
    std::printf("ok: wait with a time limit\n");
  }
  // 5d. back-pressure that runs into the time limit in the middle of a submit: the records written
  //     before the stall keep their tickets and are executed, the rest were never submitted, and
  //     the next submit continues right after them
  {
    gpuos_config cfg;
    gpuos_default_config(&cfg);
    cfg.wait_timeout_ms = 400;
    gpuos_ctx* c = nullptr;
    CHECK(gpuos_init(&c, 16, &cfg) == GPUOS_OK);
    CHECK(gpuos_register_op(c, 7, GPUOS_IMPL_ADD, nullptr) == GPUOS_OK);
    std::vector<gpuos_task> many(40, add_task(7, 256));
    uint64_t tk = ~0ull;
    standin_stall_ms(1600);
    CHECK(gpuos_submit(c, many.data(), 40, &tk) == GPUOS_E_TIMEOUT);
    CHECK(tk == 0);
    gpuos_queue_state q;
    CHECK(gpuos_peek_queue(c, &q) == GPUOS_OK);
    const uint64_t taken = q.head_submitted - tk;
    CHECK(taken == 16);                                                 // one ring's worth went in before the ring was full
    CHECK(gpuos_wait(c, GPUOS_ALL, 5000ull * 1000 * 1000) == GPUOS_OK);
    std::vector<gpuos_completion> comp(taken);
    CHECK(gpuos_get_completions(c, 0, (uint32_t)taken, comp.data()) == GPUOS_OK);
    for (uint64_t t = 0; t < taken; ++t) CHECK(comp[t].ticket == t && comp[t].status == 0);
    CHECK(gpuos_submit(c, many.data(), 3, &tk) == GPUOS_OK && tk == taken);
    CHECK(gpuos_wait(c, GPUOS_ALL, 5000ull * 1000 * 1000) == GPUOS_OK);
    CHECK(gpuos_shutdown(c) == GPUOS_OK);
    std::printf("ok: a submit that times out under back-pressure keeps what it had written\n");
  }
  // 6. profiler markers: with cfg.markers the calls are annotated through the marker library the
  //    environment names (the test driver points it at a recorder); off by default
  if (std::getenv("GPUOS_ROCTX_LIBRARY")) {
    gpuos_config cfg;
    gpuos_default_config(&cfg);
    CHECK(cfg.markers == 0);
    cfg.markers = 1;
    cfg.wait_timeout_ms = 20000;
    gpuos_ctx* c = nullptr;
    CHECK(gpuos_init(&c, 16, &cfg) == GPUOS_OK);
    uint32_t v = 0;
    CHECK(gpuos_register_op(c, 7, GPUOS_IMPL_ADD, &v) == GPUOS_OK);
    std::vector<gpuos_task> some(5, add_task(7, 256));
    uint64_t tk = 0;
    CHECK(gpuos_submit(c, some.data(), 5, &tk) == GPUOS_OK);
    CHECK(gpuos_wait(c, tk + 4, 0) == GPUOS_OK);
    CHECK(gpuos_swap_op(c, 7, GPUOS_IMPL_SUB, &v) == GPUOS_OK);
    CHECK(gpuos_stop_worker(c) == GPUOS_OK);
    CHECK(gpuos_start_worker(c) == GPUOS_OK);
    CHECK(gpuos_wait(c, GPUOS_ALL, 0) == GPUOS_OK);
    CHECK(gpuos_shutdown(c) == GPUOS_OK);
    std::printf("ok: markers\n");
  }
  // 7. the context that allocates nothing: device-side state in the library's static array, host side
  //    in the caller's block, the caller's stream; one such context per device at a time; the array
  //    is cleared of what the previous context left
  {
    gpuos_config cfg;
    gpuos_default_config(&cfg);
    cfg.wait_timeout_ms = 20000;
    const uint64_t bytes = GPUOS_STATIC_HOST_BYTES(GPUOS_STATIC_MAX_CAPACITY);
    void* block = std::aligned_alloc(256, bytes);
    void* block2 = std::aligned_alloc(256, bytes);
    CHECK(block && block2);
    std::memset(block, 0x5A, bytes);
    hipStream_t st1 = nullptr, st2 = nullptr;
    CHECK(hipStreamCreateWithFlags(&st1, 0) == hipSuccess && hipStreamCreateWithFlags(&st2, 0) == hipSuccess);
    gpuos_ctx* c = nullptr;
    gpuos_ctx* c2 = nullptr;
    CHECK(gpuos_init_static(&c, 2048, &cfg, block, bytes, st1) == GPUOS_E_INVAL && c == nullptr);        // beyond the maximum
    CHECK(std::strstr(gpuos_last_hip_error(), "GPUOS_STATIC_MAX_CAPACITY") != nullptr);
    CHECK(gpuos_init_static(&c, 64, &cfg, block, 1000, st1) == GPUOS_E_INVAL);                           // block too small
    CHECK(gpuos_init_static(&c, 64, &cfg, (char*)block + 8, bytes - 8, st1) == GPUOS_E_INVAL);           // misaligned
    CHECK(gpuos_init_static(&c, 64, &cfg, block, bytes, nullptr) == GPUOS_E_INVAL);                      // no stream
    for (uint32_t cap : {64u, 16u}) {                                                                   // twice in a row, the second one smaller
      standin_scratch_dirty();
      const uint64_t a0 = standin_alloc_calls();
      CHECK(gpuos_init_static(&c, cap, &cfg, block, bytes, st1) == GPUOS_OK && c != nullptr);
      CHECK(standin_alloc_calls() == a0);                                                                // no hipMalloc / hipHostMalloc / stream / event
      CHECK(standin_scratch_nonzero(gpuos::static_layout(cap).total) == 0);                              // what the last context left is gone
      CHECK(gpuos_init_static(&c2, 16, &cfg, block2, bytes, st2) == GPUOS_E_FULL && c2 == nullptr);      // one at a time per device
      CHECK(gpuos_register_op(c, 7, GPUOS_IMPL_ADD, nullptr) == GPUOS_OK);
      std::vector<gpuos_task> some(200, add_task(7, 256));
      uint64_t tk = 0;
      CHECK(gpuos_submit(c, some.data(), 200, &tk) == GPUOS_OK && tk == 0);                              // wraps the ring several times
      CHECK(gpuos_wait(c, GPUOS_ALL, 0) == GPUOS_OK);
      std::vector<gpuos_completion> comp(cap);
      CHECK(gpuos_get_completions(c, 200 - cap, cap, comp.data()) == GPUOS_OK);
      for (uint32_t t = 0; t < cap; ++t) CHECK(comp[t].ticket == 200 - cap + t && comp[t].status == 0 && comp[t].op_version == 1);
      gpuos_queue_state q;
      CHECK(gpuos_peek_queue(c, &q) == GPUOS_OK && q.capacity == cap && q.push_ring == 0 && q.completed == 200);
      CHECK(gpuos_stop_worker(c) == GPUOS_OK);
      float ms = 0;
      CHECK(gpuos_worker_elapsed_ms(c, &ms) == GPUOS_E_INVAL);                                           // no events on such a context
      CHECK(gpuos_start_worker(c) == GPUOS_OK);
      CHECK(gpuos_submit(c, some.data(), 5, &tk) == GPUOS_OK && tk == 200);
      CHECK(gpuos_wait(c, GPUOS_ALL, 0) == GPUOS_OK);
      const uint64_t a1 = standin_alloc_calls();
      CHECK(gpuos_shutdown(c) == GPUOS_OK);
      CHECK(standin_alloc_calls() == a1);                                                                // ... and nothing is freed that was not allocated
      c = nullptr;
    }
    CHECK(hipStreamDestroy(st1) == hipSuccess && hipStreamDestroy(st2) == hipSuccess);
    std::free(block); std::free(block2);
    std::printf("ok: a context that allocates nothing, twice in a row\n");
  }
  CHECK(standin_errors() == 0);
  std::printf("all ok: %llu records through the stand-in, 0 protocol errors\n", (unsigned long long)standin_records());
  return 0;
}
