// Montgomery form of the CRT halves of the 2048-bit size class.
#define PMK_CLASS_BITS 2048
#include "kmont.inc"
