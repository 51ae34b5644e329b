#define APT_MFMA_DT 1
#define APT_MFMA_DEAL true
#include "apt_mfma.inc"
